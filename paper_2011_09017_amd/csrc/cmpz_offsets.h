// What turns the first sweep's counts and the code lengths into a container's offsets and header: shared
// by the kernels of large tensors (k_lengths, k_scan) and by the codebook kernel, which does it for small ones.
// Internal to libcmpz.
#pragma once
#include "cmpz_internal.h"

namespace cmpz {

// Bit counts of chunks from the counts that the first sweep left behind each of them (see kRunMax).  A lane
// holds four neighbouring symbols; lens4: the code lengths of all symbols, one byte each, in LDS.
struct ChunkBits {
    const uint2 *byte_rows, *other_rows;             // kByteSyms / 4 and kOtherSyms / 4 per chunk
    const uint32_t *lens4;
    const BatchC &b;
    uint32_t byte_quad;                              // the first four symbols with a byte form
    // Elements that are no other symbol are zero residuals: their code counts for every element, and the
    // other symbols for what their codes are longer.  In container version 2 they are counted.
    int32_t zero_len;
    int lane;
    int32_t others_before = 0;
    bool have_before = false;                        // uniform

    __device__ __forceinline__ ChunkBits(const BatchC &batch, const uint32_t *lens, int ln)
        : byte_rows(reinterpret_cast<const uint2 *>(batch.chunk_hist)), other_rows(reinterpret_cast<const uint2 *>(batch.others_hist)),
          lens4(lens), b(batch), byte_quad(batch.sym_off / 4),
          zero_len(batch.zero_blocks ? 0 : (int32_t)reinterpret_cast<const uint8_t *>(lens)[batch.radius]), lane(ln)
    {
    }
    // the counts of the symbols with a byte form after global chunk g
    __device__ __forceinline__ uint2 row(uint32_t g) const { return byte_rows[(uint64_t)g * 64 + lane]; }

    __device__ __forceinline__ int32_t quad_bits(uint2 n, uint32_t quad) const
    {
        const uint32_t L = lens4[quad];
        return (int32_t)(n.x & 0xffffu) * ((int32_t)(L & 0xffu) - zero_len) + (int32_t)(n.x >> 16) * ((int32_t)((L >> 8) & 0xffu) - zero_len) +
               (int32_t)(n.y & 0xffffu) * ((int32_t)((L >> 16) & 0xffu) - zero_len) + (int32_t)(n.y >> 16) * ((int32_t)(L >> 24) - zero_len);
    }
    // the symbols without a byte form, of the counts after chunk g (the lane's share)
    static constexpr uint32_t kOthers = kOtherSyms / 4 / kWave;
    __device__ __forceinline__ void fetch_others(uint32_t g, uint2 (&n)[kOthers]) const
    {
#pragma unroll
        for (uint32_t i = 0; i < kOthers; ++i) n[i] = other_rows[(uint64_t)g * (kOtherSyms / 4) + i * kWave + lane];
    }
    __device__ __forceinline__ int32_t others_bits(const uint2 (&n)[kOthers]) const
    {
        int32_t bits = 0;
#pragma unroll
        for (uint32_t i = 0; i < kOthers; ++i) {
            const uint32_t at = i * kWave + lane;
            bits += quad_bits(n[i], at < byte_quad ? at : at + kByteSyms / 4);
        }
        return bits;
    }
    __device__ __forceinline__ int32_t others(uint32_t g) const
    {
        uint2 n[kOthers];
        fetch_others(g, n);
        return others_bits(n);
    }
    // does chunk g have quarters of 16-bit symbols?
    __device__ __forceinline__ bool is_wide(uint32_t g) const
    {
        const uint4 f = *reinterpret_cast<const uint4 *>(b.wide + (uint64_t)g * 4);
        return (f.x | f.y | f.z | f.w) != 0;
    }
    // Bits of chunk c of tensor tc, in lane 63: from its row, the row before it, whether it is wide (uniform), and
    // if so the other symbols' bits.  To be called for consecutive chunks.
    template <typename Others>
    __device__ __forceinline__ uint32_t chunk(const TensorC &tc, uint32_t c, uint2 before, uint2 now, bool wide, Others &&others_now)
    {
        const uint32_t g = tc.chunk_base + c;
        const bool first = c % tc.run == 0;          // of its run: nothing to subtract
        int32_t bits = quad_bits(now, byte_quad + lane);
        if (!first) bits -= quad_bits(before, byte_quad + lane);
        if (wide) {
            const int32_t all = others_now();
            bits += all;
            if (!first) bits -= have_before ? others_before : uniform_u32(b.has_others[g - 1]) ? others(g - 1) : 0;
            others_before = all;
        }
        have_before = wide;
        const uint32_t n = (tc.numel - c * kChunk < kChunk) ? tc.numel - c * kChunk : kChunk;
        return wave_inclusive_sum((uint32_t)bits) + n * (uint32_t)zero_len;
    }
};

// The end markers of the two offset tables, the zero padding of the outlier sections, the header, and whether the
// container fits, which is decided before any payload is written; on the device-side stack, its slot.  All
// threads of the workgroup call it; hd is LDS.
__device__ __forceinline__ void finish_container(const BatchC &b, uint32_t ti, uint64_t total_units, uint64_t n_out, uint64_t total_bits,
                                                 Header *hd, int tid)
{
    const TensorC &tc = b.t[ti];
    const Layout lay = make_layout(tc.numel, b.radius, b.sub);
    const OutRef oref = resolve_out(tc);
    const bool fixed_fit = oref.cap >= lay.off_payload;
    if (tid < (int)(kHeaderBytes / 4)) reinterpret_cast<uint32_t *>(hd)[tid] = 0;
    __syncthreads();
    if (tid == 0) {
        TensorMeta &tm = b.tmeta[ti];
        const uint64_t off_outl_idx = lay.off_payload + total_units * 16;
        const uint64_t sect = (4 * n_out + 15) & ~15ull;
        const uint64_t off_outl_val = off_outl_idx + sect;
        const uint64_t total = off_outl_val + sect;
        const bool fits = total <= oref.cap;
        const uint32_t range_events = tm.range_events;

        uint32_t *chunk_off = reinterpret_cast<uint32_t *>(oref.out + lay.off_chunk_off);
        uint32_t *outl_off = reinterpret_cast<uint32_t *>(oref.out + lay.off_outl_off);
        const uint32_t padded = (tc.nchunks + 1 + 3) & ~3u;
        if (fixed_fit) {
            chunk_off[tc.nchunks] = (uint32_t)total_units;
            outl_off[tc.nchunks] = (uint32_t)n_out;
            for (uint32_t k = tc.nchunks + 1; k < padded; ++k) { chunk_off[k] = 0; outl_off[k] = 0; }
        }
        if (fits) {
            uint32_t *oidx = reinterpret_cast<uint32_t *>(oref.out + off_outl_idx);
            uint32_t *oval = reinterpret_cast<uint32_t *>(oref.out + off_outl_val);
            for (uint64_t k = n_out; k < ((n_out + 3) & ~3ull); ++k) { oidx[k] = 0; oval[k] = 0; }
        }

        hd->magic = kMagic; hd->version = b.zero_blocks ? kVersionZB : kVersion; hd->status = fits ? 0u : kStNoSpace;
        hd->eb_bits = tc.eb_bits;
        for (int k = 0; k < 4; ++k) hd->shape[k] = tc.shape[k];
        hd->numel = tc.numel;
        hd->radius = b.radius; hd->chunk = kChunk; hd->sub = b.sub; hd->guard_shift = b.guard_shift;
        hd->nchunks = tc.nchunks; hd->n_outliers = (uint32_t)n_out;
        hd->range_events = range_events; hd->max_len = tc.numel ? tm.max_len : 0u;
        hd->total_bits = total_bits;
        hd->off_lens = lay.off_lens; hd->off_chunk_off = lay.off_chunk_off;
        hd->off_outl_off = lay.off_outl_off; hd->off_sub_bits = lay.off_sub_bits;
        hd->off_payload = lay.off_payload; hd->off_outl_idx = off_outl_idx;
        hd->off_outl_val = off_outl_val; hd->total_size = total;

        uint32_t st = 0;
        if (!fits) st |= kStNoSpace;
        if (range_events) st |= kStRange;
        if (st) atomicOr(b.status, st);
        tm.skip = fits ? 0u : 1u;
        tm.n_outliers = (uint32_t)n_out;
        tm.total_units = (uint32_t)total_units;
        tm.total_bits = total_bits;
        tm.total_size = total;
        tm.out_off = (uint64_t)(oref.out - tc.out);  // (the stack's top moves below)
        tm.range_events = 0;                         // ready for the next call
        if (tc.arena) {
            // the container's slot, and the top of the stack past it (the packing that follows fills it)
            ArenaState *as = tc.arena;
            const uint32_t slot = tc.arena_slot;
            if (slot >= as->slots_cap) {
                as->failed += 1;
            } else {
                as->slot[slot].offset = as->top;
                as->slot[slot].size = fits ? total : 0ull;           // 0: it did not fit, the slot stays empty
                if (fits) {
                    as->top += (total + kArenaAlign - 1) / kArenaAlign * kArenaAlign;
                    if (as->top > as->peak) as->peak = as->top;
                } else {
                    as->failed += 1;
                }
                if (slot + 1 > as->nslots) as->nslots = slot + 1;
            }
        }
    }
    __syncthreads();
    if (fixed_fit && tid < (int)(kHeaderBytes / 4)) reinterpret_cast<uint32_t *>(oref.out)[tid] = reinterpret_cast<const uint32_t *>(hd)[tid];
}

}  // namespace cmpz
