// Sweep 2 of compression: chunked Huffman bit-packing (the entropy-coding stage of Section 3.1)
// for all tensors of a call, in three launches with no ordering between workgroups:
//
//   k_lengths  the bit count of every chunk and of every range of up to kPackChunks chunks, from the
//              chunks' histograms (the first sweep's running counts) and the code lengths;
//   k_scan     one workgroup per tensor: exclusive prefix sums of the ranges' payload units
//              and outlier counts, the container header, the decision whether it fits;
//   k_pack     the same ranges again: chunk offsets from the range's prefix, the codewords of
//              a chunk (four neighbours merged in registers) OR-ed into a per-wave LDS image at
//              their own bit positions, 128-bit stores; the bit count of every sub-block, which the
//              offsets' prefix sum yields on the way; outlier records of the chunks that hold any.
//
// Where all tensors of the call are small (small_group), k_codebook does the work of the first two.
//
// The symbols are read once, 1 to 2 bytes per element, and packing workgroups never wait for one another:
// every wave walks its own chunks with no workgroup barrier after the offsets are known.  While the bit
// counts came from a pass over the symbols, the ResNet-18-shaped stream (591 M elements) took 138 us for
// them and 240 for the packing, whose symbols that pass had brought nearer; now 35 and 262, and 10 more in
// the first sweep.
#include "cmpz_offsets.h"

#include <type_traits>

namespace cmpz {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves   = kThreads / kWave;
static_assert(kPackChunks <= (uint32_t)kWave, "one lane per chunk of a range");


// LDS written by some lanes of a wave is read by others: the hardware keeps a wave's LDS
// operations in order, this keeps the compiler from moving them across.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The tensor a chunk range belongs to (uniform: scalar loads from the kernel arguments).
__device__ __forceinline__ uint32_t tensor_of_range(const BatchC &b, uint32_t range)
{
    uint32_t ti = 0;
    for (uint32_t k = 1; k < b.n; ++k) if (range >= b.t[k].pack_base) ti = k;
    return ti;
}

__device__ __forceinline__ void unpack8(const uint4 &v, uint32_t s[8])
{
    s[0] = v.x & 0xffffu; s[1] = v.x >> 16; s[2] = v.y & 0xffffu; s[3] = v.y >> 16;
    s[4] = v.z & 0xffffu; s[5] = v.z >> 16; s[6] = v.w & 0xffffu; s[7] = v.w >> 16;
}

// ---------------------------------------------------------------------------
// Bit counts of the chunks, from their histograms: the length of every symbol's code times how
// often it occurs.  A lane holds four neighbouring symbols; a wave takes whole chunks.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void k_lengths(BatchC b)
{
    __shared__ uint32_t lens_s[kMaxSym / 4];         // code length per symbol, one byte each
    __shared__ uint32_t bits_s[kPackChunks];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t range = blockIdx.x;
    const uint32_t ti = tensor_of_range(b, range);
    const TensorC &tc = b.t[ti];
    const uint32_t c0 = (range - tc.pack_base) * b.pack_chunks;
    const uint32_t nq = (tc.nchunks - c0 < b.pack_chunks) ? tc.nchunks - c0 : b.pack_chunks;
    // A wave takes up to kMine consecutive chunks: the rows of these and of the one before, as far as their bytes
    // go, all loads in flight together
    constexpr uint32_t kMine = kPackChunks / kWaves;
    const uint32_t per = b.pack_chunks / kWaves, q0 = wv * per;
    const uint32_t g0 = tc.chunk_base + c0 + q0;     // (rows of chunks that do not exist are not looked at)
    static_assert(kMaxSym / 4 == kThreads, "one word of the length table per thread");
    lens_s[tid] = reinterpret_cast<const uint32_t *>(b.lens + (uint64_t)ti * kMaxSym)[tid];
    __syncthreads();
    ChunkBits cb(b, lens_s, lane);
    uint2 v[kMine + 1] = {};
    uint32_t wq[kMine] = {};
    if (q0 < nq && c0 + q0) v[0] = cb.row(g0 - 1);
#pragma unroll
    for (uint32_t j = 0; j < kMine; ++j) {
        if (j < per && q0 + j < nq) {                // uniform
            v[j + 1] = cb.row(g0 + j);
            wq[j] = cb.is_wide(g0 + j);
        }
    }
#pragma unroll
    for (uint32_t j = 0; j < kMine; ++j) {
        const uint32_t q = q0 + j;
        if (j >= per || q >= nq) break;              // uniform
        const uint32_t tot = cb.chunk(tc, c0 + q, v[j], v[j + 1], uniform_u32(wq[j]) != 0, [&] { return cb.others(g0 + j); });
        if (lane == 63) { bits_s[q] = tot; b.chunk_bits[g0 + j] = tot; }
    }
    __syncthreads();
    if (wv == 0) {
        const uint32_t bits = (lane < (int)nq) ? bits_s[lane] : 0u;
        const uint32_t oc = (lane < (int)nq) ? b.outl_cnt[tc.chunk_base + c0 + lane] : 0u;
        const uint32_t tu = wave_inclusive_sum((bits + 127u) >> 7);
        const uint32_t to = wave_inclusive_sum(oc);
        const uint32_t tb = wave_inclusive_sum(bits);
        if (lane == 63) { b.range_units[range] = tu; b.range_outl[range] = to; b.range_bits[range] = tb; }
    }
}

// ---------------------------------------------------------------------------
// Offsets and header.  One workgroup per tensor turns the ranges' payload units and outlier
// counts into exclusive prefixes (in place), writes the end markers of the two offset tables,
// the zero padding of the outlier sections and the header, and decides whether the container
// fits before any payload is written.
// ---------------------------------------------------------------------------
constexpr int kScanThreads = 1024;

__global__ __launch_bounds__(kScanThreads) void k_scan(BatchC b)
{
    __shared__ uint32_t wave_u[kScanThreads / kWave], wave_o[kScanThreads / kWave];
    __shared__ unsigned long long bits_s;
    __shared__ Header hd_s;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const uint32_t ti = blockIdx.x;
    const TensorC &tc = b.t[ti];
    const uint32_t nr = (tc.nchunks + b.pack_chunks - 1) / b.pack_chunks;
    uint32_t *__restrict__ ru = b.range_units + tc.pack_base;
    uint32_t *__restrict__ ro = b.range_outl + tc.pack_base;
    const uint32_t *__restrict__ rb = b.range_bits + tc.pack_base;
    if (tid == 0) bits_s = 0;
    uint32_t base_u = 0, base_o = 0;
    unsigned long long my_bits = 0;
    for (uint32_t k0 = 0; k0 < nr; k0 += kScanThreads) {            // uniform
        const uint32_t k = k0 + tid;
        const uint32_t u = (k < nr) ? ru[k] : 0u, o = (k < nr) ? ro[k] : 0u;
        if (k < nr) my_bits += rb[k];
        const uint32_t iu = wave_inclusive_sum(u), io = wave_inclusive_sum(o);
        __syncthreads();                                             // the previous round's totals have been read
        if (lane == 63) { wave_u[wv] = iu; wave_o[wv] = io; }
        __syncthreads();
        uint32_t pu = 0, po = 0, tu = 0, to = 0;
#pragma unroll
        for (int w = 0; w < kScanThreads / kWave; ++w) {
            const uint32_t a = wave_u[w], c = wave_o[w];
            if (w < wv) { pu += a; po += c; }
            tu += a; to += c;
        }
        if (k < nr) { ru[k] = base_u + pu + iu - u; ro[k] = base_o + po + io - o; }
        base_u += tu; base_o += to;
    }
    {
        // sum of the ranges' bit counts: 64-bit, one atomic per wave
        const uint32_t lo = wave_inclusive_sum((uint32_t)(my_bits & 0xffffffu));
        const uint32_t mid = wave_inclusive_sum((uint32_t)((my_bits >> 24) & 0xffffffu));
        const uint32_t hi = wave_inclusive_sum((uint32_t)(my_bits >> 48));
        __syncthreads();                                             // bits_s is initialised
        if (lane == 63) atomicAdd(&bits_s, (unsigned long long)lo + ((unsigned long long)mid << 24) + ((unsigned long long)hi << 48));
    }
    __syncthreads();
    finish_container(b, ti, base_u, base_o, bits_s, &hd_s, tid);
}

// ---------------------------------------------------------------------------
// Packing.  A wave packs a chunk in steps of 1024 codes (16 per lane): the lanes' bit offsets come from
// a wave scan of their code lengths, every
// codeword is OR-ed into the wave's zeroed LDS image at its own position (bit k of the chunk is bit
// 31-(k%32) of little-endian word k/32), the 16-byte units that are complete go out with 128-bit
// stores, and the unit that is still open moves to the front of the image for the next step.
//
// A table entry holds 24 bits of a codeword.  A code of 25 bits and more has a share of at most
// 1 / Fibonacci(26) = 8e-6 of the elements, so few steps hold any: such a step puts its codewords into the
// image one by one, from the full codes.  (While a tensor with one codeword of 28 bits or more was packed
// from 64-bit entries throughout, the largest tensor of the ResNet-18-shaped stream, whose codes reach 28
// bits under some seeds, took that launch from 240 to 315 us.)
// ---------------------------------------------------------------------------
constexpr uint32_t kStepBitsMax = 1024 * kMaxCodeLen;
constexpr uint32_t kImageUnits = kStepBitsMax / 128 + 2;               // the open unit in front, one of slack behind
constexpr uint32_t kImageWords = kImageUnits * 4;

// ZB: container version 2; GROUP: lanes of a sub-block (16 codes each)
template <bool ZB, int GROUP>
// Five waves per SIMD: at six the 80 registers spill, which costs more than the sixth wave gives.
__global__ __launch_bounds__(kThreads, 5) void k_pack(BatchC b)
{
    __shared__ uint32_t table[kMaxSym];              // codeword left-aligned (its first 24 bits) | length
    __shared__ uint32_t byte_table[256];             // the same by the byte form: at a constant address, so that a
                                                     // byte becomes its entry's in one instruction
    __shared__ __align__(16) uint32_t images[kWaves][kImageWords];
    __shared__ uint32_t coff_s[kPackChunks], ooff_s[kPackChunks + 1], bits_s[kPackChunks];
    __shared__ uint16_t olists[kWaves][kWave];       // per wave: where in a step the outliers of one pass sit
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t ti = tensor_of_range(b, blockIdx.x);
    const TensorC &tc = b.t[ti];
    const TensorMeta &tm = b.tmeta[ti];
    if (uniform_u32(tm.skip)) return;                // the container does not fit, its header says so
    const uint32_t c0 = (blockIdx.x - tc.pack_base) * b.pack_chunks;
    const uint32_t nq = (tc.nchunks - c0 < b.pack_chunks) ? tc.nchunks - c0 : b.pack_chunks;
    const uint32_t numel = tc.numel;
    const bool long_codes = uniform_u32(tm.max_len) > kEncBits;      // some entries are not whole,
    const uint32_t long_from = uniform_u32(tm.long_from);            // those from here on
    const uint32_t n_outliers = uniform_u32(tm.n_outliers);
    const Layout lay = make_layout(numel, b.radius, b.sub);
    uint8_t *const out = tc.out + uniform_u64(tm.out_off);

    const uint16_t *__restrict__ sym = b.sym + (uint64_t)tc.chunk_base * kChunk;
    // per quarter of the wave's chunks (wv, wv + 4, ...), four bits each: 16-bit symbols, else bytes
    static_assert(kPackChunks <= (uint32_t)kWave, "one lane per quarter of a wave's chunks");
    const uint32_t flag_of = wv + (uint32_t)(lane & ~3);             // (chunk wv + 4 * (lane / 4), quarter lane % 4)
    const unsigned long long wide_mask =
        __ballot(flag_of < nq && b.wide[(uint64_t)(tc.chunk_base + c0 + flag_of) * 4 + (lane & 3)] != 0);
    // The lane's 16 symbols of a quarter, a step's worth: 32 bytes of a wide quarter, 16 of a narrow one.
    // They are fetched while the step before is packed, also across
    // chunks: the first sweep's stores are long gone to memory.
    // (A cache line each fetched a whole chunk ahead: 281 -> 299 us on the ResNet-18-shaped stream.)
    auto fetch = [&](uint32_t q, uint32_t qt, uint4 &a, uint4 &c2) {
        const bool wd = (wide_mask >> ((q & ~3u) + qt)) & 1u;
        const uint8_t *p = reinterpret_cast<const uint8_t *>(sym + (uint64_t)(c0 + q) * kChunk + 1024u * qt) + (((uint32_t)lane * 16u) << (wd ? 1 : 0));
        a = *reinterpret_cast<const uint4 *>(p);
        if (wd) c2 = *reinterpret_cast<const uint4 *>(p + 16u);
    };
    uint4 lo = make_uint4(0, 0, 0, 0), hi = lo;
    if ((uint32_t)wv < nq) fetch(wv, 0, lo, hi);
    const uint32_t *entries = b.enc32 + (uint64_t)ti * kMaxSym;
    for (int k = tid; k < (int)kMaxSym; k += kThreads) table[k] = entries[k];
    static_assert(kThreads == 256, "one byte form per thread");
    byte_table[tid] = entries[b.sym_off + tid];
    uint32_t *img = images[wv];
    uint16_t *olist = olists[wv];
    for (uint32_t k = lane; k < kImageUnits; k += kWave) reinterpret_cast<uint4 *>(img)[k] = make_uint4(0, 0, 0, 0);

    // where the range's chunks and their outlier records start
    if (wv == 0) {
        const uint32_t g = tc.chunk_base + c0 + lane;
        const uint32_t bits = (lane < (int)nq) ? b.chunk_bits[g] : 0u;
        const uint32_t oc = (lane < (int)nq) ? b.outl_cnt[g] : 0u;
        const uint32_t units = (bits + 127u) >> 7;
        const uint32_t cu = b.range_units[blockIdx.x] + wave_inclusive_sum(units) - units;
        const uint32_t co = b.range_outl[blockIdx.x] + wave_inclusive_sum(oc) - oc;
        if (lane < (int)nq) {
            reinterpret_cast<uint32_t *>(out + lay.off_chunk_off)[c0 + lane] = cu;
            reinterpret_cast<uint32_t *>(out + lay.off_outl_off)[c0 + lane] = co;
            coff_s[lane] = cu; bits_s[lane] = bits;
        }
        if (lane <= (int)nq && lane <= (int)kPackChunks) ooff_s[lane] = co;      // lane nq: the end of the last chunk's records
    }
    __syncthreads();
    // ---- from here on the waves are on their own ----

    const float *__restrict__ x = tc.x;
    const uint32_t W = tc.shape[3], HW = tc.shape[2] * W;
    uint4 *__restrict__ payload = reinterpret_cast<uint4 *>(out + lay.off_payload);
    const uint64_t off_outl_idx = lay.off_payload + (uint64_t)uniform_u32(tm.total_units) * 16;
    uint32_t *__restrict__ oidx = reinterpret_cast<uint32_t *>(out + off_outl_idx);
    int32_t *__restrict__ oval = reinterpret_cast<int32_t *>(out + off_outl_idx + ((4ull * n_outliers + 15) & ~15ull));
    bool failed = false;

    for (uint32_t q = wv; q < nq; q += kWaves) {
        const uint32_t c = c0 + q;
        const uint32_t e0 = c * kChunk;
        const bool full = numel - e0 >= kChunk;
        const uint32_t chunk_bits = uniform_u32(bits_s[q]), chunk_units = (chunk_bits + 127u) >> 7;
        uint4 *__restrict__ dst = payload + uniform_u32(coff_s[q]);
        uint32_t orank = uniform_u32(ooff_s[q]);
        const bool has_outl = uniform_u32(ooff_s[q + 1]) != orank;
        uint16_t *__restrict__ sub_bits = reinterpret_cast<uint16_t *>(out + lay.off_sub_bits) + (uint64_t)c * lay.nsub;
        uint32_t bitpos = 0;                         // bits of the chunk packed so far
        uint32_t ubase = 0;                          // units of the chunk stored so far: image unit 0 is stream unit ubase

        // Bits from each lane into offsets in the image.  The scan's first steps leave in a lane the sum over
        // the 2, 4 and 8 lanes that end in it (of its row of 16): the last lane of a sub-block
        // stores the sub-block's bit count from there.
        auto offsets = [&](uint32_t bits, uint32_t i0) -> uint32_t {
            const bool ends = ((uint32_t)lane & (GROUP - 1)) == GROUP - 1;
            uint16_t *at = sub_bits + (i0 - e0) / (16u * GROUP);
            uint32_t inc = bits + dpp_u32<0x111, 0xf>(bits);                           // row_shr:1
            if (GROUP == 2 && ends) *at = (uint16_t)inc;
            inc += dpp_u32<0x112, 0xf>(inc);                                           // row_shr:2
            if (GROUP == 4 && ends) *at = (uint16_t)inc;
            inc += dpp_u32<0x114, 0xf>(inc);                                           // row_shr:4
            if (GROUP == 8 && ends) *at = (uint16_t)inc;
            inc += dpp_u32<0x118, 0xf>(inc);                                           // row_shr:8
            inc += dpp_u32<0x142, 0xa>(inc);                                           // row_bcast:15 into rows 1 and 3
            inc += dpp_u32<0x143, 0xc>(inc);                                           // row_bcast:31 into rows 2 and 3
            const uint32_t pos = bitpos - ubase * 128u + inc - bits;                   // bit position in the image
            bitpos += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
            return pos;
        };
        // up to 64 left-aligned bits into the image
        auto put = [&](uint32_t pos, uint32_t hi, uint32_t lo) {
            const uint32_t o = pos & 31u;
            uint32_t *w = img + (pos >> 5);
            atomicOr(w, hi >> o);
            atomicOr(w + 1, __builtin_amdgcn_alignbit(hi, lo, o));
            atomicOr(w + 2, __builtin_amdgcn_alignbit(lo, 0u, o));           // the part that spills over
        };
        // complete units go out; at the end of the chunk also the open one (zero padded)
        auto flush = [&](bool last) {
            wave_sync();
            uint32_t done = last ? chunk_units : (bitpos >> 7);
            if (done > chunk_units) { done = chunk_units; failed = true; }   // never past the chunk's own units
            const uint32_t nu = done - ubase;
            const bool carry = !last && (bitpos & 127u) != 0;        // uniform
            uint4 open = make_uint4(0, 0, 0, 0);
            if (nu < kImageUnits) {
                for (uint32_t k = lane; k < nu; k += kWave) dst[ubase + k] = reinterpret_cast<const uint4 *>(img)[k];
                if (carry && lane == 0) open = reinterpret_cast<const uint4 *>(img)[nu];
            } else {
                failed = true;                       // cannot happen: a step never holds more than the image
            }
            wave_sync();
            const uint32_t dirty = (nu + 1 < kImageUnits) ? nu + 1 : kImageUnits;
            for (uint32_t k = lane; k < dirty; k += kWave) reinterpret_cast<uint4 *>(img)[k] = make_uint4(0, 0, 0, 0);
            wave_sync();
            if (carry && lane == 0) reinterpret_cast<uint4 *>(img)[0] = open;
            wave_sync();
            ubase = done;
        };

        // one step: the lane's 16 consecutive symbols s[] starting at element i0.  narrow: s[] holds the
        // bytes of a quarter stored with 8 bits per symbol, i.e. symbol - sym_off (no outlier among them)
        auto step = [&](const uint32_t *s, auto narrow_c, uint32_t i0, bool last, auto fetch_next) {
            constexpr int n = 16;
            constexpr bool narrow = decltype(narrow_c)::value;
            const uint32_t zero_sym = narrow ? b.radius - b.sym_off : b.radius;    // the zero residual, as s[] has it
            const uint32_t there = full ? 16u : i0 >= numel ? 0u : numel - i0 < 16u ? numel - i0 : 16u;    // elements that exist
            uint32_t outl = 0;                       // bit k: symbol k is the outlier symbol
            if (!narrow && has_outl) { _Pragma("unroll") for (int k = 0; k < n; ++k) outl |= (s[k] == 0u && (uint32_t)k < there) ? 1u << k : 0u; }
            // version 2: a sub-block of zero residuals (n symbols per lane: sub / n lanes) has no bits
            bool coded = true;
            if (ZB) {
                bool az = true;
                _Pragma("unroll") for (int k = 0; k < n; ++k) az = az && (s[k] == zero_sym || (uint32_t)k >= there);
                coded = !group_all(az, (uint32_t)lane, GROUP);
            }
            uint32_t e[n];
            _Pragma("unroll") for (int k = 0; k < n; ++k) e[k] = narrow ? byte_table[s[k]] : table[s[k]];
            if (!full) { _Pragma("unroll") for (int k = 0; k < n; ++k) e[k] = (uint32_t)k < there ? e[k] : 0u; }
            if (ZB) { _Pragma("unroll") for (int k = 0; k < n; ++k) e[k] = coded ? e[k] : 0u; }
            // Codewords go into the image in groups: two of them (at most 48 bits together) merged
            // in registers cost three LDS atomics, and so do four when they fit 64 bits, which they
            // nearly always do (uniform test over the wave; otherwise two by two).  Sums of entries hold the
            // sums of lengths in their low eight bits, and shifts look at their low six (48 at most) anyway.
            fetch_next();                            // the next step's symbols, now that these are looked up
            // Outlier records: rank the outliers of the step; then one lane per outlier recomputes its residual from x,
            // so that the loads of all of them are in flight together.  Behind the fetch, or the next step would wait
            // for the records' stores as well (63 planes of 1077x630 at eb 7e-4: 88 -> 84 us).
            if (!narrow && has_outl) {
                const uint32_t mine = (uint32_t)__popc(outl);
                const uint32_t inc = wave_inclusive_sum(mine);
                const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
                const uint32_t step0 = i0 - (uint32_t)lane * (uint32_t)n;          // first element of the step
                for (uint32_t r0 = 0; r0 < total; r0 += kWave) {                 // uniform; one pass unless outliers crowd
                    uint32_t rk = inc - mine - r0;                               // place of the lane's next outlier in this pass
                    for (uint32_t rest = outl; rest; rest &= rest - 1u, ++rk)
                        if (rk < (uint32_t)kWave) olist[rk] = (uint16_t)((uint32_t)(lane * n) + (uint32_t)__builtin_ctz(rest));
                    wave_sync();
                    const uint32_t me = r0 + (uint32_t)lane;
                    if (me < total) {
                        const uint32_t i = step0 + olist[lane];
                        const uint32_t p = tc.divHW.div(i);
                        const uint32_t rem = i - p * HW;
                        const uint32_t h = tc.divW.div(rem), w = rem - h * W;
                        const uint32_t at = orank + me;
                        if (at < n_outliers) {
                            oidx[at] = i;
                            oval[at] = delta_from_x(x, i, h, w, W, tc.r);
                        }
                    }
                    wave_sync();
                }
                orank += total;
            }
            uint32_t bits = 0, longest = 0, quad_len[n / 4];
            _Pragma("unroll") for (int k = 0; k < n; k += 4) {
                const uint32_t len = (e[k] + e[k + 1] + e[k + 2] + e[k + 3]) & 0xffu;
                quad_len[k / 4] = len;
                bits += len;
                longest = len > longest ? len : longest;
            }
            uint32_t pos = offsets(bits, i0);
            if (long_codes) {
                uint32_t most = 0;
                _Pragma("unroll") for (int k = 0; k < n; ++k) most = e[k] > most ? e[k] : most;
                if (__any(most >= long_from)) {
                    // (a rolled loop that looks everything up again: small, and nothing has to be kept for it above)
                    const uint4 *mine = reinterpret_cast<const uint4 *>(reinterpret_cast<const uint8_t *>(sym + e0 + ((i0 - e0) & ~1023u)) +
                                                                        (narrow ? 16u : 32u) * lane);
                    const uint32_t count = coded ? there : 0u;
                    uint4 v = mine[0];
#pragma unroll 1
                    for (uint32_t k = 0; k < count; ++k) {
                        if (!narrow && k == 8) v = mine[1];
                        constexpr uint32_t kBits = narrow ? 8u : 16u;
                        const uint32_t sy = v.x & ((1u << kBits) - 1u);
                        v.x = __builtin_amdgcn_alignbit(v.y, v.x, kBits);
                        v.y = __builtin_amdgcn_alignbit(v.z, v.y, kBits);
                        v.z = __builtin_amdgcn_alignbit(v.w, v.z, kBits);
                        v.w >>= kBits;
                        const uint32_t en = narrow ? byte_table[sy] : table[sy];
                        const uint32_t len = en & 0xffu;
                        uint64_t place = (uint64_t)(en & ~0xffu) << 32;              // left-aligned in 64 bits
                        if (len > kEncBits) place = b.codes[(uint64_t)ti * kMaxSym + sy + (narrow ? b.sym_off : 0u)] << (64u - len);
                        put(pos, (uint32_t)(place >> 32), (uint32_t)place);
                        pos += len;
                    }
                    flush(last);
                    return;
                }
            }
            // two codewords, left-aligned in 64 bits
            auto pair_of = [](uint32_t ea, uint32_t eb) -> uint64_t {
                const uint64_t second = ((uint64_t)(eb & ~0xffu) << 32) >> (ea & 63u);
                return second | ((uint64_t)(ea & ~0xffu) << 32);
            };
            if (!__any(longest > 64u)) {
                _Pragma("unroll") for (int k = 0; k < n; k += 4) {
                    const uint64_t quad = pair_of(e[k], e[k + 1]) | (pair_of(e[k + 2], e[k + 3]) >> ((e[k] + e[k + 1]) & 63u));
                    put(pos, (uint32_t)(quad >> 32), (uint32_t)quad);
                    pos += quad_len[k / 4];
                }
            } else {
                _Pragma("unroll") for (int k = 0; k < n; k += 2) {
                    const uint64_t pair = pair_of(e[k], e[k + 1]);
                    put(pos, (uint32_t)(pair >> 32), (uint32_t)pair);
                    pos += (e[k] + e[k + 1]) & 0xffu;
                }
            }
            flush(last);
        };

#pragma unroll 1
        for (uint32_t it = 0; it < 4; ++it) {
            const uint32_t i0 = e0 + it * 1024u + (uint32_t)lane * 16u;
            const bool wide = (wide_mask >> ((q & ~3u) + it)) & 1u;
            auto fetch_next = [&]() {
                if (it < 3) fetch(q, it + 1, lo, hi);
                else if (q + kWaves < nq) fetch(q + kWaves, 0, lo, hi);
            };
            uint32_t s[16];
            if (wide) {
                unpack8(lo, s); unpack8(hi, s + 8);
                if (!full) {                     // (past the end stands whatever was there)
#pragma unroll
                    for (int k = 0; k < 16; ++k) s[k] &= kMaxSym - 1u;
                }
                step(s, std::false_type{}, i0, it == 3, fetch_next);
            } else {
                const uint32_t w4[4] = {lo.x, lo.y, lo.z, lo.w};
#pragma unroll
                for (int k = 0; k < 16; ++k) s[k] = (w4[k >> 2] >> (8 * (k & 3))) & 0xffu;
                step(s, std::true_type{}, i0, it == 3, fetch_next);
            }
        }
        if (bitpos != chunk_bits) failed = true;      // the two passes disagree: cannot happen
    }
    if (failed && lane == 0) atomicOr(b.status, kStInternal);
}

// What the first sweep accumulates for the tensors of a group, back to zero (a compress that was
// begun and cannot be finished, or scratch of unknown content).
__global__ __launch_bounds__(kThreads) void k_clear(BatchC b)
{
    const uint32_t ti = blockIdx.x;
    uint32_t *h = b.hist + (uint64_t)ti * kHistCopies * kMaxSym;
    for (uint32_t k = threadIdx.x; k < kHistCopies * kMaxSym; k += kThreads) h[k] = 0;
    if (threadIdx.x == 0) b.tmeta[ti].range_events = 0;
}

// Quarter chunks stored with 8 bits per symbol, rewritten in place with 16 (for inspection of the
// symbols).  One workgroup of 64 threads per quarter.
__global__ __launch_bounds__(64) void k_widen(uint16_t *sym, uint32_t *wide, uint32_t sym_off)
{
    const uint32_t qd = blockIdx.x, lane = threadIdx.x;
    if (wide[qd]) return;                            // uniform
    uint16_t *slot = sym + (uint64_t)qd * 1024u;
    const uint4 v = *reinterpret_cast<const uint4 *>(reinterpret_cast<const uint8_t *>(slot) + 16u * lane);
    __syncthreads();                                 // every byte is read before the slot is overwritten
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    uint32_t o[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const uint32_t a = ((w[k >> 1] >> (16 * (k & 1))) & 0xffu) + sym_off;
        const uint32_t b2 = ((w[k >> 1] >> (16 * (k & 1) + 8)) & 0xffu) + sym_off;
        o[k] = a | (b2 << 16);
    }
    *reinterpret_cast<uint4 *>(slot + 16u * lane) = make_uint4(o[0], o[1], o[2], o[3]);
    *reinterpret_cast<uint4 *>(slot + 16u * lane + 8u) = make_uint4(o[4], o[5], o[6], o[7]);
    __syncthreads();
    if (lane == 0) wide[qd] = 1;
}

// ---- the stack of containers (one thread each: a few words of bookkeeping) ----
__global__ void k_arena_init(ArenaState *st, uint32_t slots)
{
    st->top = 0; st->peak = 0; st->nslots = 0; st->failed = 0; st->slots_cap = slots; st->pad = 0; st->parts_read.n = 0;
    for (uint32_t k = 0; k < kReaderParts; ++k) st->readers[k].n = 0;
    for (uint32_t k = 0; k < slots; ++k) { st->slot[k].offset = 0; st->slot[k].size = 0; }
}

}  // namespace

void launch_arena_init(ArenaState *st_dev, uint32_t slots, hipStream_t st)
{
    hipLaunchKernelGGL(k_arena_init, dim3(1), dim3(1), 0, st, st_dev, slots);
}
void launch_widen(uint16_t *sym, uint32_t *wide, uint32_t sym_off, uint32_t nchunks, hipStream_t st)
{
    if (nchunks) hipLaunchKernelGGL(k_widen, dim3(4 * nchunks), dim3(64), 0, st, sym, wide, sym_off);
}

void launch_clear(const BatchC &b, Profiler *prof, hipStream_t st)
{
    if (b.n) launch(prof, kKClear, k_clear, dim3(b.n), dim3(kThreads), st, b);
}

// Bit counts, offsets and header (unless the codebook kernel has done these), packing: up to three launches over all
// tensors of the group.
void launch_pack(const BatchC &b, Profiler *prof, hipStream_t st)
{
    if (!small_group(b)) {
        if (b.pack_wgs) launch(prof, kKLengths, k_lengths, dim3(b.pack_wgs), dim3(kThreads), st, b);
        launch(prof, kKScan, k_scan, dim3(b.n), dim3(kScanThreads), st, b);
    }
    if (b.pack_wgs) {
        auto pack = [&](auto group) {
            constexpr int kGroup = decltype(group)::value;
            if (b.zero_blocks) launch(prof, kKPack, k_pack<true, kGroup>, dim3(b.pack_wgs), dim3(kThreads), st, b);
            else launch(prof, kKPack, k_pack<false, kGroup>, dim3(b.pack_wgs), dim3(kThreads), st, b);
        };
        switch (b.sub) {
        case 32:  pack(std::integral_constant<int, 2>{}); break;
        case 64:  pack(std::integral_constant<int, 4>{}); break;
        default:  pack(std::integral_constant<int, 8>{}); break;
        }
    }
}

}  // namespace cmpz
