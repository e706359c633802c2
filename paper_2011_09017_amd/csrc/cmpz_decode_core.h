// Huffman decode core shared by the decompression kernels: table layout and the
// per-lane decode loop.  Internal to libcmpz.
//
// One lookup table, indexed by where the next 32 bits of the stream lie in the left-aligned code space.  Canonical
// codes grow with their length when left-aligned, so a code of L bits starts where about 2^-L times the codes of its
// length are left of the space, and on a logarithmic scale of x, how far the bits lie below the top of the space,
// an entry is about as wide as the code whatever its length: 2^m entries for every power of two of x.  The conversion
// of x to floating point is the logarithm: its exponent and the first m bits of its mantissa, less those of the
// smallest number of the scale, are the index.  Every codebook takes one of five scales, by what they leave of the
// code space to the search below and by what their index costs (build_tables):
//   x, m = 7      codes of up to 24 bits: steep codebooks
//   x + 2^j, (j, m) = (24, 8)   codes of up to 16 bits in the upper 256th of the space, of fewer below
//                     (28, 9)   13 bits in the upper sixteenth, fewer below
//                     (30, 10)  every code of up to 12 bits: of at most 1024 codes those of 11 bits lie in the upper half of
//                               the space and those of 12 in its upper quarter
//                     (32, 11)  linear: every code of up to 11 bits
// Share of the code space left to the search, with 2048 + 256 linear entries in two levels / with these five: eb 1e-2
// 0.0003 / 0.00001, eb 1e-3 0.02 / below 0.0006, eb 5e-4 (codes of 10 to 12 bits) 0 / 0.  Restored in us, two levels / five scales:
// 64x256x56x56 at eb 5e-3 with 128 codes per sub-block 214 / 149; 128x96x55x55 at eb 1e-3 with 32 codes 150 / 82 (90 with m = 8 on x
// itself, which leaves 0.002), with 128 316 / 200; 3x256x51x53 at eb 5e-4 with 128 codes 55 / 51 (91 on the linear scale).
// Whatever the table leaves is found by canonical search: decode_lds compares with the limits in range[]
// for lengths below 32 and from there on with first[], as decode_run does for all of them.
#pragma once
#include "cmpz_internal.h"

namespace cmpz {

constexpr uint32_t kTableSize = 2304;        // entries: 4608 bytes of LDS, with the fused decoder's other arrays five
                                             // workgroups just fit a CU
constexpr uint32_t kLinearBits = 11;         // of the index on a linear scale (2048 entries)
// Bits of x that the index looks at: as many as keep the conversion, and the sum with 2^j, exact (24 bits)
constexpr uint32_t kLog7Mask = ~0xffu, kOffsetMask = ~0x1ffu;
constexpr uint32_t kPowers7 = 17;            // powers of two there (entries no narrower than kLog7Mask allows)

// Table entries: symbol in bits 0..9, code length in bits 10..15; 0 = not resolved here.
struct DecodeTables {
    uint16_t entry[kTableSize];
    uint32_t sorted3[(kMaxSym + 2) / 3];   // symbols ordered by (length, symbol), each as its residual
                                  // (symbol - radius) in 10 bits, two's complement, three to a word
                                  // (read only for codewords that the table does not resolve)
    uint64_t first[kMaxCodeLen + 2];   // first canonical code of each length (indexed by the length)
    // Per length, side by side so that the search takes both with one access:
    //   .x  largest left-aligned 32-bit value that belongs to a code of at most that length (exact up to 32
    //       bits, and from the length of the shortest code on; rounded down beyond: no limit to search by)
    //   .y  what turns a code of that length into its index in the ordered symbols (mod 2^32)
    uint2    range[kMaxCodeLen + 2];
    uint32_t scale_min;           // the smallest number of the scale, as the bits of a float
    uint32_t scale_shift;         // 23 - m
    float    offset;              // 2^j, or 0
    uint32_t from;                // shortest length that the table leaves to the search, for some of its codes
    uint32_t max_len;
    uint32_t payload_units;
    uint32_t n_outliers;
};

// Entry i of the symbols ordered by (length, symbol).
__device__ __forceinline__ uint32_t sorted_at(const DecodeTables &T, uint32_t i)
{
    const uint32_t w = i / 3u;
    return (T.sorted3[w] >> (10u * (i - 3u * w))) & 1023u;
}

// Codes of length L: the first code of the next length is twice the one after the last of these.
__device__ __forceinline__ uint64_t codes_of_length(const DecodeTables &T, uint32_t L)
{
    return (T.first[L + 1] >> 1) - T.first[L];
}

// Cooperative copy global -> LDS (both are the same struct).
__device__ __forceinline__ void load_tables(DecodeTables &dst, const DecodeTables *__restrict__ src, int tid,
                                            int nthreads)
{
    static_assert(sizeof(DecodeTables) % 4 == 0, "copied as words");
    const uint32_t *s = reinterpret_cast<const uint32_t *>(src);
    uint32_t *d = reinterpret_cast<uint32_t *>(&dst);
    for (uint32_t k = tid; k < sizeof(DecodeTables) / 4; k += nthreads) d[k] = s[k];
}

// Validation of the container header and code lengths, and construction of the decode tables
// in LDS, by one workgroup of NT >= 256 threads (every workgroup of the fused decode kernel does
// this for itself, and no separate kernel or round trip through memory).  10 400 clock cycles, 4.3 us, of which 1900 until the
// code lengths are here; latencies bound it, so a thread looks up its nine entries side by side, the waves evaluate a
// scale each, and the header's check has a wave of its own (12 400 with that check before the ranks, one more barrier and the
// shares in 64 bits; 17 300 with one entry after the other, all scales in one wave and a pass per length for the ranks:
// 1x64x56x56 17.3 / 15.3 / 14.5 us).
// `scratch` is LDS the caller does not need yet (at least 12 KB; the ordered symbols are laid out
// there as 16-bit values while the tables are filled).  Returns 0 or the status bits
// of the defect found; contains barriers, so all NT threads must call it.
//
// Canonical codes are ascending in (length, symbol) when left-aligned, so with
//   s[l] = count[l] << (48 - l)  and  P[l] = sum of s[j] over 1 <= j < l
// the first code of length l is P[l] >> (48 - l), the code is complete iff the total is 2^48,
// and a left-aligned value v belongs to the shortest length l with v < P[l+1].
template <int NT>
__device__ __forceinline__ uint32_t build_tables(DecodeTables &T, const DecompressArgs &a, uint32_t *scratch)
{
    static_assert(NT == 256 && kTableSize % NT == 0, "four waves: four symbols and nine entries per thread");
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    Header *hd = reinterpret_cast<Header *>(scratch);                 // 64 words
    uint32_t *ends = scratch + 64;                                    // 4 words
    uint32_t *bad_s = scratch + 68, *bad2_s = scratch + 69;       // defects found in the header or in a length / in the lengths together
    uint32_t *used_s = scratch + 70;
    uint32_t *lim = scratch + 72;                                     // 64: P[l+1] in units of 2^-32, below 2^32
    uint32_t *left_s = scratch + 136;                                 // per scale: share of the code space left to the search, 2^-31
    uint32_t *from_s = scratch + 144;                                 // per scale: the shortest length that has some of it; 0: none
    uint32_t (*wave_cnt)[64] = reinterpret_cast<uint32_t (*)[64]>(scratch + 200);   // 16 x 64: [pass*4 + wave][length]
    uint16_t *sorted = reinterpret_cast<uint16_t *>(scratch + 1224);  // kMaxSym x u16
    uint32_t (*wave_off)[64] = reinterpret_cast<uint32_t (*)[64]>(scratch + 1736);  // the same: symbols in earlier passes and waves
    const uint32_t nsym = 2 * a.radius;

    bool bad_here = false;                                            // the reserved tail of the header must be zero
    if (tid < (int)(kHeaderBytes / 4)) {
        const uint32_t v = reinterpret_cast<const uint32_t *>(a.buf)[tid];
        scratch[tid] = v;
        bad_here = tid >= (int)(offsetof(Header, zero) / 4) && v != 0;
    }
    if (tid >= 64 && tid < 68) {
        const uint32_t *chunk_off = reinterpret_cast<const uint32_t *>(a.buf + a.lay.off_chunk_off);
        const uint32_t *outl_off = reinterpret_cast<const uint32_t *>(a.buf + a.lay.off_outl_off);
        const int k = tid - 64;
        ends[k] = (k == 0) ? chunk_off[0] : (k == 1) ? chunk_off[a.lay.nchunks] : (k == 2) ? outl_off[0] : outl_off[a.lay.nchunks];
    }
    if (tid == 68) { *bad_s = 0; *bad2_s = 0; }
    // code lengths, 4 symbols per thread (symbol q*256 + tid)
    const uint32_t padded = (nsym + 15u) & ~15u;
    uint32_t L[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t k = q * 256u + tid;
        uint32_t v = 0;
        if (k < padded) v = a.buf[a.lay.off_lens + k];
        if ((k >= nsym && v) || v > kMaxCodeLen) { bad_here = true; v = 0; }
        L[q] = v;
    }
    // rank of every symbol among the symbols of its length in its wave and pass (the wave's own rows: no barrier)
    uint32_t in_wave[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        wave_cnt[q * 4 + wv][lane] = 0;
        in_wave[q] = 0;
        if (!__any(L[q] != 0)) continue;                              // (uniform; a small tensor's symbols lie close together)
        unsigned long long same = ~0ull;                              // the lanes with this length
#pragma unroll
        for (uint32_t k = 0; k < 6; ++k) {
            const bool set = (L[q] >> k) & 1u;
            const unsigned long long those = __ballot(set);
            same &= set ? those : ~those;
        }
        in_wave[q] = (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");        // (the row is cleared)
        if (L[q] && in_wave[q] == 0) wave_cnt[q * 4 + wv][L[q]] = (uint32_t)__popcll(same);
    }
    __syncthreads();
    if (bad_here) atomicOr(bad_s, kStFormat);

    // Every wave, lane = length: totals per length, the part of the code space of every length.  Wave 0 writes them down.
    {
        uint32_t cnt = 0;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const uint32_t c = wave_cnt[k][lane];
            wave_off[k][lane] = cnt;                                  // (every wave, the same)
            cnt += c;
        }
        const uint32_t sum = wave_inclusive_sum(cnt);
        const uint32_t offs = sum - cnt, used = (uint32_t)__builtin_amdgcn_readlane((int)sum, 63);
        // s < 2^58: three limbs of 24 bits, each scanned in 32 bits without overflow
        const uint64_t sl = (lane >= 1 && lane <= (int)kMaxCodeLen) ? ((uint64_t)cnt << (kMaxCodeLen - lane)) : 0ull;
        const uint32_t i0 = wave_inclusive_sum((uint32_t)(sl & 0xffffffu));
        const uint32_t i1 = wave_inclusive_sum((uint32_t)((sl >> 24) & 0xffffffu));
        const uint32_t i2 = wave_inclusive_sum((uint32_t)(sl >> 48));
        const uint64_t incl = (uint64_t)i0 + ((uint64_t)i1 << 24) + ((uint64_t)i2 << 48);
        const uint64_t excl = incl - sl, one = 1ull << kMaxCodeLen;
        if (wv == 0) {
            const unsigned long long present = __ballot(cnt != 0);
            const uint32_t max_len = present ? 63u - (uint32_t)__builtin_clzll(present) : 0u;
            const uint64_t first = (lane >= 1 && lane <= (int)kMaxCodeLen) ? (excl >> (kMaxCodeLen - lane)) : 0ull;
            if (lane <= (int)kMaxCodeLen) {
                T.first[lane] = first;
                T.range[lane] = make_uint2((uint32_t)(incl >> (kMaxCodeLen - 32)) - 1u, offs - (uint32_t)first);
            }
            if (lane == (int)kMaxCodeLen) T.first[lane + 1] = (first + cnt) << 1;
            // (the top of the space is 2^32 here: one less is above every entry's smallest value too)
            lim[lane] = incl < one ? (uint32_t)(incl >> (kMaxCodeLen - 32)) : 0xffffffffu;
            if (lane == 63) {
                uint32_t bad = 0;
                if (used >= 2 && incl != one) bad = kStFormat;
                if (used == 1 && max_len != 1) bad = kStFormat;
                // no codeword at all: an empty tensor, or (version 2) nothing but sub-blocks of zero residuals
                if (used == 0 && a.numel != 0 && !(a.zero_blocks && hd->total_bits == 0)) bad = kStFormat;
                if (hd->max_len != max_len) bad = kStFormat;
                if (bad) *bad2_s = bad;
                *used_s = used;
                T.max_len = max_len;
            }
            const unsigned long long beyond = __ballot(cnt != 0 && lane > (int)kLinearBits);
            if (lane == (int)kLinearBits) {
                left_s[4] = incl < one ? (uint32_t)((one - incl) >> (kMaxCodeLen - 31)) : 0u;
                from_s[4] = beyond ? (uint32_t)__ffsll((long long)beyond) - 1u : 0u;
            }
        }
        if (tid == 192) {
            uint32_t bad = 0;
            const Layout &l = a.lay;
            if (hd->magic != kMagic || (hd->version != kVersion && hd->version != kVersionZB) || hd->status != 0) bad = kStFormat;
            if (!bad) {
                if (hd->eb_bits != a.eb_bits) bad = kStMismatch;
                if (hd->version != (a.zero_blocks ? kVersionZB : kVersion)) bad = kStMismatch;
                for (int k = 0; k < 4; ++k) if (hd->shape[k] != a.shape[k]) bad = kStMismatch;
                if (hd->radius != a.radius || hd->chunk != kChunk || hd->sub != a.sub ||
                    hd->guard_shift != a.guard_shift) bad = kStMismatch;
            }
            if (!bad) {
                const uint64_t n_out = hd->n_outliers;
                const uint64_t sect = (4 * n_out + 15) & ~15ull;
                if (hd->numel != a.numel || hd->nchunks != l.nchunks) bad = kStFormat;
                else if (hd->off_lens != l.off_lens || hd->off_chunk_off != l.off_chunk_off ||
                         hd->off_outl_off != l.off_outl_off || hd->off_sub_bits != l.off_sub_bits ||
                         hd->off_payload != l.off_payload) bad = kStFormat;
                else if (hd->total_size > a.size || n_out > a.numel || hd->range_events > a.numel) bad = kStFormat;
                else if (hd->off_outl_idx < l.off_payload || ((hd->off_outl_idx - l.off_payload) & 15)) bad = kStFormat;
                else if (hd->off_outl_val != hd->off_outl_idx + sect || hd->total_size != hd->off_outl_val + sect)
                    bad = kStFormat;
                else if (((hd->off_outl_idx - l.off_payload) >> 4) >= (1ull << 32)) bad = kStFormat;
                if (!bad) {
                    const uint32_t units = (uint32_t)((hd->off_outl_idx - l.off_payload) >> 4);
                    if (ends[0] != 0 || ends[1] != units) bad = kStFormat;
                    if (ends[2] != 0 || ends[3] != (uint32_t)n_out) bad = kStFormat;
                    T.payload_units = units;
                    T.n_outliers = (uint32_t)n_out;
                }
            }
            if (bad) atomicOr(bad_s, bad);
        }
        // The wave's scale: what it leaves of the codes of this lane's length, x in [xl, xh).  They have no entry where the
        // entries are wider than they are, and on x itself below the smallest x (whose own entry is not used: what lies
        // below ends up there).
        // In units of 2^-31, which are exact up to 24 bits; no scale has longer codes.
        const uint32_t m = 7u + wv, added = wv == 0 ? 0u : wv == 1 ? 1u << 23 : wv == 2 ? 1u << 27 : 1u << 29;
        const uint32_t xh = (uint32_t)((one - excl) >> (kMaxCodeLen - 31)), xl = (uint32_t)((one - incl) >> (kMaxCodeLen - 31));
        uint32_t left = xh - xl;
        if (lane <= 24) {
            const uint32_t wide_from = lane <= (int)m ? 0xffffffffu : 1u << (32u + m - (uint32_t)lane);      // of x + 2^j
            const uint32_t from = wide_from > xl + added ? wide_from - added : xl, b = from < xh ? from : xh;      // no entry in [b, xh)
            const uint32_t smallest = wv == 0 ? (1u << (31 - kPowers7)) + (1u << (31 - kPowers7 - 7)) : 0u, d = smallest < b ? smallest : b;
            left = (xh - b) + (xl < d ? d - xl : 0u);                                                        // nor in [xl, d)
        }
        left = cnt ? left : 0u;
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_sum(left), 63);
        const unsigned long long some = __ballot(left != 0 || (cnt != 0 && lane > 24));
        if (lane == 0) {
            left_s[wv] = total;
            from_s[wv] = some ? (uint32_t)__ffsll((long long)some) - 1u : 0u;
        }
    }
    __syncthreads();
    if (*bad_s) return *bad_s;
    if (*bad2_s) return *bad2_s;

    // The scale to take.  An index on x with m = 7 takes two instructions more than a linear one and one on x + 2^j three, of some
    // sixteen per codeword; a search takes about ten codewords' time, and the 64 lanes of a wave wait for any of them.
    uint32_t scale = 4, least = left_s[4];
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
        const uint32_t cost = left_s[k] + (k ? 3u << 18 : 1u << 18);  // (2^18: 0.00012 of the space)
        if (cost < least) { least = cost; scale = k; }
    }
    scale = uniform_u32(scale);
    const uint32_t m = 7u + scale, j = scale == 1u ? 24u : scale == 2u ? 28u : scale == 3u ? 30u : 32u;
    const uint32_t shift = 23u - m, least_f = (127u + (scale ? j : 32u - kPowers7)) << 23;
    const uint32_t added8 = scale ? 1u << (j - 8u) : 0u;
    if (tid == 0) {
        T.scale_min = least_f; T.scale_shift = shift;
        T.offset = scale ? __uint_as_float((127u + j) << 23) : 0.0f;
        T.from = from_s[scale] ? from_s[scale] : 1u;
    }

    // symbols ordered by (length, symbol)
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (L[q]) sorted[T.range[L[q]].y + (uint32_t)T.first[L[q]] + wave_off[q * 4 + wv][L[q]] + in_wave[q]] = (uint16_t)((q * 256 + tid - a.radius) & 1023u);

    // the table: an entry holds a codeword only if all of it lies inside that code's part of the space
    {
        constexpr uint32_t kPer = kTableSize / NT;
        uint32_t v[kPer], longest[kPer], l[kPer];                // its smallest left-aligned value; the longest code it may hold
#pragma unroll
        for (uint32_t i = 0; i < kPer; ++i) {
            const uint32_t idx = tid + i * NT;
            // x where the entry begins (with 2^j added) and ends, in units of 2^8, which no entry divides
            const uint32_t f = least_f + (idx << shift), power = (f >> 23) - 127u;                 // at most 33
            const uint32_t begin = (((f << 2) & 0x1ffffffu) | 0x2000000u) >> (33u - power);
            const uint32_t end = begin + (1u << (power - m - 8u)) - added8;
            v[i] = 0u - (end << 8);
            longest[i] = end <= (1u << 24) && (idx || added8) ? 32u - (power - m) : 0u;
            l[i] = 0;                                            // lengths whose codes all lie below v (no more than 31 count)
        }
#pragma unroll
        for (uint32_t step = 16; step >= 1; step >>= 1) {
#pragma unroll
            for (uint32_t i = 0; i < kPer; ++i) l[i] += (v[i] >= lim[l[i] + step]) ? step : 0u;
        }
        uint32_t at[kPer];
#pragma unroll
        for (uint32_t i = 0; i < kPer; ++i) { ++l[i]; at[i] = T.range[l[i]].y + (v[i] >> (32u - l[i])); }
        __syncthreads();                                         // the symbols are in order
#pragma unroll
        for (uint32_t i = 0; i < kPer; ++i) {
            const uint32_t e = sorted[at[i] & (kMaxSym - 1u)] | (l[i] << 10);
            T.entry[tid + i * NT] = (uint16_t)(l[i] <= longest[i] ? e : 0u);
        }
    }
    // the ordered symbols in their packed form, if there are codewords that the table leaves
    if (from_s[scale]) {                                         // uniform
        const uint32_t used = *used_s;
        for (uint32_t w = tid; w < (kMaxSym + 2) / 3; w += NT) {
            uint32_t v = 0;
#pragma unroll
            for (uint32_t j = 0; j < 3; ++j)
                if (3 * w + j < used) v |= (uint32_t)sorted[3 * w + j] << (10 * j);
            T.sorted3[w] = v;
        }
    }
    __syncthreads();
    return 0;
}

// Table entries are length << 10 | residual, the residual (symbol - radius) in 10 bits.
__device__ __forceinline__ int32_t entry_residual(uint32_t e)
{
    return __builtin_amdgcn_sbfe((int)e, 0, 10);
}

// Where in the table (in bytes) the entry for the next 32 bits of a stream lies; an entry of 0: not resolved.
enum Scale : int { kScaleLinear = 0, kScaleOffset = 1, kScaleLog7 = 2 };
struct ScaleArgs {
    uint32_t min, shift, base;                                // (uniform)
    float    offset;
    __device__ __forceinline__ explicit ScaleArgs(const DecodeTables &T)
        : min(uniform_u32(T.scale_min)), shift(uniform_u32(T.scale_shift)), base(0u - ((min >> shift) << 1)),
          offset(__uint_as_float(uniform_u32(__float_as_uint(T.offset))))
    {
    }
    __device__ __forceinline__ int scale() const { return offset == 0.0f ? kScaleLog7 : shift == 23u - kLinearBits ? kScaleLinear : kScaleOffset; }
    // ~hi & mask in one instruction
    static __device__ __forceinline__ uint32_t x_of(uint32_t hi, uint32_t mask)
    {
        uint32_t x;
        asm("v_bfi_b32 %0, %1, 0, %2" : "=v"(x) : "v"(hi), "s"(mask));
        return x;
    }
    // five instructions (kScaleOffset, which does for kScaleLinear too), four or two
    template <int SCALE>
    __device__ __forceinline__ uint32_t place(uint32_t hi) const
    {
        if (SCALE == kScaleLinear) return ~(hi >> (31u - kLinearBits)) & ((2u << kLinearBits) - 2u);
        if (SCALE == kScaleOffset) return ((__float_as_uint((float)x_of(hi, kOffsetMask) + offset) >> shift) << 1) + base;
        // (what lies below the smallest x saturates to entry 0, which is empty)
        const uint32_t above = __builtin_elementwise_sub_sat(__float_as_uint((float)x_of(hi, kLog7Mask)), min);
        uint32_t r;                                           // (above >> 16) * 2 in one instruction
        asm("v_mad_u32_u16 %0, %1, 2, 0 op_sel:[1,0,0,0]" : "=v"(r) : "v"(above));
        return r;
    }
    // the same for any scale; mask: kLog7Mask or kOffsetMask, uniform
    __device__ __forceinline__ uint32_t mask() const { return offset == 0.0f ? kLog7Mask : kOffsetMask; }
    __device__ __forceinline__ uint32_t place_any(uint32_t hi, uint32_t mask) const
    {
        const uint32_t f = __float_as_uint((float)x_of(hi, mask) + offset);
        return (((f > min ? f : min) >> shift) << 1) + base;
    }
};

// Canonical search over the lengths that the table does not resolve, for the entry it would have; v: the next 64
// bits of the stream, of which kMaxCodeLen count.  As in decode_lds.
__device__ __forceinline__ uint32_t search(const DecodeTables &T, uint64_t v, bool &bad)
{
    const uint32_t hi = (uint32_t)(v >> 32), max_len = T.max_len;
    uint32_t L = T.from;
    uint2 r = T.range[L];
    while (L < 32u && hi > r.x) r = T.range[++L];
    if (L <= max_len && L < 32u) {
        const uint32_t i = (hi >> (32u - L)) + r.y;
        if (i < kMaxSym) return sorted_at(T, i) | (L << 10);
    }
    if (max_len >= 32u) {
        for (; L <= max_len; ++L) {
            const uint64_t code = v >> (64 - L);
            if (code >= T.first[L] && code - T.first[L] < codes_of_length(T, L)) return sorted_at(T, T.range[L].y + (uint32_t)code) | (L << 10);
        }
    }
    bad = true;
    return 1u << 10;                                             // no match: residual 0, one bit further on
}

// Decode `count` codewords that start at bit `start` of a chunk stream whose 32-bit words
// are read through rd(word index); rd must be safe for any index (clamp) -- words past the
// stream only ever reach bits that a well-formed stream does not consume.  put(k, symbol) is
// called for k >= klo, where the second argument is the residual symbol - radius (the outlier
// marker, symbol 0, arrives as -radius).  Returns the bit position after the last codeword; sets bad when a
// bit pattern matches no codeword.
//
// The bit window is refilled from a word fetched one refill ahead, so the only memory
// latency on the per-symbol dependency chain is the table lookup.
template <class RD, class PUT>
__device__ __forceinline__ uint32_t decode_run(const DecodeTables &T, RD rd, uint32_t start, uint32_t count,
                                               uint32_t klo, PUT put, bool &bad)
{
    uint32_t wi = start >> 5;
    uint64_t win = ((((uint64_t)rd(wi)) << 32) | rd(wi + 1)) << (start & 31);
    int avail = 64 - (int)(start & 31);
    wi += 2;
    uint32_t nxt = rd(wi);
    const ScaleArgs sc(T);
    const uint32_t mask = sc.mask();
    const char *table = reinterpret_cast<const char *>(T.entry);
    for (uint32_t k = 0; k < count; ++k) {
        if (avail <= 32) {
            // touch the prefetched word only here, so that its latency is waited for once per consumed
            // word and not on every step
            win |= ((uint64_t)nxt) << (32 - avail);
            avail += 32;
            ++wi;
            nxt = rd(wi);
        }
        const uint32_t hi = (uint32_t)(win >> 32);
        uint32_t e = *reinterpret_cast<const uint16_t *>(table + sc.place_any(hi, mask));
        if (e == 0) {
            {
                // canonical search on a fresh 64-bit window
                uint32_t pos = 32u * wi - (uint32_t)avail;
                const uint32_t w0 = pos >> 5, off = pos & 31;
                uint64_t w64 = ((((uint64_t)rd(w0)) << 32) | rd(w0 + 1)) << off;
                if (off) w64 |= (uint64_t)(rd(w0 + 2) >> (32 - off));
                uint32_t len = 0, sy = 0;                    // no match: residual 0
                for (uint32_t L = T.from; L <= T.max_len; ++L) {
                    const uint64_t code = w64 >> (64 - L);
                    if (code >= T.first[L] && code - T.first[L] < codes_of_length(T, L)) {
                        sy = sorted_at(T, T.range[L].y + (uint32_t)code);
                        len = L;
                        break;
                    }
                }
                if (len == 0) { bad = true; len = 1; }
                pos += len;
                wi = pos >> 5;
                win = ((((uint64_t)rd(wi)) << 32) | rd(wi + 1)) << (pos & 31);
                avail = 64 - (int)(pos & 31);
                wi += 2;
                nxt = rd(wi);
                e = sy | (64u << 10);            // length already consumed: marker above any real length
            }
        }
        const uint32_t len = e >> 10;
        if (len < 64u) { win <<= len; avail -= (int)len; }
        if (k >= klo) put(k, entry_residual(e));
    }
    return 32u * wi - (uint32_t)avail;
}

// Decoder for a bit stream staged in LDS.  Word k of the stream is S[kStagePad + k].  Decodes
// `count` codewords from bit `pos` on and calls put(k, residual) for k >= skip; returns the bit
// position after the last codeword.
//
// The 32 bits from position p on are alignbit(S[j], S[j+1], -p mod 32) with j = (p + 31) / 32 - 1
// (stream words): counted this way the shift stays below 32 also when p is a multiple of 32.
// Word indices are not clamped: a codeword has at most kMaxCodeLen bits, so `count` codewords
// starting inside the staged words read at most count * kMaxCodeLen / 32 + 3 words past them,
// whatever the stream holds; the caller's buffer has that many words behind the staged ones
// (stage_tail_words).
constexpr uint32_t stage_tail_words(uint32_t count) { return count * kMaxCodeLen / 32 + 4; }
//
constexpr int kStagePad = 4;
template <int SCALE, class PUT>
__device__ __forceinline__ uint32_t decode_lds(const DecodeTables &T, const uint32_t *S, uint32_t pos,
                                               uint32_t count, uint32_t skip, PUT put, bool &bad)
{
    const ScaleArgs sc(T);
    const char *table = reinterpret_cast<const char *>(T.entry);
    // The three stream words around the position live in registers: wa, wb are the window of the
    // current codeword, wc the word after them.  A codeword of the table is at
    // most 24 bits long, so the window moves on by one word at most, and the word that then
    // becomes wc is fetched a whole step before it can be needed: the only LDS access a step
    // has to wait for is the table look-up.
    uint32_t npos = 0u - pos;                                 // alignbit takes its shift from -pos mod 32
    // stream word J-1 holds bit pos (or ends just before it), J = ceil(pos / 32); kept as N = -J, which is
    // one arithmetic shift of npos
    int32_t N = (int32_t)npos >> 5;
    const uint32_t *Sw = S + kStagePad;
    // LDS byte address of stream word 1: word 1 - Nn is then one multiply-add away
    typedef const uint32_t __attribute__((address_space(3))) *lds_word_ptr;
    const uint32_t sw1 = (uint32_t)(uintptr_t)(lds_word_ptr)(Sw + 1);
    uint32_t wa = Sw[-1 - N], wb = Sw[-N], wc = Sw[1 - N];
#pragma unroll 4
    for (uint32_t k = 0; k < count; ++k) {
        const uint32_t hi = __builtin_amdgcn_alignbit(wa, wb, npos);
        uint32_t e = *reinterpret_cast<const uint16_t *>(table + sc.place<SCALE>(hi));
        if (__builtin_expect(e == 0, 0)) {
            {
                // Canonical search over the lengths that the table does not resolve.  Up to 31 bits the
                // length is the first one whose limit is not below the window; the next length's limit is
                // fetched beside the present one's.  (search() in place of this, where it is hardly ever reached,
                // makes the whole loop slower: 64x256x56x56 at eb 5e-3 with 128 codes 145 -> 160 us, a plane of 399x225 221 -> 245.)
                uint32_t len = 0, sy = 0;                     // no match: residual 0
                const uint32_t max_len = T.max_len;
                uint32_t L = T.from;
                uint2 r = T.range[L], next = T.range[L + 1];
                while (L < 32u && hi > r.x) {
                    ++L; r = next;
                    if (L < 32u && hi > r.x) { ++L; r = T.range[L]; next = T.range[L + 1]; }
                }
                if (L <= max_len && L < 32u) {
                    const uint32_t i = (hi >> (32u - L)) + r.y;
                    if (i < kMaxSym) { sy = sorted_at(T, i); len = L; }    // (always, with the lengths of a complete code)
                }
                if (len == 0 && max_len >= 32u) {
                    const uint32_t lo = __builtin_amdgcn_alignbit(wb, wc, npos);
                    const uint64_t v = (((uint64_t)hi) << 32) | lo;
                    // (past 32 bits a limit is rounded down, and a window above it may still hold a codeword of
                    // that length: from here on by first codes)
                    for (; L <= max_len; ++L) {
                        const uint64_t code = v >> (64 - L);
                        if (code >= T.first[L] && code - T.first[L] < codes_of_length(T, L)) {
                            sy = sorted_at(T, T.range[L].y + (uint32_t)code);
                            len = L;
                            break;
                        }
                    }
                }
                if (len == 0) { bad = true; len = 1; }
                e = sy | (len << 10);
                // such a codeword may end two words further on: take the first of the two moves here
                const int32_t Nf = (int32_t)(npos - len) >> 5;
                if (Nf < N - 1) { wa = wb; wb = wc; wc = Sw[2 - N]; --N; }
            }
        }
        npos -= e >> 10;
        const int32_t Nn = (int32_t)npos >> 5;
        const bool moved = Nn != N;
        wa = moved ? wb : wa;
        wb = moved ? wc : wb;
        {
            uint32_t at;                                     // sw1 - 4 * Nn (|Nn| is a word index: far inside 24 bits)
            asm("v_mad_i32_i24 %0, %1, -4, %2" : "=v"(at) : "v"(Nn), "s"(sw1));
            wc = *(lds_word_ptr)(uintptr_t)at;
        }
        N = Nn;
        if (k >= skip) put(k, entry_residual(e));
    }
    return 0u - npos;
}

// decode_lds for complete sub-blocks of 32 codes, whose residuals are summed along the rows: bit k of
// `keep` is 0 where element k starts a row; my[k] takes the sum.  Four codewords at a time: one that the table does
// not resolve has entry 0, which moves nothing, so that the ones behind it find the same; whether there was any is
// looked at once, behind the four.  Against a look behind every one (17 vector and 3 scalar
// instructions per codeword, now 15.5 and 1): a ResNet-18-shaped stream 911 -> 892 us, 8x64x375x500 469 -> 456.
template <int SCALE>
__device__ __forceinline__ uint32_t decode_rows_32(const DecodeTables &T, const uint32_t *S, uint32_t pos, uint32_t keep,
                                                   int16_t *my, bool &bad)
{
    const ScaleArgs sc(T);
    const char *table = reinterpret_cast<const char *>(T.entry);
    uint32_t npos = 0u - pos;
    int32_t N = (int32_t)npos >> 5;
    const uint32_t *Sw = S + kStagePad;
    typedef const uint32_t __attribute__((address_space(3))) *lds_word_ptr;
    const uint32_t sw1 = (uint32_t)(uintptr_t)(lds_word_ptr)(Sw + 1);
    uint32_t wa = Sw[-1 - N], wb = Sw[-N], wc = Sw[1 - N];
    int32_t run = 0;
    auto look = [&](uint32_t hi) -> uint32_t {
        uint32_t e = *reinterpret_cast<const uint16_t *>(table + sc.place<SCALE>(hi));
        asm("" : "+v"(e));                                    // (or it is kept as 16 bits and extended again)
        return e;
    };
    // one codeword on (see decode_lds)
    auto advance = [&](uint32_t e, uint32_t k) {
        npos -= e >> 10;
        const int32_t Nn = (int32_t)npos >> 5;
        const bool moved = Nn != N;
        wa = moved ? wb : wa;
        wb = moved ? wc : wb;
        uint32_t at;
        asm("v_mad_i32_i24 %0, %1, -4, %2" : "=v"(at) : "v"(Nn), "s"(sw1));
        wc = *(lds_word_ptr)(uintptr_t)at;
        N = Nn;
        // run * (0 where the row restarts, else 1) + residual in one multiply-add: the sums of a
        // lane's 32 in-range residuals stay far inside 24 bits
        const uint32_t keep01 = __builtin_amdgcn_ubfe(keep, k, 1);
        asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(run) : "v"(run), "v"(keep01), "v"(entry_residual(e)));
        // (volatile: or two of them become one access that is not aligned)
        *(volatile int16_t __attribute__((address_space(3))) *)(my + k) = (int16_t)run;
    };
#pragma unroll 1
    for (uint32_t group = 0; group < 32u; group += 4) {
        const uint32_t k = uniform_u32(group);                // (the branch below would take it to a vector register)
        uint32_t e[4];
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) {
            e[j] = look(__builtin_amdgcn_alignbit(wa, wb, npos));
            advance(e[j], k + j);
        }
        if (__builtin_expect(e[3] == 0, 0)) {
            uint32_t at = k + (e[0] != 0) + (e[1] != 0) + (e[2] != 0);
            run = at ? my[at - 1] : 0;
#pragma unroll 1
            for (; at < k + 4; ++at) {
                const uint32_t hi = __builtin_amdgcn_alignbit(wa, wb, npos);
                uint32_t en = look(hi);
                if (en == 0) {
                    en = search(T, ((uint64_t)hi << 32) | __builtin_amdgcn_alignbit(wb, wc, npos), bad);
                    // such a codeword may end two words further on: take the first of the two moves here
                    const int32_t Nf = (int32_t)(npos - (en >> 10)) >> 5;
                    if (Nf < N - 1) { wa = wb; wb = wc; wc = Sw[2 - N]; --N; }
                }
                advance(en, at);
            }
        }
    }
    return 0u - npos;
}

}  // namespace cmpz
