// Huffman codebook on the GPU: histogram -> code lengths -> canonical codes.
// One workgroup per tensor; no host round trip between the two sweeps of a compress.  For small tensors it
// finds the container's offsets and writes its header too.
//
// Rule (fixes one of the equally optimal codebooks): leaves sorted ascending by
// (count, symbol); two FIFO queues, leaves and internal nodes in creation order;
// the lighter head is taken, a leaf before an internal node of equal weight.
// Codes are canonical: ordered by (length, symbol), first code 0, read MSB first.
//
// The merge runs in rounds that join up to 32 pairs at once (see step 4).  Sorting is by
// counting ranks in blocks of 64 and binary search across blocks, depths by pointer jumping,
// ranks within a length by wave ballots.
#include "cmpz_offsets.h"

namespace cmpz {
namespace {

constexpr int kCbThreads = 1024;
constexpr uint32_t kInf = 0xffffffffu;       // "no such node"; real weights stay below 2^32 - 8192, the largest tensor

__device__ __forceinline__ uint32_t rdlane(uint32_t v, uint32_t l)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)l);
}

// LDS written by some lanes of a wave is read by others: the hardware keeps a wave's LDS
// operations in order, this keeps the compiler from moving them across.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// One exchange of a bitonic merge: a and b hold the keys of the lower and the upper lane of the
// lane's pair; the lower lane keeps the smaller one.
__device__ __forceinline__ uint64_t keep_of_pair(uint64_t a, uint64_t b, bool upper)
{
    return ((b < a) != upper) ? b : a;
}
template <int CTRL>
__device__ __forceinline__ uint64_t exchange_dpp(uint64_t k, bool upper)
{
    const uint64_t p = ((uint64_t)dpp_u32<CTRL, 0xf>((uint32_t)(k >> 32)) << 32) | dpp_u32<CTRL, 0xf>((uint32_t)k);
    return ((p < k) != upper) ? p : k;
}
// lane ^ 4: four lanes up in the even banks of a row, four down in the odd ones
__device__ __forceinline__ uint32_t lane_xor4(uint32_t v)
{
    const int up = __builtin_amdgcn_update_dpp((int)v, (int)v, 0x104, 0xf, 0x5, false);     // row_shl:4
    return (uint32_t)__builtin_amdgcn_update_dpp(up, (int)v, 0x114, 0xf, 0xA, false);       // row_shr:4
}

// A bitonic sequence of distinct keys, one per lane, into ascending order over the lanes.
__device__ __forceinline__ uint64_t bitonic_merge_64(uint64_t k, int lane)
{
    {   // lane ^ 32: the swap of halves leaves both keys of a pair in both its lanes
        const auto h = __builtin_amdgcn_permlane32_swap((uint32_t)(k >> 32), (uint32_t)(k >> 32), false, false);
        const auto l = __builtin_amdgcn_permlane32_swap((uint32_t)k, (uint32_t)k, false, false);
        k = keep_of_pair(((uint64_t)h[0] << 32) | l[0], ((uint64_t)h[1] << 32) | l[1], (lane & 32) != 0);
    }
    {   // lane ^ 16: the same by rows
        const auto h = __builtin_amdgcn_permlane16_swap((uint32_t)(k >> 32), (uint32_t)(k >> 32), false, false);
        const auto l = __builtin_amdgcn_permlane16_swap((uint32_t)k, (uint32_t)k, false, false);
        k = keep_of_pair(((uint64_t)h[0] << 32) | l[0], ((uint64_t)h[1] << 32) | l[1], (lane & 16) != 0);
    }
    k = exchange_dpp<0x128>(k, (lane & 8) != 0);             // row_ror:8
    {
        const uint64_t p = ((uint64_t)lane_xor4((uint32_t)(k >> 32)) << 32) | lane_xor4((uint32_t)k);
        k = ((p < k) != ((lane & 4) != 0)) ? p : k;
    }
    k = exchange_dpp<0x4E>(k, (lane & 2) != 0);              // quad_perm 2,3,0,1
    return exchange_dpp<0xB1>(k, (lane & 1) != 0);           // quad_perm 1,0,3,2
}

// The same for keys of 32 bits: one instruction each for the smaller and the larger key of a pair.
template <int CTRL>
__device__ __forceinline__ uint32_t exchange_dpp(uint32_t k, bool upper)
{
    const uint32_t p = dpp_u32<CTRL, 0xf>(k), least = p < k ? p : k, most = p < k ? k : p;
    return upper ? most : least;
}
__device__ __forceinline__ uint32_t bitonic_merge_64(uint32_t k, int lane)
{
    const auto h = __builtin_amdgcn_permlane32_swap(k, k, false, false);
    k = (lane & 32) ? (h[0] > h[1] ? h[0] : h[1]) : (h[0] < h[1] ? h[0] : h[1]);
    const auto r = __builtin_amdgcn_permlane16_swap(k, k, false, false);
    k = (lane & 16) ? (r[0] > r[1] ? r[0] : r[1]) : (r[0] < r[1] ? r[0] : r[1]);
    k = exchange_dpp<0x128>(k, (lane & 8) != 0);             // row_ror:8
    {
        const uint32_t p = lane_xor4(k), least = p < k ? p : k, most = p < k ? k : p;
        k = (lane & 4) ? most : least;
    }
    k = exchange_dpp<0x4E>(k, (lane & 2) != 0);              // quad_perm 2,3,0,1
    return exchange_dpp<0xB1>(k, (lane & 1) != 0);           // quad_perm 1,0,3,2
}

// SMALL: the tensors' offsets and headers too (see small_group).
template <bool SMALL>
__global__ __launch_bounds__(kCbThreads) void k_codebook(BatchC b)
{
    // one workgroup per tensor of the group
    const uint32_t ti = blockIdx.x;
    uint32_t *__restrict__ g_hist = b.hist + (uint64_t)ti * kHistCopies * kMaxSym;
    const OutRef oref = resolve_out(b.t[ti]);
    uint8_t *__restrict__ out = oref.out;
    alignas(16) __shared__ uint64_t key[kMaxSym];    // used symbols, compacted: count << 10 | symbol; then all ones
    __shared__ uint64_t skey[kMaxSym];           // the same, every block of 64 in ascending order
    __shared__ uint32_t leaf_w[kMaxSym + 192];   // leaf weights, ascending, padded with kInf
    __shared__ uint16_t leaf_sym[kMaxSym];
    __shared__ uint32_t node_w[kMaxSym + 192];   // internal node weights in creation order, kInf = not made
    __shared__ uint32_t link[2 * kMaxSym];       // of leaves 0..n-1, internal nodes n..2n-2: a node above, and how far << 16
    __shared__ uint32_t len_of[kMaxSym];         // code length per symbol
    __shared__ uint32_t wave_cnt[16][64];
    __shared__ uint64_t first_code[64];
    __shared__ uint32_t wave_used[16];

    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const uint32_t nsym = 2 * b.radius;

    // 1. fetch the histogram, leave it zeroed for the next call, keep a copy for inspection
    uint32_t part[kHistCopies], cnt = 0;
#pragma unroll
    for (uint32_t k = 0; k < kHistCopies; ++k) part[k] = g_hist[k * kMaxSym + tid];
#pragma unroll
    for (uint32_t k = 0; k < kHistCopies; ++k) { cnt += part[k]; g_hist[k * kMaxSym + tid] = 0; }
    if ((uint32_t)tid >= nsym) cnt = 0;
    b.hist_copy[ti * kMaxSym + tid] = cnt;
    len_of[tid] = 0;

    // 2. compact the used symbols (ballot + per-wave offsets)
    const unsigned long long used_mask = __ballot(cnt != 0);
    if (lane == 0) wave_used[wv] = (uint32_t)__popcll(used_mask);
    __syncthreads();
    uint32_t n = 0, my_slot = 0;
    for (int k = 0; k < 16; ++k) { if (k < wv) my_slot += wave_used[k]; n += wave_used[k]; }
    my_slot += (uint32_t)__popcll(used_mask & ((1ull << lane) - 1ull));
    if (cnt) key[my_slot] = ((uint64_t)cnt << 10) | (uint64_t)tid;
    if ((uint32_t)tid >= n) key[tid] = ~0ull;                        // heavier than any key
    __syncthreads();

    // 3. sort (keys are distinct).  Every wave orders its own 64 keys by counting the smaller ones
    //    among them; the rank of a key is then, by binary search, the number of smaller keys in every block.  Four
    //    searches at a time: they are chains of seven LDS accesses.
    const uint32_t nblocks = (n + 63u) >> 6;                         // uniform
    const uint64_t mine = key[tid];
    if ((uint32_t)wv < nblocks) {
        const ulonglong2 *block = reinterpret_cast<const ulonglong2 *>(key + ((uint32_t)wv << 6));
        uint32_t in_block = 0;
#pragma unroll
        for (uint32_t j = 0; j < 32; ++j) {
            const ulonglong2 two = block[j];
            in_block += (two.x < mine) ? 1u : 0u;
            in_block += (two.y < mine) ? 1u : 0u;
        }
        if ((uint32_t)tid >= n) in_block = (uint32_t)lane;
        skey[((uint32_t)wv << 6) + in_block] = mine;
    }
    __syncthreads();
    if ((uint32_t)tid < n) {
        uint32_t rank = 0;
        for (uint32_t w = 0; w < nblocks; w += 4) {
            const uint64_t *blk[4];
            uint32_t pos[4] = {};
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) blk[j] = skey + ((w + j < nblocks ? w + j : w) << 6);
#pragma unroll
            for (uint32_t step = 32; step >= 1; step >>= 1) {
#pragma unroll
                for (uint32_t j = 0; j < 4; ++j) pos[j] += (blk[j][pos[j] + step - 1] < mine) ? step : 0u;
            }
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) {
                pos[j] += (blk[j][pos[j]] < mine) ? 1u : 0u;         // a count of 63 may be 64
                if (w + j < nblocks) rank += pos[j];
            }
        }
        leaf_w[rank] = (uint32_t)(mine >> 10);
        leaf_sym[rank] = (uint16_t)(mine & 1023u);
    }
    if ((uint32_t)tid < 192) leaf_w[n + tid] = kInf;
    node_w[tid] = kInf;
    if (tid < 192) node_w[kMaxSym + tid] = kInf;
    if (tid == 0 && n) link[2 * n - 2] = 2 * n - 2;                  // the root
    __syncthreads();

    // 4. the two-queue merge, by wave 0, in rounds of up to 32 nodes.  The sequential rule takes the
    //    unused nodes of both queues in one fixed order -- by weight, a leaf before an internal node
    //    of the same weight, each queue in its own order -- and joins them two by two.  A node made
    //    now weighs at least t, the sum of the two lightest unused nodes, and queues up behind every
    //    node that exists already; so all unused nodes of weight <= t keep their places in that
    //    order whatever is made from them, and a whole round of them can be joined at once: the next
    //    64 nodes of either queue are merged into their common order, one node per lane, and the
    //    pairs (0,1), (2,3), ... become the new nodes, already in order of weight.  Activation
    //    histograms need about twenty rounds where the sequential rule needs hundreds of steps.
    //    Both windows are ascending, so the lighter of leaf i and node 63-i, over all lanes, are the
    //    64 lightest of the 128 as a bitonic sequence, which six exchanges between lanes sort
    //    without touching LDS.  A round is one wave's latency and nothing else.  Against places found
    //    by binary search in LDS (four dependent accesses), LDS counters for the lengths and a serial
    //    loop over the first codes the kernel went from 22.6 to 14.8 us on one 64x56x56 activation,
    //    32.6 to 22.4 us on 64x256x56x56 (eb 5e-3) and 39.4 to 26.0 us with all 1024 symbols in use.
    //    Keys of 32 bits instead of 64 in all rounds but the last ones of large tensors, the histogram's loads and
    //    the searches of the sort in flight together, pointer jumping for the depths and ballots over the bits of
    //    the lengths: 13.6 to 10.6 us, 20.4 to 15.2 us and 25.6 to 19.7 us, between the first and the last of its
    //    own instructions (370 to 270 ns per round).
    if (__builtin_amdgcn_readfirstlane(wv) == 0 && __builtin_amdgcn_readfirstlane((int)n) >= 2) {
        const uint32_t nu = (uint32_t)__builtin_amdgcn_readfirstlane((int)n);   // n came from LDS: tell the compiler it is uniform
        const uint32_t steps = nu - 1;
        uint32_t ql = 0, qi = 0, m = 0;                      // leaves used, internal nodes used, internal nodes made
        // one round: the 64 lightest nodes in order, each lane's weight and place (leaves from 0, nodes from 64 on)
        auto join = [&](uint32_t w, uint32_t id, uint32_t t) {
            uint32_t npairs = (uint32_t)__popcll(__ballot(w <= t)) >> 1;         // (a prefix of the lanes)
            npairs = npairs < steps - m ? npairs : steps - m;
            // the two lightest nodes always weigh <= t, so a round joins at least one pair; a histogram
            // whose counts do not add up below 2^32 (damaged scratch memory) could break that: leave
            // rather than spin
            if (npairs == 0) {
                if (lane == 0) atomicOr(b.status, kStInternal);
                m = steps;
                return;
            }
            const bool used = (uint32_t)lane < 2u * npairs, leaf = id < 64u;
            const uint32_t sum = w + dpp_u32<0xB1, 0xf>(w);                      // with the pair's other node
            if (used) link[leaf ? ql + id : nu + qi + (id - 64u)] = (nu + m + ((uint32_t)lane >> 1)) | (1u << 16);
            if (used && !(lane & 1)) node_w[m + ((uint32_t)lane >> 1)] = sum;
            wave_lds_sync();
            const uint32_t nl = (uint32_t)__popcll(__ballot(used && leaf));
            ql += nl;
            qi += 2u * npairs - nl;
            m += npairs;
        };
        // while t is below 2^25 - 1, weight and place fit 32 bits: heavier nodes have no part in the round
        constexpr uint32_t kMost = (1u << 25) - 1u;
        while (m < steps) {
            const uint32_t lw = leaf_w[ql + lane], iw = node_w[qi + 63 - lane];  // kInf past the last leaf; at and past node m
            const uint32_t kl = ((lw < kMost ? lw : kMost) << 7) | (uint32_t)lane;
            const uint32_t ki = ((iw < kMost ? iw : kMost) << 7) | (uint32_t)(127 - lane);
            const uint32_t k = bitonic_merge_64(ki < kl ? ki : kl, lane);
            const uint32_t t = (rdlane(k, 0) >> 7) + (rdlane(k, 1) >> 7);
            if (t >= kMost) break;
            join(k >> 7, k & 127u, t);
        }
        while (m < steps) {
            const uint32_t lw = leaf_w[ql + lane], iw = node_w[qi + 63 - lane];
            // place in the window, leaves before nodes: the order among equal weights
            const uint64_t kl = ((uint64_t)lw << 32) | (uint32_t)lane, ki = ((uint64_t)iw << 32) | (uint32_t)(127 - lane);
            const uint64_t k = bitonic_merge_64(ki < kl ? ki : kl, lane);
            const uint32_t w = (uint32_t)(k >> 32);
            const uint64_t t = (uint64_t)rdlane(w, 0) + rdlane(w, 1);
            join(w, (uint32_t)k, (t < (uint64_t)kInf) ? (uint32_t)t : kInf - 1u);
        }
    }
    __syncthreads();

    // 5. depth of every leaf = its code length: every node's link is replaced by the link of the node it leads to
    //    until it leads to the root, at twice the distance each time.  The words are read and written
    //    whole, so a link is right whether the other has been replaced already or not: no barriers.
    {
        const uint32_t root = n > 1 ? 2 * n - 2 : 0;             // (no tree: nobody has a way to go)
        volatile uint32_t *const links = link;
        const uint32_t leaf = tid, node = n + tid;
        const bool is_leaf = n > 1 && leaf < n, is_node = node < root && n > 1;
        uint32_t a = is_leaf ? links[leaf] : root, c = is_node ? links[node] : root;
        // (bounded: a step goes at least one node up, and a complete tree has at most kMaxCodeLen levels)
        for (uint32_t k = 0; k < 64u; ++k) {
            const bool more_a = (a & 0xffffu) != root, more_c = (c & 0xffffu) != root;
            if (!__any(more_a || more_c)) break;
            if (more_a || more_c) {
                const uint32_t qa = links[a & (2 * kMaxSym - 1)], qc = links[c & (2 * kMaxSym - 1)];
                a = (qa & 0xffffu) | ((a & 0xffff0000u) + (qa & 0xffff0000u));
                c = (qc & 0xffffu) | ((c & 0xffff0000u) + (qc & 0xffff0000u));
                if (is_leaf) links[leaf] = a;
                if (is_node) links[node] = c;
            }
        }
        if (leaf < n) len_of[leaf_sym[leaf]] = n == 1 ? 1u : a >> 16;
    }
    __syncthreads();

    // 6. canonical codes.  Every wave ranks its symbols within their lengths; then wave 0, a lane per
    //    length, turns the waves' counts into offsets and finds the first code of its length: with
    //    P = the sum of count[j] << (48 - j) over all shorter lengths j it is P >> (48 - length).
    const uint32_t L = len_of[tid] & 63u;
    wave_cnt[wv][lane] = 0;
    wave_lds_sync();
    unsigned long long same = ~0ull;                      // the lanes with this length
#pragma unroll
    for (uint32_t k = 0; k < 6; ++k) {
        const bool set = (L >> k) & 1u;
        const unsigned long long those = __ballot(set);
        same &= set ? those : ~those;
    }
    const uint32_t in_wave = (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
    if (L && in_wave == 0) wave_cnt[wv][L] = (uint32_t)__popcll(same);
    __syncthreads();
    if (wv == 0) {
        uint32_t total = 0;
#pragma unroll
        for (int k = 0; k < kCbThreads / kWave; ++k) {
            const uint32_t c = wave_cnt[k][lane];
            wave_cnt[k][lane] = total;                    // symbols of this length in earlier waves
            total += c;
        }
        const unsigned long long present = __ballot(total != 0);
        const uint32_t max_len = present ? 63u - (uint32_t)__builtin_clzll(present) : 0u;
        // (below 2^48 in all: three limbs of 24 bits, each scanned in 32 bits without overflow)
        const bool real = lane >= 1 && lane <= (int)kMaxCodeLen;
        const uint64_t sl = real ? ((uint64_t)total << (kMaxCodeLen - lane)) : 0ull;
        const uint32_t i0 = wave_inclusive_sum((uint32_t)(sl & 0xffffffu));
        const uint32_t i1 = wave_inclusive_sum((uint32_t)((sl >> 24) & 0xffffffu));
        const uint32_t i2 = wave_inclusive_sum((uint32_t)(sl >> 48));
        const uint64_t excl = (uint64_t)i0 + ((uint64_t)i1 << 24) + ((uint64_t)i2 << 48) - sl;
        first_code[lane] = real ? (excl >> (kMaxCodeLen - lane)) : 0ull;
        if (lane == 0) b.tmeta[ti].max_len = max_len;
        if (lane == (int)kEncBits + 1) b.tmeta[ti].long_from = (uint32_t)(excl >> (kMaxCodeLen - 32));
    }
    __syncthreads();
    const uint32_t rank = wave_cnt[wv][L] + in_wave;
    const uint64_t entry = L ? (((uint64_t)L << 56) | (first_code[L] + rank)) : 0ull;
    b.codes[ti * kMaxSym + tid] = entry;
    b.lens[ti * kMaxSym + tid] = (uint8_t)L;
    // what the packing kernel looks up: the first 24 bits of the codeword, left-aligned, above its length
    const uint64_t left = L ? (first_code[L] + rank) << (64u - L) : 0ull;
    b.enc32[ti * kMaxSym + tid] = ((uint32_t)(left >> 32) & ~0xffu) | L;
    // container section `lens`: 2*radius bytes, zero padded to a multiple of 16
    const uint32_t padded = (nsym + 15u) & ~15u;
    if ((uint32_t)tid < padded && oref.cap >= kHeaderBytes + padded) out[kHeaderBytes + tid] = ((uint32_t)tid < nsym) ? (uint8_t)L : 0;
    if (!SMALL) return;

    // 7. a small tensor's bit counts, offsets and header, without the two launches that spread this over the chip.
    //    Bound by the latency of the loads: every wave takes consecutive chunks, four at a time, and learns
    //    beforehand which of them have symbols without a byte form.
    const TensorC &tc = b.t[ti];
    uint8_t *lens_s = reinterpret_cast<uint8_t *>(leaf_w);           // (what the tree was built in is free)
    uint32_t *bits_s = node_w;
    static_assert(kSmallChunks <= kMaxSym && kSmallChunks <= (uint32_t)kCbThreads, "a thread and a word of node_w per chunk");
    lens_s[tid] = (uint8_t)L;
    __syncthreads();
    {
        ChunkBits cb(b, leaf_w, lane);
        constexpr uint32_t kTogether = 4;                            // chunks whose loads are in flight together
        const uint32_t per = (tc.nchunks + 15u) >> 4, first = wv * per;
        const uint32_t end = first + per < tc.nchunks ? first + per : tc.nchunks;
        uint2 before = make_uint2(0, 0);
        if (first < end && first) before = cb.row(tc.chunk_base + first - 1);
        uint64_t wide = 0;                                           // of the wave's chunks from c on
        static_assert(kSmallChunks <= 16 * kWave, "a lane per chunk of a wave");
        if (first + lane < end) wide = cb.is_wide(tc.chunk_base + first + lane);
        wide = __ballot(wide != 0);
        for (uint32_t c = first; c < end; c += kTogether, wide >>= kTogether) {          // uniform
            uint2 v[kTogether] = {}, o[kTogether][ChunkBits::kOthers] = {};
#pragma unroll
            for (uint32_t j = 0; j < kTogether; ++j) {
                if (c + j < end) v[j] = cb.row(tc.chunk_base + c + j);
                if ((wide >> j) & 1u) cb.fetch_others(tc.chunk_base + c + j, o[j]);
            }
#pragma unroll
            for (uint32_t j = 0; j < kTogether; ++j) {
                if (c + j >= end) break;
                const uint32_t bits = cb.chunk(tc, c + j, before, v[j], (wide >> j) & 1u, [&] { return cb.others_bits(o[j]); });
                if (lane == 63) bits_s[c + j] = bits;
                before = v[j];
            }
        }
    }
    __syncthreads();
    const bool there = (uint32_t)tid < tc.nchunks;
    const uint32_t bits = there ? bits_s[tid] : 0u, outl = there ? b.outl_cnt[tc.chunk_base + tid] : 0u, units = (bits + 127u) >> 7;
    const uint32_t iu = wave_inclusive_sum(units), io = wave_inclusive_sum(outl), ib = wave_inclusive_sum(bits);
    uint32_t (*sums)[64] = wave_cnt;                                 // [0..2][wave]
    if (lane == 63) { sums[0][wv] = iu; sums[1][wv] = io; sums[2][wv] = ib; }
    __syncthreads();
    uint32_t pu = 0, po = 0, tu = 0, to = 0;
    uint64_t tb = 0;
    for (int k = 0; k < kCbThreads / kWave; ++k) {
        if (k < wv) { pu += sums[0][k]; po += sums[1][k]; }
        tu += sums[0][k]; to += sums[1][k]; tb += sums[2][k];
    }
    if (there) {
        b.chunk_bits[tc.chunk_base + tid] = bits;
        if ((uint32_t)tid % b.pack_chunks == 0) {
            b.range_units[tc.pack_base + (uint32_t)tid / b.pack_chunks] = pu + iu - units;
            b.range_outl[tc.pack_base + (uint32_t)tid / b.pack_chunks] = po + io - outl;
        }
    }
    finish_container(b, ti, tu, to, tb, reinterpret_cast<Header *>(skey), tid);
}

}  // namespace

bool small_group(const BatchC &b)
{
    for (uint32_t k = 0; k < b.n; ++k)
        if (b.t[k].nchunks > kSmallChunks) return false;
    return true;
}

void launch_codebook(const BatchC &b, Profiler *prof, hipStream_t st)
{
    if (small_group(b)) launch(prof, kKCodebook, k_codebook<true>, dim3(b.n), dim3(kCbThreads), st, b);
    else launch(prof, kKCodebook, k_codebook<false>, dim3(b.n), dim3(kCbThreads), st, b);
}

}  // namespace cmpz
