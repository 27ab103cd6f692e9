// hb_ragged.hip -- packed batches of any lengths in one launch, with no workspace in HBM.
//
// A workgroup takes a tile of consecutive messages (hb_plan_rules.hpp).  If they have one block
// count, or sorting would save too little, it hashes them in index order, one lane each; else
// it sorts them by block count in LDS and hashes them longest first: its longest messages (up
// to 32) by a chain pair -- two of its four waves, hb_chain.hpp -- and the others 64 of
// near-equal length at a time by the waves that are free.  A mixed batch gives each tile one workgroup per algorithm, which
// takes the tile's messages of that algorithm, so every wave is algorithm-uniform and the
// three algorithms' chains run beside each other.
//
// What bounds it: the longest message of the batch (a SHA-1 message of 64 KiB takes 836 us
// alone), or with many messages the integer VALU.  One lane per message in index order left
// most lanes of a wave idle behind its longest message and paid the memory latency every
// second block of it, and a mixed batch took one such launch per algorithm: 200,003 SHA-1
// messages of log-normal lengths (median 256, at most 64 KiB) 3,078 us, now 933; 50,021 of
// all three algorithms 8,784, now 1,981; 10^6 SM3 messages of 0 to 4,096 bytes 2,328, now
// 1,127.
#include <algorithm>

#include "hb_chain.hpp"
#include "hb_device.hpp"
#include "hb_internal.hpp"
#include "hb_plan_rules.hpp"
#include "hb_ragged.hpp"

namespace hb {

namespace {

constexpr int kRaggedThreads = int(kTileThreads);
constexpr int kPerThread = int(kTileMax) / kRaggedThreads;
// (Tiles of 512 would read fewer cache lines twice, as sorting 512 at a time does for short
// messages (ragged_tile), but the longest messages of more, smaller tiles start later: 1,000,003
// of log-normal lengths up to 64 KiB MD5 1,087 us for 715, SHA-1 2,167 for 1,053.)
constexpr uint32_t kLenBins = 256;

struct RaggedArgs {
    const uint8_t *msgs;
    const uint64_t *offs;
    const uint64_t *lens;
    const uint8_t *algos;  // per-message ids, or null
    uint8_t *out;
    uint64_t n;
    uint32_t stride;
    uint32_t tile;         // messages per tile
};

// Bin of a block count: itself below 64, then sixteen bins per power of two (messages of
// one bin differ by less than a sixteenth), the last one open.
__device__ __forceinline__ uint32_t len_bin(uint32_t nb)
{
    if (nb < 64u) return nb;
    const uint32_t e = 31u - uint32_t(__builtin_clz(nb));
    return min(kLenBins - 1u, 64u + (e - 6u) * 16u + ((nb >> (e - 4u)) & 15u));
}

struct RaggedLds {
    uint16_t order[kTileMax];     // the tile's messages, longest bin first
    uint32_t bins[kLenBins];      // counts, then first positions
    uint32_t part[kRaggedThreads / 64];
    // of each wave's messages: block counts in all, the largest, the smallest (0 where
    // another algorithm's message is)
    uint32_t blocks[kRaggedThreads / 64], longest[kRaggedThreads / 64], least[kRaggedThreads / 64];
    uint32_t next;                // next position to hand out
    ChainSync sync;
    uint32_t tails[kChainTailWords<>];
    uint32_t simd[kRaggedThreads / 64];  // SIMD of each wave
    uint32_t group;                      // the workgroup's number on its CU
};

// This wave's SIMD and its workgroup's number on the CU (bits 5:4 and 19:16 of HW_ID).
__device__ __forceinline__ uint32_t wave_simd() { return __builtin_amdgcn_s_getreg(4 | (4 << 6) | ((2 - 1) << 11)); }
__device__ __forceinline__ uint32_t group_on_cu() { return __builtin_amdgcn_s_getreg(4 | (16 << 6) | ((4 - 1) << 11)); }

// Fewest blocks of a tile's longest message that a chain pair is for: below, handing the
// schedules over costs more than it saves (16,000 messages, us with / without a pair: MD5 of
// 0 to 2,048 bytes 32.9 / 30.1, 0 to 4,096 55.3 / 56.1; SHA-1 of 0 to 257 14.0 / 13.7, 0 to
// 1,024 27.6 / 29.3; SM3 of 0 to 130 13.7 / 15.2).
template <int A> constexpr uint32_t kChainLeast = A == MD5 ? 48u : (A == SHA1 ? 8u : 3u);
// Operations per block, and how many of them per message sorting has to save (ragged_tile).
template <int A> constexpr uint32_t kBlockOps = A == MD5 ? 324u : (A == SHA1 ? 613u : 1348u);
constexpr uint32_t kSortOps = 700;

// Messages of one block count that a tile's chain pair takes: MD5's chains gain least, and less
// the more of them a pair runs (of 16 KiB, us, by lanes / by chain pairs: 8 to a pair 160 / 155,
// 21 165 / 185).
template <int A> constexpr uint32_t kChainsAlike = A == MD5 ? kTileChainsMd5 : kTileChains;

constexpr uint64_t kNoMessage = ~0ull;
constexpr uint32_t kNoLong = 0xffffffffu;

// The chain pair of a workgroup (its other two waves return at once): message i in lane
// l < 32 (kNoMessage past the last; lane 0's has at least three blocks).  L.simd, L.group and
// the zeroed L.sync are set, with a barrier since.
template <int A>
__device__ __forceinline__ void chain_pair(const RaggedArgs &r, uint64_t i, RaggedLds &L, uint32_t *ring)
{
    // Workgroups that share a CU run their chain waves on different SIMDs: the wave on the
    // SIMD of the workgroup's number (that wave number if none is there), the next but one
    // for the schedules.  With every chain wave the same wave of its workgroup, three
    // workgroups' chains shared one SIMD and took 3.3 times as long.
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64u);
    const uint32_t want = L.group % 4u;
    uint32_t chain_wave = want;
#pragma unroll
    for (uint32_t w = 0; w < kRaggedThreads / 64; ++w)
        if (L.simd[w] == want) chain_wave = w;
    const uint32_t role = __builtin_amdgcn_readfirstlane(wave ^ chain_wave);  // 0 chains, 2 schedules
    if (role != 0 && role != 2) return;
    uint64_t address = 0, len = 0;
    uint32_t blocks = 0;
    if (i != kNoMessage) {
        len = r.lens[i];
        address = uint64_t(reinterpret_cast<uintptr_t>(r.msgs)) + r.offs[i];
        blocks = uint32_t(block_count(len));
    }
    if (role == 0) {
        uint32_t s[8];
        __builtin_amdgcn_s_setprio(3);
        chain_run<A>(blocks, ring, &L.sync, s);
        __builtin_amdgcn_s_setprio(0);
        if (blocks) store_digest<A>(r.out + i * r.stride, s, r.stride);
    } else {
        __builtin_amdgcn_s_setprio(2);
        chain_schedule<A>(address, len, blocks, ring, L.tails, &L.sync);
        __builtin_amdgcn_s_setprio(0);
    }
}

// Messages of at least `from` blocks (by their capped sort key) and fewer than 2^31 are the
// business of other workgroups (k_long_tiles).
__device__ __forceinline__ bool is_long(uint32_t nb, uint32_t from) { return min(nb, kBins - 1u) >= from && nb < 0x80000000u; }

// Lane 63: op over the wave (rows of 16 lanes, then their last lanes into the rows after).
// Cross-lane moves, not LDS: every tile does three of these before it can start hashing.
template <class Op>
__device__ __forceinline__ uint32_t reduce_to_last(uint32_t x, uint32_t none, Op op)
{
#define HB_STEP(ctrl) x = op(x, uint32_t(__builtin_amdgcn_update_dpp(int(none), int(x), ctrl, 0xf, 0xf, false)))
    HB_STEP(0x111); HB_STEP(0x112); HB_STEP(0x114); HB_STEP(0x118);  // row_shr:1, 2, 4, 8
    HB_STEP(0x142); HB_STEP(0x143);                                  // row_bcast:15, 31
#undef HB_STEP
    return x;
}

template <int A, bool MANY, int PER>
__device__ __forceinline__ void ragged_tile(const RaggedArgs &r, uint64_t base, uint32_t long_from, RaggedLds &L,
                                            uint32_t *ring)
{
    const uint32_t tid = threadIdx.x, lane = tid % 64u, wave = __builtin_amdgcn_readfirstlane(tid / 64u);
    const uint32_t have = uint32_t(min<uint64_t>(r.tile, r.n - base));
    // this thread's messages: block counts, 0 for none or one that is not this workgroup's
    uint32_t nb[PER], longest = 0, least = 0xffffffffu, blocks = 0;
    // the first one's place, kept for the case that nothing is sorted
    const uint64_t i0 = base + min(tid, have - 1u), off0 = r.offs[i0], len0 = r.lens[i0];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const uint32_t t = uint32_t(j) * kRaggedThreads + tid;
        nb[j] = 0;
        if (t < have) {
            const uint64_t i = base + t;
            const uint8_t id = r.algos ? r.algos[i] : uint8_t(A);
            if (id == A) nb[j] = uint32_t(min<uint64_t>(block_count(j == 0 ? len0 : r.lens[i]), 0xffffffffull));
            if (A == MD5 && id > SM3) {  // unknown id: an all-zero slot
                HB_GLOBAL uint32_t *o = reinterpret_cast<HB_GLOBAL uint32_t *>(reinterpret_cast<uintptr_t>(r.out + i * r.stride));
                for (uint32_t q = 0; q < r.stride / 4u; ++q) o[q] = 0u;
            }
            if (is_long(nb[j], long_from)) nb[j] = 0;
            longest = max(longest, nb[j]);
            least = min(least, nb[j]);
            blocks += min(nb[j], 1u << 20);  // so that a tile's sum fits
        }
    }
    L.bins[tid] = 0;
    longest = reduce_to_last(longest, 0u, [](uint32_t x, uint32_t y) { return max(x, y); });
    least = reduce_to_last(least, 0xffffffffu, [](uint32_t x, uint32_t y) { return min(x, y); });
    blocks = reduce_to_last(blocks, 0u, [](uint32_t x, uint32_t y) { return x + y; });
    if (lane == 63) {
        L.simd[wave] = wave_simd();
        L.longest[wave] = longest;
        L.least[wave] = least;
        L.blocks[wave] = blocks;
    }
    if (tid == 0) {
        L.group = group_on_cu();
        L.sync.filled = 0; L.sync.taken = 0;
    }
    __syncthreads();
    longest = 0, least = 0xffffffffu, blocks = 0;
#pragma unroll
    for (uint32_t w = 0; w < kRaggedThreads / 64; ++w) {
        longest = max(longest, L.longest[w]);
        least = min(least, L.least[w]);
        blocks += L.blocks[w];
    }
    longest = __builtin_amdgcn_readfirstlane(longest);
    least = __builtin_amdgcn_readfirstlane(least);
    blocks = __builtin_amdgcn_readfirstlane(blocks);
    if (longest == 0) return;  // no message of this algorithm
    // The chain pair takes the longest messages when the longest of all would take at least
    // twice the time that the two waves left need for all the others; nearer to even, two
    // waves fewer for those cost more than the faster chains give; and it has enough blocks.
    const bool chains = longest >= kChainLeast<A> && longest < 0x80000000u && uint64_t(longest) * 64u > blocks;
    // Nothing to gain from sorting: one block count throughout, or one wave a SIMD and no
    // chain pair, where the time is the longest message's in any order.  With one message a
    // thread, sorting has each wave do about the mean of the block counts, not the largest,
    // and takes some 2 us: it is left out where it saves fewer than kSortOps operations a
    // message (262,144 messages, us with / without: MD5 of 0 to 64 bytes 14.3 / 12.2, 0 to 130
    // 17.7 / 16.8; SHA-1 18.4 / 16.2 and 23.6 / 22.5; MD5 of 0 to 257 20.2 sorted, 22.6 before).
    const bool worth = PER > 1 || (uint64_t(longest) * have - blocks) * kBlockOps<A> > uint64_t(kSortOps) * have;
    const bool sorted = least == longest ? have <= kChainsAlike<A> && chains : chains || least == 0 || (MANY && worth);
    // Short messages of one algorithm are sorted within 512 at a time (the last 512 to 1,023 of
    // the tile), each with bins of its own: neighbours in memory share cache lines, and hashed
    // a whole tile apart they were read twice (4,000,000 messages of 0 to 257 / 1,024 bytes,
    // us: MD5 320 / 790 and 284 / 715, SHA-1 353 / 940 and 314 / 859; SM3, bound by its
    // compression, gained nothing).
    constexpr uint32_t kSub = 512, kSubBins = kLenBins * kSub / kTileMax;
    const bool local = A != SM3 && PER == kPerThread && !chains && !r.algos && longest < kSubBins;
    auto bin_of = [&](int j, uint32_t blocks_of) {
        if (!local) return len_bin(blocks_of);
        const uint32_t sub = min(uint32_t(j) * kRaggedThreads / kSub, max(r.tile / kSub, 1u) - 1u);
        return (kTileMax / kSub - 1u - sub) * kSubBins + blocks_of;
    };
    uint32_t count = have;
    if (sorted) {
        uint32_t rank[PER];  // within the bin
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            rank[j] = 0;
            if (nb[j]) {
                const uint32_t bin = bin_of(j, nb[j]), first = __builtin_amdgcn_readfirstlane(bin);
                const uint64_t active = __ballot(1);
                if (__ballot(bin == first) == active) {  // one atomic for the wave
                    const uint32_t below = __builtin_amdgcn_mbcnt_hi(uint32_t(active >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(active), 0u));
                    uint32_t b = 0;
                    if (below == 0) b = atomicAdd(&L.bins[first], uint32_t(__popcll(active)));
                    rank[j] = __builtin_amdgcn_readfirstlane(b) + below;
                } else {
                    rank[j] = atomicAdd(&L.bins[bin], 1u);
                }
            }
        }
        __syncthreads();
        // first position of each bin, longest first: an exclusive scan over the reversed bins
        const uint32_t c = L.bins[kLenBins - 1u - tid];
        uint32_t sum = c;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t up = __shfl_up(sum, d);
            if (lane >= uint32_t(d)) sum += up;
        }
        if (lane == 63) L.part[wave] = sum;
        __syncthreads();
        uint32_t before = 0;
        count = 0;
#pragma unroll
        for (uint32_t w = 0; w < kRaggedThreads / 64; ++w) {
            before += w < wave ? L.part[w] : 0u;
            count += L.part[w];
        }
        L.bins[kLenBins - 1u - tid] = before + sum - c;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < PER; ++j)
            if (nb[j]) L.order[L.bins[bin_of(j, nb[j])] + rank[j]] = uint16_t(uint32_t(j) * kRaggedThreads + tid);
    }
    const uint32_t nchain = sorted && chains ? min(count, kChainMessages) : 0u;
    if (sorted) {
        if (tid == 0) L.next = nchain;
        __syncthreads();
    }
    if (nchain) {
        chain_pair<A>(r, lane < nchain ? base + L.order[lane] : kNoMessage, L, ring);
    }
    // 64 positions at a time: in index order each wave every fourth, sorted whoever is free
    uint32_t p = wave * 64u;
    for (;; p += kRaggedThreads) {
        if (sorted) {
            if (lane == 0) p = atomicAdd(&L.next, 64u);
            p = __builtin_amdgcn_readfirstlane(p);
        }
        if (p >= count) break;
        // A lane past the last message hashes that one again and stores nothing: a wave with
        // half its lanes off issues more slowly (33 messages of 2 KiB MD5, one to a
        // workgroup: 30.8 us with the others off, 23.5 so).
        const uint32_t at = min(p + lane, count - 1u);
        uint64_t i = i0, off = off0, len = len0;
        if (sorted || (PER > 1 && p >= kRaggedThreads)) {
            i = base + (sorted ? L.order[at] : at);
            off = r.offs[i];
            len = r.lens[i];
        }
        uint32_t s[8];
        hash_message<A, kDefaultBurst<A>, MANY>(r.msgs + off, len, s);
        if (p + lane < count) store_digest<A>(r.out + i * r.stride, s, r.stride);
    }
}

template <int A, bool MANY, int PER>
__global__ __launch_bounds__(kRaggedThreads, 4) void k_ragged(RaggedArgs r)
{
    __shared__ RaggedLds L;
    __shared__ __align__(16) uint32_t ring[kChainRingWords<A>];
    ragged_tile<A, MANY, PER>(r, uint64_t(xcd_contiguous(blockIdx.x, gridDim.x)) * r.tile, kNoLong, L, ring);
}

// Three workgroups per tile, one per algorithm; SM3's (the longest chains) first.
template <bool MANY, int PER>
__global__ __launch_bounds__(kRaggedThreads, MANY ? 4 : 3) void k_ragged_mixed(RaggedArgs r, uint32_t tiles)
{
    __shared__ RaggedLds L;
    __shared__ __align__(16) uint32_t ring[kChainRingWords<SM3>];
    const uint64_t base = uint64_t(xcd_contiguous(blockIdx.x % tiles, tiles)) * r.tile;
    if (blockIdx.x < tiles) ragged_tile<SM3, MANY, PER>(r, base, kNoLong, L, ring);
    else if (blockIdx.x < 2u * tiles) ragged_tile<SHA1, MANY, PER>(r, base, kNoLong, L, ring);
    else ragged_tile<MD5, MANY, PER>(r, base, kNoLong, L, ring);
}

// ---------------------------------------------------------------------------------------
// Batches of more tiles than the chip holds at once: the longest messages first
// ---------------------------------------------------------------------------------------
//
// A long message in a tile that starts late would end late.  Up to kLongGroups groups of 32
// messages, the longest by blocks x operations per block, are therefore picked out over the
// whole batch and hashed by chain pairs of their own in the launch's first workgroups; the
// tiles leave them out.

constexpr uint32_t kLongGroups = 512;  // two workgroups on each CU, beside two of the tiles'

__host__ __device__ constexpr uint32_t block_ops(int a) { return a == MD5 ? 292u : (a == SHA1 ? 446u : 923u); }  // on a chain

// Groups are numbered SM3's first: the algorithm of slot o.
__device__ __forceinline__ int long_slot(int o) { return o == 0 ? SM3 : (o == 1 ? SHA1 : MD5); }

__global__ __launch_bounds__(kRaggedThreads) void k_long_zero(LongWs w)
{
    const uint32_t t = blockIdx.x * kRaggedThreads + threadIdx.x, step = gridDim.x * kRaggedThreads;
    for (uint32_t i = t; i < 3 * kBins; i += step) { w.hist[i] = 0; w.cursor[i] = 0; }
    if (t == 0) w.meta->max_key = 0;
}

// Counts of the messages of at least min_key blocks, by algorithm and key.
__global__ __launch_bounds__(kRaggedThreads) void k_long_count(RaggedArgs r, int algo, LongWs w)
{
    __shared__ uint32_t top;
    if (threadIdx.x == 0) top = 0;
    __syncthreads();
    uint32_t mine = 0;
    const uint64_t step = uint64_t(gridDim.x) * kRaggedThreads;
    for (uint64_t i = uint64_t(blockIdx.x) * kRaggedThreads + threadIdx.x; i < r.n; i += step) {
        const uint64_t nb = block_count(r.lens[i]);
        if (nb < w.min_key || nb >= 0x80000000u) continue;
        const int a = r.algos ? int(r.algos[i]) : algo;
        if (a > SM3) continue;
        const uint32_t key = uint32_t(min<uint64_t>(nb, kBins - 1u));
        atomicAdd(&w.hist[uint32_t(a) * kBins + key], 1u);
        mine = max(mine, key);
    }
    if (mine) atomicMax(&top, mine);
    __syncthreads();
    if (threadIdx.x == 0 && top) atomicMax(&w.meta->max_key, top);
}

constexpr int kPickThreads = 1024;

// First position of each key, longest first, within its algorithm; then the smallest chain
// cost (blocks x operations) from which up the messages fit the groups.  One workgroup.
__global__ __launch_bounds__(kPickThreads) void k_long_pick(LongWs w)
{
    __shared__ uint32_t part[kPickThreads / 64];
    LongMeta *m = w.meta;
    const uint32_t lane = threadIdx.x % 64u, wave = threadIdx.x / 64u, top = m->max_key;
    const uint32_t nkeys = top >= w.min_key ? top - w.min_key + 1u : 0u, per = (nkeys + kPickThreads - 1) / kPickThreads;
    for (int a = 0; a < 3; ++a) {
        const uint32_t *hist = w.hist + uint32_t(a) * kBins;
        uint32_t local = 0;
        for (uint32_t k = 0; k < per; ++k) {
            const uint32_t x = threadIdx.x * per + k;
            if (x < nkeys) local += hist[top - x];
        }
        uint32_t sum = local;
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t up = __shfl_up(sum, d);
            if (lane >= uint32_t(d)) sum += up;
        }
        if (lane == 63) part[wave] = sum;
        __syncthreads();
        uint32_t run = sum - local;
        for (uint32_t v = 0; v < wave; ++v) run += part[v];
        for (uint32_t k = 0; k < per; ++k) {
            const uint32_t x = threadIdx.x * per + k;
            if (x < nkeys) {
                w.start[uint32_t(a) * kBins + top - x] = run;
                run += hist[top - x];
            }
        }
        __syncthreads();
    }
    __threadfence_block();
    __syncthreads();
    // messages of algorithm a whose cost reaches c, and the key that takes
    auto key_for = [&](int a, uint64_t c) {
        const uint64_t k = (c + block_ops(a) - 1) / block_ops(a);
        return uint32_t(min<uint64_t>(max<uint64_t>(k, w.min_key), 0xffffffffull));
    };
    auto messages = [&](int a, uint64_t c) {
        const uint32_t k = key_for(a, c);
        return k > top ? 0u : w.start[uint32_t(a) * kBins + k] + w.hist[uint32_t(a) * kBins + k];
    };
    auto fits = [&](uint64_t c) {
        uint32_t g = 0;
        for (int a = 0; a < 3; ++a) g += (messages(a, c) + kChainMessages - 1u) / kChainMessages;
        return g <= kLongGroups;
    };
    // the smallest c that fits, a thousandth of what is left of the range at a time
    uint64_t lo = 0, hi = uint64_t(kBins) * block_ops(SM3);  // hi fits: no message has that cost
    if (!fits(0)) {
        while (hi - lo > 1) {  // lo does not fit
            const uint64_t d = (hi - lo + kPickThreads) / (kPickThreads + 1u);
            const uint64_t c = min<uint64_t>(lo + d * (threadIdx.x + 1u), hi);
            const uint32_t nfit = uint32_t(__syncthreads_count(fits(c)));  // fits is monotone in c
            const uint64_t first = kPickThreads - nfit;                     // the first thread whose c fits
            hi = min<uint64_t>(lo + d * (first + 1u), hi);
            lo = min<uint64_t>(lo + d * first, hi - 1u);
        }
    } else {
        hi = 0;
    }
    if (threadIdx.x == 0) {
        uint32_t pos = 0, group = 0;
        for (int o = 0; o < 3; ++o) {
            const int a = long_slot(o);
            m->from[a] = key_for(a, hi);
            m->count[a] = messages(a, hi);
            m->pos[a] = pos;
            m->group[o] = group;
            pos += m->count[a];
            group += (m->count[a] + kChainMessages - 1u) / kChainMessages;
        }
        m->group[3] = group;
    }
}

__global__ __launch_bounds__(kRaggedThreads) void k_long_scatter(RaggedArgs r, int algo, LongWs w)
{
    const uint64_t step = uint64_t(gridDim.x) * kRaggedThreads;
    for (uint64_t i = uint64_t(blockIdx.x) * kRaggedThreads + threadIdx.x; i < r.n; i += step) {
        const uint64_t nb = block_count(r.lens[i]);
        if (nb < w.min_key || nb >= 0x80000000u) continue;
        const int a = r.algos ? int(r.algos[i]) : algo;
        if (a > SM3 || !is_long(uint32_t(nb), w.meta->from[a])) continue;
        const uint32_t bin = uint32_t(a) * kBins + uint32_t(min<uint64_t>(nb, kBins - 1u));
        w.sorted[w.meta->pos[a] + w.start[bin] + atomicAdd(&w.cursor[bin], 1u)] = uint32_t(i);
    }
}

// Group k of algorithm A's `groups`.  The 32 longest messages lead a group each, with the
// shortest of the long ones beside them, so that they soon run alone (a chain takes 10 %
// longer beside 31 others); the rest follow in order, 32 of near-equal length to a group, so
// that most groups end early and leave their places to the tiles.
template <int A>
__device__ __forceinline__ void long_group(const RaggedArgs &r, const LongWs &w, uint32_t k, uint32_t groups, RaggedLds &L,
                                           uint32_t *ring)
{
    const uint32_t lane = threadIdx.x % 64u, count = w.meta->count[A], lead = min(groups, kChainMessages);
    const uint32_t beside = min(lead * (kChainMessages - 1u), count - lead);  // of them, from the end of the order
    uint32_t at = kNoLong;
    if (lane < kChainMessages) {
        if (k >= lead) {
            const uint32_t x = lead + (k - lead) * kChainMessages + lane;
            if (x < count - beside) at = x;
        } else if (lane == 0) {
            at = k;
        } else {
            const uint32_t x = k + (lane - 1u) * lead;
            if (x < beside) at = count - 1u - x;
        }
    }
    if (lane == 0) L.simd[threadIdx.x / 64u] = wave_simd();
    if (threadIdx.x == 0) { L.group = group_on_cu(); L.sync.filled = 0; L.sync.taken = 0; }
    __syncthreads();
    chain_pair<A>(r, at != kNoLong ? w.sorted[w.meta->pos[A] + at] : kNoMessage, L, ring);
}

// The long groups' workgroups, then the tiles'.  ALGO: the batch's algorithm, or -1 for a
// mixed one (three workgroups a tile).
template <int ALGO>
__global__ __launch_bounds__(kRaggedThreads, 4) void k_long_tiles(RaggedArgs r, LongWs w, uint32_t tiles)
{
    __shared__ RaggedLds L;
    __shared__ __align__(16) uint32_t ring[kChainRingWords<ALGO < 0 ? int(SM3) : ALGO>];
    const LongMeta *m = w.meta;
    if (blockIdx.x < kLongGroups) {
        const uint32_t g = blockIdx.x;
        if (g >= m->group[3]) return;
        if constexpr (ALGO >= 0) long_group<ALGO>(r, w, g, m->group[3], L, ring);
        else if (g < m->group[1]) long_group<SM3>(r, w, g, m->group[1], L, ring);
        else if (g < m->group[2]) long_group<SHA1>(r, w, g - m->group[1], m->group[2] - m->group[1], L, ring);
        else long_group<MD5>(r, w, g - m->group[2], m->group[3] - m->group[2], L, ring);
        return;
    }
    const uint32_t b = blockIdx.x - kLongGroups;
    const uint64_t base = uint64_t(xcd_contiguous(b % tiles, tiles)) * r.tile;
    if constexpr (ALGO >= 0) ragged_tile<ALGO, true, kPerThread>(r, base, m->from[ALGO], L, ring);
    else if (b < tiles) ragged_tile<SM3, true, kPerThread>(r, base, m->from[SM3], L, ring);
    else if (b < 2u * tiles) ragged_tile<SHA1, true, kPerThread>(r, base, m->from[SHA1], L, ring);
    else ragged_tile<MD5, true, kPerThread>(r, base, m->from[MD5], L, ring);
}

// ---------------------------------------------------------------------------------------
// Fixed-length batches of few messages
// ---------------------------------------------------------------------------------------
//
// With at most 128 messages to a CU half its SIMDs would be idle and each wave's time is its
// instructions: one workgroup on each CU runs two chain pairs of up to 64 messages, their
// schedules on the other two SIMDs.  (Windows of 64 entries: the schedule wave works with all
// its lanes.)  1,000 x 4 KiB: SHA-1 84.9 us with a lane to a message, 64.2 so; SM3 172 and 127.

template <int A>
__global__ __launch_bounds__(kRaggedThreads) void k_fixed_chain(const uint8_t *__restrict__ msgs, uint64_t n, uint64_t len,
                                                               uint32_t per, uint8_t *__restrict__ out)
{
    constexpr uint32_t E = 64;
    __shared__ __align__(16) uint32_t ring[2][kChainRingWords<A, E>];
    __shared__ uint32_t tails[2][kChainTailWords<E>], simds[kRaggedThreads / 64];
    __shared__ ChainSync sync[2];
    const uint32_t lane = threadIdx.x % 64u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64u);
    if (lane == 0) simds[wave] = wave_simd();
    if (threadIdx.x < 2) sync[threadIdx.x] = ChainSync{0, 0};
    __syncthreads();
    // chain waves on two SIMDs, schedule waves on the other two (by wave number if the four
    // waves should not be on four SIMDs)
    uint32_t seen = 0;
#pragma unroll
    for (uint32_t w = 0; w < kRaggedThreads / 64; ++w) seen |= 1u << simds[w];
    const uint32_t role = __builtin_amdgcn_readfirstlane(seen == 15u ? simds[wave] : wave), pair = role % 2u;
    const uint64_t first = (uint64_t(xcd_contiguous(blockIdx.x, gridDim.x)) * 2u + pair) * per, i = first + lane;
    if (first >= n) return;  // both waves of the last pair
    const uint32_t blocks = lane < per && i < n ? uint32_t(block_count(len)) : 0u;
    if (role < 2u) {
        uint32_t s[8];
        __builtin_amdgcn_s_setprio(3);
        chain_run<A, E>(blocks, ring[pair], &sync[pair], s);
        if (blocks) store_digest<A>(out + i * Traits<A>::kDigest, s, Traits<A>::kDigest);
    } else {
        const uint64_t address = uint64_t(reinterpret_cast<uintptr_t>(msgs)) + (blocks ? i : first) * len;
        __builtin_amdgcn_s_setprio(2);
        chain_schedule<A, E, E>(address, len, blocks, ring[pair], tails[pair], &sync[pair]);
    }
}

Tiling ragged_tiling(uint64_t n, bool mixed, int algo)
{
    return tiling(n, mixed, device_simds() / 4u, !mixed && algo == MD5 ? kTileChainsMd5 : kTileChains);
}

// A form each for tiles of one message a thread, two and more: unrolled for eight, the short
// batches' launches spent a microsecond passing over code they had no messages for (300,007
// messages of 16 bytes in tiles of 512, MD5 / SHA-1 / SM3, us: 11.2 / 14.0 / 21.5 unrolled for
// eight, 10.6 / 13.4 / 20.7 for two).
template <int A> auto *ragged_form(uint64_t tile, bool few)
{
    return tile > 2u * kRaggedThreads ? k_ragged<A, true, kPerThread>
         : tile > kRaggedThreads      ? k_ragged<A, true, 2>
         : few                        ? k_ragged<A, false, 1>
                                      : k_ragged<A, true, 1>;
}

}  // namespace

hipError_t launch_ragged(const uint8_t *algos, int algo, const uint8_t *msgs, const uint64_t *offs, const uint64_t *lens,
                         uint64_t n, uint8_t *out, uint32_t stride, hipStream_t stream)
{
    const Tiling t = ragged_tiling(n, algos != nullptr, algo);
    const uint64_t tile = t.tile, tiles = t.tiles, per = t.per;
    if (tiles * per > 0x7fffffffull) return hipErrorInvalidConfiguration;
    const RaggedArgs r{msgs, offs, lens, algos, out, n, stride, uint32_t(tile)};
    const dim3 grid{uint32_t(tiles * per), 1, 1}, block{kRaggedThreads, 1, 1};
    // one wave to a SIMD (see few_waves); a mixed batch's workgroups have a third of a tile each
    // (12,000 / 16,384 messages of 16 KiB, us: 852 / 861 with the form for shared SIMDs, 725 / 728
    // without)
    const bool few = tiles * per * ((tile + 64u * per - 1) / (64u * per)) <= device_simds();
    if (algos) {
        hipLaunchKernelGGL((tile > 2u * kRaggedThreads ? k_ragged_mixed<true, kPerThread> : few ? k_ragged_mixed<false, 2> : k_ragged_mixed<true, 2>),
                           grid, block, 0, stream, r, uint32_t(tiles));
        return hipGetLastError();
    }
    auto *kernel = algo == MD5 ? ragged_form<MD5>(tile, few) : algo == SHA1 ? ragged_form<SHA1>(tile, few)
                 : algo == SM3 ? ragged_form<SM3>(tile, few) : nullptr;
    if (!kernel) return hipErrorInvalidValue;
    hipLaunchKernelGGL(kernel, grid, block, 0, stream, r);
    return hipGetLastError();
}

bool fixed_chain_applies(int algo, uint64_t n, uint64_t len, bool staged)
{
    // Where it was measured faster than a lane to a message (us, lane / chain): SM3 from three
    // blocks on (120 bytes: 14.7 / 13.4; 512: 28.3 / 24.9), SHA-1 from four (250 bytes: 13.2 /
    // 11.8; 120: 10.5 / 10.5), and past 32 messages to a pair, where a window is one block and
    // the schedules take longer than the rounds, from 32 (20,011 x 512: 16.0 / 17.3; x 4 KiB:
    // 89 / 79).  MD5, whose schedule is one addition to
    // a word, for its loads: from 64 blocks, up to 32 messages to a pair (144 x 2 KiB 27.2 / 27.0,
    // x 35,664 bytes 562 / 309; 12,000 x 4 KiB 58.8 / 48.1; 20,011 x 4 KiB 50.3 / 51.5).
    // The padding-only block of a length divisible by 64 does not count against a lane that has
    // its words formed on the scalar unit (SM3 of 128 bytes, up to 32,768 messages: 11.1-11.7 us
    // / 11.9-12.4; of 192 level).
    const uint64_t nb = block_count(len) - (staged && len % 64u == 0 ? 1u : 0u), cus = device_simds() / 4u;
    if (n > 128u * cus || nb >= 0x80000000u) return false;
    if (algo == MD5) return n <= 64u * cus && nb >= 64;
    return algo == SM3 ? nb >= 3 : algo == SHA1 && nb >= (n <= 64u * cus ? 4u : 32u);
}

hipError_t launch_fixed_chain(int algo, const uint8_t *msgs, uint64_t n, uint64_t len, uint8_t *out, hipStream_t stream)
{
    const uint64_t pairs = 2u * uint64_t(device_simds() / 4u);
    const uint32_t per = uint32_t((n + pairs - 1) / pairs);  // messages of a pair
    const dim3 grid{uint32_t((n + 2u * per - 1) / (2u * per)), 1, 1}, block{kRaggedThreads, 1, 1};
    if (algo == SHA1) hipLaunchKernelGGL(k_fixed_chain<SHA1>, grid, block, 0, stream, msgs, n, len, per, out);
    else if (algo == MD5) hipLaunchKernelGGL(k_fixed_chain<MD5>, grid, block, 0, stream, msgs, n, len, per, out);
    else if (algo == SM3) hipLaunchKernelGGL(k_fixed_chain<SM3>, grid, block, 0, stream, msgs, n, len, per, out);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

bool ragged_in_one_round(uint64_t n, bool mixed) { return ragged_tiling(n, mixed, SM3).rounds <= 1; }

hipError_t launch_ragged_long(const LongWs &w, const uint8_t *algos, int algo, const uint8_t *msgs, const uint64_t *offs,
                              const uint64_t *lens, uint64_t n, uint8_t *out, uint32_t stride, hipStream_t stream)
{
    const Tiling t = ragged_tiling(n, algos != nullptr, algo);
    if (t.tiles * t.per + kLongGroups > 0x7fffffffull) return hipErrorInvalidConfiguration;
    const RaggedArgs r{msgs, offs, lens, algos, out, n, stride, uint32_t(t.tile)};
    const dim3 block{kRaggedThreads, 1, 1}, sweep{device_simds(), 1, 1}, grid{uint32_t(kLongGroups + t.tiles * t.per), 1, 1};
    hipLaunchKernelGGL(k_long_zero, sweep, block, 0, stream, w);
    hipLaunchKernelGGL(k_long_count, sweep, block, 0, stream, r, algo, w);
    hipLaunchKernelGGL(k_long_pick, dim3(1), dim3(kPickThreads), 0, stream, w);
    hipLaunchKernelGGL(k_long_scatter, sweep, block, 0, stream, r, algo, w);
    if (algos) hipLaunchKernelGGL(k_long_tiles<-1>, grid, block, 0, stream, r, w, uint32_t(t.tiles));
    else if (algo == MD5) hipLaunchKernelGGL(k_long_tiles<MD5>, grid, block, 0, stream, r, w, uint32_t(t.tiles));
    else if (algo == SHA1) hipLaunchKernelGGL(k_long_tiles<SHA1>, grid, block, 0, stream, r, w, uint32_t(t.tiles));
    else if (algo == SM3) hipLaunchKernelGGL(k_long_tiles<SM3>, grid, block, 0, stream, r, w, uint32_t(t.tiles));
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace hb
