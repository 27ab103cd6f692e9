// hb_chain.hpp -- a pair of waves of one workgroup that runs up to 32 long messages.
//
// A message's blocks must be compressed one after another, and a wave that has its SIMD to
// itself issues one instruction per four cycles or slower, so a long message takes its
// block count times the instructions of one block, whatever else the chip has free.  Here
// one wave (the chain wave) runs only what depends on the chaining value -- the rounds, 923
// of SM3's 1,350 instructions a block, 446 of SHA-1's 614, 292 of MD5's 340 -- and another
// (the schedule wave) does the rest ahead of it: it reads the message blocks, pads the last
// ones, expands the schedule words and hands them over in LDS.
//
// The LDS ring has a few windows of E entries (32 or 64), an entry holding one block's words.
// A window covers the next E / m blocks of each message, m being the number of messages still
// running rounded up to a power of two, so a single message is read 2 KiB at a time by 32
// lanes, and the latency of its loads is paid once: the schedule wave loads two windows
// ahead of the one it expands.  Both waves derive the windows from the same block counts.
#pragma once

#include <type_traits>

#include "hb_long.hpp"
#include "hb_plan_rules.hpp"

namespace hb {

constexpr uint32_t kChainMessages = kTileChains;  // of a pair, at most, where a batch has more than pairs for all

// Windows in the ring: MD5's schedules take about as long as its rounds, so its schedule
// wave needs the slack of a third.
template <int A> constexpr uint32_t kChainSlots = A == MD5 ? 3 : 2;

// 4-byte words of LDS the ring takes for algorithm A.
template <int A, uint32_t E = kChainMessages> constexpr uint32_t kChainRingWords = kChainSlots<A> * E * SchedWords<A>::kN;

// Hand-over counters, in LDS, zero at the start.
struct ChainSync {
    uint32_t filled;  // windows the schedule wave has written
    uint32_t taken;   // windows the chain wave has read
};

// One window of the messages with nb blocks (one per lane, 0 in the lanes past them):
// blocks first .. first + (E >> shift) - 1 of lanes 0 .. (1 << shift) - 1; none left when
// `more` is false.
struct ChainWindow {
    uint32_t shift;
    bool more;
};

__device__ __forceinline__ ChainWindow chain_window(uint32_t nb, uint32_t first)
{
    const uint64_t live = __ballot(nb > first);
    ChainWindow w;
    w.more = live != 0;
    const uint32_t top = 63u - uint32_t(__builtin_clzll(live | 1u));  // last live lane
    w.shift = top ? 32u - uint32_t(__builtin_clz(top)) : 0u;
    return w;
}

__device__ __forceinline__ void chain_wait(const uint32_t *counter, uint32_t at_least)
{
    while (int32_t(__hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) - at_least) < 0)
        __builtin_amdgcn_s_sleep(1);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ void chain_post(uint32_t *counter, uint32_t value)
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    if (__lane_id() == 0) __hip_atomic_store(counter, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The schedule words of one block, four at a time as they are formed: put(g, a, b, c, d) for
// word group g.  The barriers keep the compiler from forming them all first, which SM3's 128
// would not fit the registers for.
template <int A, class Put> __device__ __forceinline__ void schedule_groups(const uint32_t M[16], Put put)
{
    if constexpr (A == MD5) {
        constexpr const uint32_t *T = kMd5T;
#pragma unroll
        for (int g = 0; g < 16; ++g) {
            uint32_t o[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i = 4 * g + q, j = i & 15;
                o[q] = M[i < 16 ? j : (i < 32 ? (1 + 5 * j) & 15 : (i < 48 ? (5 + 3 * j) & 15 : (7 * j) & 15))] + T[i];
            }
            put(g, o[0], o[1], o[2], o[3]);
        }
    } else if constexpr (A == SHA1) {
        uint32_t W[16];
#pragma unroll
        for (int t = 0; t < 16; ++t) W[t] = M[t];
#pragma unroll
        for (int g = 0; g < 20; ++g) {
            uint32_t o[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int t = 4 * g + q;
                if (t >= 16)
                    W[t & 15] = rotl<1>(bitop3<TT_XOR3>(W[(t - 3) & 15], W[(t - 8) & 15], W[(t - 14) & 15]) ^ W[t & 15]);
                o[q] = W[t & 15] + (t < 20 ? 0x5a827999u : (t < 40 ? 0x6ed9eba1u : (t < 60 ? 0x8f1bbcdcu : 0xca62c1d6u)));
            }
            put(g, o[0], o[1], o[2], o[3]);
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
        uint32_t W[68];
#pragma unroll
        for (int j = 0; j < 16; ++j) W[j] = M[j];
#pragma unroll
        for (int g = 0; g < 16; ++g) {
#pragma unroll
            for (int i = 4 * g + 4; i < 4 * g + 8; ++i) {
                if (i < 16) continue;
                const uint32_t x = bitop3<TT_XOR3>(W[i - 16], W[i - 9], rotl<15>(W[i - 3]));
                W[i] = bitop3<TT_XOR3>(bitop3<TT_XOR3>(x, rotl<15>(x), rotl<23>(x)), rotl<7>(W[i - 13]), W[i - 6]);
            }
            const uint32_t *w = W + 4 * g;
            put(g, w[0] ^ w[4], w[1] ^ w[5], w[2] ^ w[6], w[3] ^ w[7]);
            put(16 + g, w[0], w[1], w[2], w[3]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// One lane's block of a window, loaded but not yet scheduled.
struct ChainFetch {
    uint32_t raw[17];  // whole blocks only: the last, partial ones wait in LDS (chain_tails)
    uint32_t sel, whole, nb;  // its message: selector, whole blocks, all blocks
    uint32_t blk;
    uint32_t shift;    // the window's (wave-uniform)
    bool more;         // there is such a window (wave-uniform)
};

// LDS words for the partial blocks and the lengths of up to M messages.
template <uint32_t M = kChainMessages> constexpr uint32_t kChainTailWords = 19 * M;

// The schedule wave.  Lane l < M <= E brings message l (its address and length, and its block
// count nb; nb = 0 past the last); message 0 has at least one whole block.  Two windows are in
// flight ahead of the one being scheduled: with 17 to 32 messages a window is one block of
// each, 0.6 to 1.8 us of the chain wave's time.  So that the waits for them can be counted,
// every fetch is the same five loads, made by every lane: a lane without a whole block in the
// window reads message 0's first, and the dwords of each message's partial block are read at
// the start and kept in LDS (`tails`).
template <int A, uint32_t E = kChainMessages, uint32_t M = kChainMessages>
__device__ __forceinline__ void chain_schedule(uint64_t address, uint64_t length, uint32_t nb, uint32_t *ring,
                                               uint32_t *tails, ChainSync *sync)
{
    constexpr int N = SchedWords<A>::kN;
    const uint32_t lane = __lane_id();
    const uint32_t e = lane % E;  // the entry this lane fills (lanes E.. only shadow)
    const Msg m0 = make_msg<A>(reinterpret_cast<const uint8_t *>(uint64_t(__shfl(address, 0))), 64);
    if (nb) {
        const Msg m = make_msg<A>(reinterpret_cast<const uint8_t *>(address), length);
        const uint32_t lim = length % 64u ? uint32_t(length % 64u) + m.r : 0u;  // dword k is read iff 4k < lim
        const HB_GLOBAL uint32_t *q = m.p + length / 64u * 16u;
        uint32_t t[17];
#pragma unroll
        for (uint32_t k = 0; k < 17; ++k) t[k] = 4 * k < lim ? q[k] : 0u;
#pragma unroll
        for (uint32_t k = 0; k < 17; ++k) tails[k * M + lane] = t[k];
        tails[17 * M + lane] = uint32_t(length);
        tails[18 * M + lane] = uint32_t(length >> 32);
    }
    Msg m = m0;
    uint32_t mnb = 0, mwhole = 0, shift = 0xffffffffu, first = 0, k = 0;
    // the next window: entry e gets block first + (e >> shift) of message e mod (1 << shift)
    auto fetch = [&](ChainFetch &f) {
        const ChainWindow w = chain_window(nb, first);
        if (w.more && w.shift != shift) {  // deal the messages out anew
            shift = w.shift;
            const int l = int(e & ((1u << shift) - 1u));
            m = make_msg<A>(reinterpret_cast<const uint8_t *>(uint64_t(__shfl(address, l))), __shfl(length, l));
            mnb = lane < E ? uint32_t(__shfl(nb, l)) : 0u;
            mwhole = uint32_t(m.len / 64u);
        }
        const uint32_t blk = first + (e >> shift);
        f.more = w.more;
        f.shift = shift;
        f.sel = m.sel;
        f.blk = blk;
        f.whole = mwhole;
        f.nb = w.more ? mnb : 0u;
        const bool whole = blk < f.nb && blk < mwhole;
        const HB_GLOBAL uint32_t *q = whole ? m.p + uint64_t(blk) * 16u : m0.p;
        const uint32_t r = whole ? m.r : m0.r;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const u32x4 v = *reinterpret_cast<const HB_GLOBAL u32x4_a4 *>(q + 4 * g);
            f.raw[4 * g] = v.x; f.raw[4 * g + 1] = v.y; f.raw[4 * g + 2] = v.z; f.raw[4 * g + 3] = v.w;
        }
        f.raw[16] = q[r ? 16 : 15];
        first += E >> shift;
        __builtin_amdgcn_sched_barrier(0);  // one fetch's loads before the next one's
    };
    auto produce = [&](ChainFetch &f) {
        uint32_t words[16];
        const bool have = f.more, on = f.blk < f.nb;
        if (__any(on && f.blk >= f.whole)) {
            const uint32_t l = e & ((1u << f.shift) - 1u);
            const uint64_t len = tails[17 * M + l] | uint64_t(tails[18 * M + l]) << 32;
            // message bytes from the block's start (any value past the end stands for none)
            const int32_t rem = f.blk < f.whole ? 64 : (f.blk == f.whole ? int32_t(len % 64u) : -1);
            uint32_t raw[17], t[17];
#pragma unroll
            for (uint32_t i = 0; i < 17; ++i) t[i] = tails[i * M + l];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < 17; ++i) raw[i] = rem >= 64 ? f.raw[i] : (rem > 0 ? t[i] : 0u);
            Msg of{};
            of.sel = f.sel;
            of.bits = len << 3;
            assemble_block<Traits<A>::kBE>(of, rem, f.blk + 1 == f.nb, raw, words);
        } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) words[i] = perm(f.raw[i + 1], f.raw[i], f.sel);
        }
        fetch(f);
        // the wait comes first so that each word goes to the ring as it is formed: held back,
        // SM3's 128 would not fit the registers
        if (have && k >= kChainSlots<A>) chain_wait(&sync->taken, k - kChainSlots<A> + 1u);
        if (on) {
            u32x4 *slot = reinterpret_cast<u32x4 *>(ring) + (k % kChainSlots<A>) * (N / 4) * E + e;
            schedule_groups<A>(words, [&](int g, uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
                slot[g * int(E)] = u32x4{a, b, c, d};
            });
        }
        if (have) chain_post(&sync->filled, ++k);
    };
    // no way out between the two: on a path that skipped one's loads, their number in flight
    // could not be known and every wait would be for all of them
    ChainFetch f0, f1;
    fetch(f0);
    fetch(f1);
    while (f0.more) {
        produce(f0);
        produce(f1);
    }
}

// A quarter of a block's rounds, and the schedule words they take (SM3: W' and W).
template <int A> constexpr int kChunkRounds = A == SHA1 ? 20 : 16;
template <int A> constexpr int kChunkWords = A == SM3 ? 32 : kChunkRounds<A>;

// Quarter C of the rounds (MD5 steps) on the working variables v from their words.
template <int A, int C> __device__ __forceinline__ void quarter(uint32_t v[8], const uint32_t *ww)
{
    if constexpr (A == MD5) {
        constexpr int sh[4][4] = {{7, 12, 17, 22}, {5, 9, 14, 20}, {4, 11, 16, 23}, {6, 10, 15, 21}};
        constexpr uint32_t tt[4] = {TT_CH, TT_MD5_G, TT_XOR3, TT_MD5_I};
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const uint32_t t = v[0] + bitop3<tt[C]>(v[1], v[2], v[3]) + ww[i];
            const uint32_t b = v[1] + __builtin_amdgcn_alignbit(t, t, 32u - uint32_t(sh[C][i & 3]));
            v[0] = v[3]; v[3] = v[2]; v[2] = v[1]; v[1] = b;
        }
    } else if constexpr (A == SHA1) {
#pragma unroll
        for (int i = 0; i < 20; ++i) {
            const uint32_t f = bitop3<C == 0 ? TT_CH : (C == 2 ? TT_MAJ : TT_XOR3)>(v[1], v[2], v[3]);
            const uint32_t T = rotl<5>(v[0]) + f + (v[4] + ww[i]);
            v[4] = v[3]; v[3] = v[2]; v[2] = rotl<30>(v[1]); v[1] = v[0]; v[0] = T;
        }
    } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) {  // ww: W' of the sixteen rounds, then their W
            const int j = 16 * C + i;
            const uint32_t a12 = rotl<12>(v[0]);
            const uint32_t ss1 = rotl<7>(a12 + v[4] + sm3_tj(j));
            const uint32_t ff = j < 16 ? bitop3<TT_XOR3>(v[0], v[1], v[2]) : bitop3<TT_MAJ>(v[0], v[1], v[2]);
            const uint32_t gg = j < 16 ? bitop3<TT_XOR3>(v[4], v[5], v[6]) : bitop3<TT_CH>(v[4], v[5], v[6]);
            const uint32_t tt1 = xad(ss1, a12, v[3] + ww[i] + ff);
            const uint32_t tt2 = gg + v[7] + ss1 + ww[16 + i];
            v[3] = v[2]; v[2] = rotl<9>(v[1]); v[1] = v[0]; v[0] = tt1;
            v[7] = v[6]; v[6] = rotl<19>(v[5]); v[5] = v[4]; v[4] = sm3_p0(tt2);
        }
    }
}

// The words of quarter C of an entry: q is the entry's place in the window's first word
// group.
template <int A, int C, uint32_t E> __device__ __forceinline__ void load_chunk(const u32x4 *q, uint32_t *ww)
{
    constexpr int kGroupsPer = kChunkRounds<A> / 4;  // SM3: of W', then as many of W
#pragma unroll
    for (int g = 0; g < kChunkWords<A> / 4; ++g) {
        const int group = g < kGroupsPer ? kGroupsPer * C + g : 16 + kGroupsPer * C + g - kGroupsPer;
        const u32x4 x = q[group * int(E)];
        ww[4 * g] = x.x; ww[4 * g + 1] = x.y; ww[4 * g + 2] = x.z; ww[4 * g + 3] = x.w;
    }
}

// The chain wave: digest state s of message `lane` (nb blocks; nb = 0 past the last).  One
// block of every message at a time; lanes whose message has ended run along on another
// lane's words and keep their state, so that there is no divergent branch.  Each quarter's
// words are read while the quarter before it runs, the last one's over the first words of
// the next block -- after a window's last block, of the next window if that is filled by
// then, asked for a quarter earlier: waiting for it between blocks costs 150-250 ns.
template <int A, uint32_t E = kChainMessages>
__device__ __forceinline__ void chain_run(uint32_t nb, const uint32_t *ring, ChainSync *sync, uint32_t s[8])
{
    constexpr uint32_t kWindow = SchedWords<A>::kN / 4 * E;  // in 16-byte units
    const u32x4 *base = reinterpret_cast<const u32x4 *>(ring);
    const uint32_t lane = __lane_id();
    uint32_t top = nb;
    for (int d = 32; d > 0; d >>= 1) top = max(top, uint32_t(__shfl_xor(top, d)));
    const uint32_t longest = __builtin_amdgcn_readfirstlane(top);
    init_state<A>(s);
    uint32_t b0[kChunkWords<A>], b1[kChunkWords<A>];
    uint32_t blk = 0, k = 0, at = 0, slot = 0;
    bool ready = false;  // b0 holds the first words of window k
    // one block, the first words of entry `next` read on the way; LAST: those of `next` if
    // window k is filled, else this entry's again, for nothing
    auto block = [&](auto last, uint32_t next) {
        constexpr bool LAST = decltype(last)::value;
        const u32x4 *q = base + at;
        uint32_t v[8], filled = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = s[i];
        // the barriers keep each quarter's loads ahead of the rounds they run under
        load_chunk<A, 1, E>(q, b1);
        __builtin_amdgcn_sched_barrier(0);
        quarter<A, 0>(v, b0);
        __builtin_amdgcn_sched_barrier(0);
        load_chunk<A, 2, E>(q, b0);
        __builtin_amdgcn_sched_barrier(0);
        quarter<A, 1>(v, b1);
        __builtin_amdgcn_sched_barrier(0);
        load_chunk<A, 3, E>(q, b1);
        if constexpr (LAST) filled = __hip_atomic_load(&sync->filled, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __builtin_amdgcn_sched_barrier(0);
        quarter<A, 2>(v, b0);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (LAST) {
            // arithmetic and no branch: past one, the compiler would put this before the rounds
            const uint32_t missing = uint32_t(int32_t(__builtin_amdgcn_readfirstlane(filled) - (k + 1u)) >> 31);
            ready = missing == 0;
            at += ~missing & (next - at);
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        } else {
            at = next;
        }
        load_chunk<A, 0, E>(base + at, b0);
        __builtin_amdgcn_sched_barrier(0);
        quarter<A, 3>(v, b1);
        const bool live = nb > blk;
#pragma unroll
        for (int i = 0; i < Traits<A>::kWords; ++i) {
            const uint32_t n = A == SM3 ? s[i] ^ v[i] : s[i] + v[i];
            s[i] = live ? n : s[i];
        }
        ++blk;
    };
    for (ChainWindow w = chain_window(nb, 0); w.more;) {
        const uint32_t per = 1u << w.shift;
        if (!ready) {
            chain_wait(&sync->filled, k + 1u);
            at = slot * kWindow + (lane & (per - 1u));
            load_chunk<A, 0, E>(base + at, b0);
        }
        ++k;
        slot = slot + 1u == kChainSlots<A> ? 0u : slot + 1u;
        // (no block past the longest message's last)
        for (uint32_t left = min(E >> w.shift, longest - blk) - 1u; left; --left) block(std::false_type{}, at + per);
        w = chain_window(nb, blk + 1u);
        block(std::true_type{}, slot * kWindow + (lane & ((1u << w.shift) - 1u)));
        if (w.more) chain_post(&sync->taken, k);
    }
}

}  // namespace hb
