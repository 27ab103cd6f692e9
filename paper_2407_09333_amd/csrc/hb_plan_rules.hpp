// hb_plan_rules.hpp -- sizing rules that the host can check without a GPU: block counts,
// sort keys, the long-chain scratch region of a plan's wave, and the tiles of a packed batch.
// Free of HIP calls; compiled into the device kernels and into host-only checks alike.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__) || defined(__HIP__)
#define HB_HD __host__ __device__
#else
#define HB_HD
#endif

namespace hb {

constexpr uint32_t kBins = 16448;  // block-count keys per algorithm: key = min(nb, kBins - 1)

// Blocks of the padded L-byte message: the message, the 0x80 byte, zeros and the 8-byte
// length field fill floor((L + 8) / 64) + 1 blocks (RFC 1321 Sec. 3.1-3.2, FIPS 180-4
// Sec. 5.1.1, GB/T 32905 Sec. 5.2).
HB_HD inline uint64_t block_count(uint64_t len) { return (len + 8u) / 64u + 1u; }

// Sort key of an L-byte message: its block count, saturated at kBins - 1.  Every message
// of kBins - 1 blocks (about 1.05 MB) or more shares that key, so the bucketing sort leaves
// them in no particular order among themselves.
HB_HD inline uint32_t sort_key(uint64_t len)
{
    const uint64_t nb = block_count(len);
    return nb >= kBins ? kBins - 1 : uint32_t(nb);
}

// Scratch wave-blocks a long-chain wave needs: the largest block count among its `lanes`
// messages, len_at(l) giving lane l's length in sorted order.  Below the saturated key the
// sort is exact and descending, so lane 0 holds the largest; once lane 0's key is
// saturated the order is arbitrary and every lane is looked at.  The result is clamped to
// `limit`; a caller passing (scratch capacity + 1) reads `limit` as "cannot fit".
template <class LenAt>
HB_HD inline uint64_t wave_region_blocks(LenAt len_at, uint32_t lanes, uint64_t limit)
{
    const uint64_t len0 = len_at(0u);
    uint64_t r = block_count(len0);
    if (sort_key(len0) == kBins - 1)
        for (uint32_t l = 1; l < lanes; ++l) {
            const uint64_t b = block_count(len_at(l));
            r = b > r ? b : r;
        }
    return r < limit ? r : limit;
}

constexpr uint32_t kTileThreads = 256;  // four waves
constexpr uint32_t kTileMax = 2048;     // messages of a tile, at most
constexpr uint32_t kTileChains = 32;    // messages that a tile's chain pair takes, at most
constexpr uint32_t kTileChainsMd5 = 8;  // of MD5 messages of one length (kChainsAlike, hb_ragged.hip)

// How a packed batch is dealt out: messages per tile, tiles, workgroups per tile (one per
// algorithm), and how many times over its workgroups fill the chip.
struct Tiling {
    uint64_t tile, tiles, per, rounds;
};

// chains: kTileChainsMd5 for a batch of MD5 messages, else kTileChains.
inline Tiling tiling(uint64_t n, bool mixed, uint64_t cus, uint64_t chains = kTileChains)
{
    const uint64_t per = mixed ? 3u : 1u, wide = mixed ? 2u : 1u, slots = cus * 4u;
    const uint64_t rounds = (n * per + slots * kTileMax - 1) / (slots * kTileMax);
    const uint64_t one = (n + cus - 1) / cus, all = (n * per + slots * rounds - 1) / (slots * rounds);
    uint64_t tile;
    if (const uint64_t at_once = cus > per ? cus / per : 1u, few = (n + at_once - 1) / at_once; few <= chains * wide) {
        // One workgroup on each CU takes so few that its chain pair takes them all however alike
        // their lengths, and none is left to a lane of its own (of a mixed tile's 64 each
        // algorithm has about 21; of MD5's the pair takes eight).  In tiles of 64, half of 64 equal messages or more were:
        // plans of 64 messages of 64 KiB took, MD5 / SHA-1 / SM3, 613 / 1,314 / 2,689 us, and
        // take 564 / 842 / 1,837 so; 1,000 of 16 KiB 155 / 328 / 677 and 151 / 220 / 472.
        tile = few;
    } else if (one <= kTileThreads) {
        // Up to 256 messages to a workgroup while one on each CU takes them all, one wave to
        // a SIMD (64 to a workgroup and four workgroups to a CU would put the four busy waves
        // on one SIMD: 65,536 x 1 KiB MD5 43 us against 21).  A mixed batch's tiles are twice
        // as large, a workgroup hashing about a third of one: three times as large, half the
        // workgroups would have a few messages more than their four waves take at once.
        tile = (one + 63u) / 64u * 64u * wide;
    } else {
        // Then 256 up to four workgroups on each CU (a SIMD for each one's chain wave: with
        // five, two chains shared one), and past those as many as fill them once, or a whole
        // number of times: larger tiles sort better, but a last round that is half empty
        // costs more.  Past 512, one algorithm's tiles grow by a wave's 64 messages, so that
        // all four workgroups of a CU have work: by 256, three of 768 for some CUs and four
        // for others (600,011 messages of 16 bytes, MD5 / SHA-1 / SM3, us: 16.6 / 22.6 / 36.3,
        // so 15.5 / 20.9 / 32.0).  Up to 512 the whole step is faster (300,007: of 320 11.7 /
        // 14.7 / 22.7, of 512 10.6 / 13.4 / 20.7).
        const uint64_t step = mixed || all <= 512u ? 256u : 64u;
        tile = all < kTileThreads * wide ? kTileThreads * wide : (all + step - 1) / step * step;
        tile = tile < kTileMax ? tile : kTileMax;
    }
    return {tile, (n + tile - 1) / tile, per, rounds};
}

}  // namespace hb
