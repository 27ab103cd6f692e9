// Host check of the tiles that a packed batch is dealt out in (hb_plan_rules.hpp): they cover
// the batch, and a batch that one workgroup on each CU can take by chain pairs alone is dealt
// out so.
#include <cstdio>
#include <cstdlib>
#include <random>

#include "../../paper_2407_09333_amd/csrc/hb_plan_rules.hpp"

namespace {

void fail(const char *what, uint64_t n, bool mixed, uint64_t cus)
{
    const hb::Tiling t = hb::tiling(n, mixed, cus);
    std::printf("%s: n=%llu mixed=%d cus=%llu tile=%llu tiles=%llu\n", what, (unsigned long long)n, int(mixed),
                (unsigned long long)cus, (unsigned long long)t.tile, (unsigned long long)t.tiles);
    std::exit(1);
}

void check(uint64_t n, bool mixed, uint64_t cus)
{
    const hb::Tiling t = hb::tiling(n, mixed, cus), md5 = hb::tiling(n, mixed, cus, hb::kTileChainsMd5);
    if (!mixed && (n <= hb::kTileChainsMd5 * cus ? md5.tile > hb::kTileChainsMd5 : md5.tile % 64u != 0))
        fail("MD5", n, mixed, cus);
    if (t.tile == 0 || t.tile > hb::kTileMax || t.per != (mixed ? 3u : 1u)) fail("tile", n, mixed, cus);
    if (t.tiles * t.tile < n || (t.tiles - 1) * t.tile >= n) fail("tiles", n, mixed, cus);
    if (t.tiles * t.per > t.rounds * cus * 4u + t.per) fail("rounds", n, mixed, cus);
    if (n <= (mixed ? 2u : 1u) * hb::kTileChains * (cus / t.per) &&
        (t.tile > (mixed ? 2u : 1u) * hb::kTileChains || t.tiles * t.per > cus))
        fail("few messages", n, mixed, cus);
    // tiles past two messages a thread: the busiest CU's waves of 64 are within an eighth of
    // the mean, and one a workgroup
    const uint64_t waves = (t.tiles + cus - 1) / cus * ((t.tile + 63) / 64);
    if (!mixed && t.tile > 512 && double(waves) > 1.125 * double(n) / 64.0 / double(cus) + 4.0 * double(t.rounds))
        fail("busiest CU", n, mixed, cus);
}

}  // namespace

int main()
{
    std::mt19937_64 rng(5);
    for (uint64_t cus : {256u, 304u, 64u, 3u})
        for (bool mixed : {false, true}) {
            for (uint64_t n = 1; n <= 20'000; ++n) check(n, mixed, cus);
            for (int i = 0; i < 200'000; ++i) check(1 + (rng() >> (32 + rng() % 28)), mixed, cus);
            for (uint64_t k = 1; k <= 40; ++k)
                for (uint64_t d : {uint64_t(-1), uint64_t(0), uint64_t(1)}) check(k * cus * 64u + d, mixed, cus);
        }
    std::puts("tiling ok");
    return 0;
}
