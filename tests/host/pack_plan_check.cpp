// Host-only check of the ballot pack's plan (csrc/pack_plan.h): for many sources, walk every wave of one image's workgroups
// through the functions the launcher and the kernel use and check that
//   - every tile of the rows and every group of 64 channels is taken by exactly one wave, tiles of at most 64 positions,
//   - tiles cover the row, groups the channels,
//   - the launch stays below 2^32 threads, whatever the number of images (up to 2^31 - 1 output words);
// that neither this plan nor that of the kernel through LDS takes an image beyond the kernels' 32-bit arithmetic; and that measured calls go to the kernel that is faster on them.
// Prints "mismatches: N"; exit status 0 = none.  With an argument and lines "element bytes, address, outer, channels, source channels, inner" on
// stdin: the vectors of a row in the kernel through LDS (0: another kernel's call) and whether its loads pass the caches' lines by.
#include "pack_plan.h"

#include <cstdio>
#include <vector>

using namespace bcnn;

static long check(int esz, int64_t outer, int64_t channels, int64_t inner, long* taken)
{
    const BallotPlan p = plan_ballot(esz, 0, outer, channels, channels, inner);
    if (p.nv == 0) return 0;
    ++*taken;
    long bad = 0;
    const int64_t positions = (int64_t)p.nv * 16 / esz;
    if (positions > 64 || positions * p.tiles < inner || 64ll * p.groups < channels) ++bad;
    if (p.blocks_per_image * outer > MAX_BLOCKS_256 || p.blocks_per_image * outer < 1) {
        if (!bad) printf("launch of %lld workgroups: %d bytes [%lld][%lld][%lld]\n", (long long)(p.blocks_per_image * outer), esz,
                         (long long)outer, (long long)channels, (long long)inner);
        ++bad;
    }
    std::vector<int> seen((size_t)p.tiles * p.groups, 0);
    for (int64_t at = 0; at < p.blocks_per_image; ++at)
        for (int wave = 0; wave < 4; ++wave) {
            int tile, g;
            if (!ballot_place((int)at, wave, p.tw_shift, p.groups, p.tiles, tile, g)) continue;
            if (tile < 0 || g < 0) { ++bad; continue; }
            ++seen[(size_t)tile * p.groups + g];
        }
    for (int n : seen)
        if (n != 1) ++bad;
    return bad;
}

// What both kernels compute in 32 bits of a source that a plan takes: an image's output by offsets of which one, 0x7FFFFF00, lies
// past every buffer, channels and waves by number.
static long check_addresses(int esz, int64_t outer, int64_t channels, int64_t inner, long* staged)
{
    const bool lds = staged_vectors(esz, 0, outer, channels, channels, inner) != 0;
    const bool ballot = plan_ballot(esz, 0, outer, channels, channels, inner).nv != 0;
    *staged += lds;
    if (!lds && !ballot) return 0;
    const int64_t words = (channels + 31) / 32;
    const bool fits = inner * words * 4 <= 0x7FFFFF00 && channels + 64 <= 0x7FFFFFFF && outer * ((channels + 63) / 64) <= 0x7FFFFFFF;
    if (!fits)
        printf("image beyond 32 bits: %s, %d bytes [%lld][%lld][%lld]\n", lds ? "through LDS" : "ballot", esz, (long long)outer, (long long)channels,
               (long long)inner);
    return fits ? 0 : 1;
}

int main(int argc, char**)
{
    if (argc > 1) {
        int esz;
        long long src, outer, channels, source, inner;
        while (scanf("%d %lld %lld %lld %lld %lld", &esz, &src, &outer, &channels, &source, &inner) == 6)
            printf("%d %d\n", staged_vectors(esz, (uintptr_t)src, outer, channels, source, inner), (int)staged_streams(esz, inner * esz, outer * source * inner * esz));
        return 0;
    }
    long bad = 0, taken = 0, staged = 0;
    for (int esz : {1, 2, 4})
        for (int64_t channels : {33ll, 64ll, 1000ll, 1ll << 20, (1ll << 24) - 64, 1ll << 24, 272696320ll, 275000000ll, 1ll << 28, (1ll << 31) - 64, 1ll << 31, 1ll << 32, 1ll << 33})
            for (int64_t inner : {5, 9, 16, 31, 32, 49, 63, 64, 100, 784})
                for (int64_t outer : {1ll, 2ll, 7ll, 600ll, 2048ll, 1ll << 20})
                    if (outer * inner <= 0x7FFFFFFF / ((channels + 31) / 32)) bad += check_addresses(esz, outer, channels, inner, &staged);
    if (staged < 100) ++bad;
    const int64_t counts[] = {1, 2, 3, 4, 8, 20, 31, 32, 33, 64, 65, 100, 128, 192, 256, 257, 320, 512, 1000, 1024, 2048, 4096};
    for (int esz : {1, 2, 4})
        for (int64_t channels : counts)
            for (int64_t inner = 1; inner <= 260; inner += inner < 70 ? 1 : 13)
                for (int64_t outer : {1ll, 2ll, 7ll, 64ll, 300ll, 2048ll, 5000ll, 1ll << 20, (1ll << 24) - 1, 1ll << 24, 1ll << 26, 1ll << 29}) {
                    if (outer * inner * ((channels + 31) / 32) > 0x7FFFFFFF) continue;   // refused by the entry point
                    bad += check(esz, outer, channels, inner, &taken);
                }
    if (taken < 1000) ++bad;
    // calls that the other kernels are faster on, by 1.1 to 50 times, and some that this one is
    const struct { int esz; int64_t outer, channels, inner; bool ballot; } routes[] = {
        {1, 5000000, 2, 2, false}, {4, 2222222, 3, 3, false}, {2, 416666, 16, 3, false}, {1, 104166, 64, 3, false}, {1, 208333, 48, 2, false},
        {4, 312500, 32, 2, false}, {4, 21428, 2, 7, false}, {1, 156250, 2, 64, false}, {1, 39062, 32, 16, false}, {4, 6510, 96, 32, false},
        {4, 244, 64, 64, false}, {2, 256, 1024, 49, true}, {4, 1024, 1024, 9, true}, {4, 1562, 64, 3, true}, {4, 1, 64, 196, true},
        {2, 39062, 8, 64, true}, {1, 19531, 256, 4, true}, {4, 64, 64, 9, true}, {2, 25000, 32, 25, true},
    };
    for (const auto& r : routes)
        if ((plan_ballot(r.esz, 0, r.outer, r.channels, r.channels, r.inner).nv != 0) != r.ballot) {
            printf("route: %d bytes [%lld][%lld][%lld]\n", r.esz, (long long)r.outer, (long long)r.channels, (long long)r.inner);
            ++bad;
        }
    // sources that are read past the caches' lines: [outer][channels][inner]
    const struct { int esz; int64_t outer, channels, inner; bool streams; } loads[] = {
        {2, 256, 1024, 49, false}, {2, 2000, 1024, 49, false}, {2, 3009, 1024, 49, false}, {2, 3010, 1024, 49, true}, {1, 8000, 512, 49, false}, {1, 12038, 512, 49, true},
        {4, 83, 1024, 49, false}, {4, 84, 1024, 49, true}, {4, 600, 256, 28, false}, {4, 10533, 256, 28, true}, {4, 2000, 1024, 9, false},
    };
    for (const auto& r : loads)
        if (!staged_vectors(r.esz, 0, r.outer, r.channels, r.channels, r.inner) ||
            staged_streams(r.esz, r.inner * r.esz, r.outer * r.channels * r.inner * r.esz) != r.streams) {
            printf("loads: %d bytes [%lld][%lld][%lld]\n", r.esz, (long long)r.outer, (long long)r.channels, (long long)r.inner);
            ++bad;
        }
    const struct { int s; int64_t channels, m; bool eight; } pools[] = {
        {2, 8, 1, true}, {2, 2048, 100, true}, {3, 64, 324, false}, {4, 64, 19528, false}, {4, 8, 585, false},
        {3, 16, 138834, true}, {4, 8, 156212, true}, {5, 8, 1 << 20, false}, {1, 8, 1 << 20, false},
    };
    for (const auto& r : pools)
        if (pool_by_eight(r.s, r.channels, r.m) != r.eight) { printf("pool: %d %lld %lld\n", r.s, (long long)r.channels, (long long)r.m); ++bad; }
    const struct { int64_t outer, channels, source; bool eight; } rows[] = {
        {1, 9, 9, false}, {2, 130, 65, false}, {8, 9, 9, true}, {8, 33, 33, true}, {8, 21, 7, false}, {3000, 301, 301, true}, {40000, 2048, 2048, true}, {8, 2049, 2049, false},
    };
    for (const auto& r : rows)
        if (ragged8_applies(r.outer, r.channels, r.source) != r.eight) { printf("rows: %lld %lld\n", (long long)r.outer, (long long)r.channels); ++bad; }
    const struct { int s; int64_t channels, m; bool four; } ragged[] = {
        {2, 99, 49, true}, {2, 3, 100000, false}, {4, 5, 1, true}, {1, 99, 784, false}, {1, 99, 62720, true}, {8, 99, 980, false}, {8, 99, 9800, true}, {1, 3, 1 << 20, false},
    };
    for (const auto& r : ragged)
        if (pool_ragged_by_four(r.s, r.channels, r.m) != r.four) { printf("ragged pool: %d %lld %lld\n", r.s, (long long)r.channels, (long long)r.m); ++bad; }
    printf("plans: %ld\nmismatches: %ld\n", taken, bad);
    return bad ? 1 : 0;
}
