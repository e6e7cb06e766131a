// Host-side check of the tiled prefill's split of its key tiles (tail_share in internal.h): over all
// small and many random splits, the ranges' shares of the tail are contiguous in some order, cover it
// exactly once, and no range has more tiles than the fairest split of all tiles that leaves the prefix's
// where they are.  Prints "ok <cases>" or the first failure.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "internal.h"

using namespace fka;

static bool share_ok(int32_t PT, int32_t RP, int32_t R, int32_t tail)
{
    TileSplit s{};
    s.ranges = exact_div(R);
    s.extra = exact_div(std::max(1, R - RP));
    s.pre_each = PT / RP;
    s.pre_more = PT % RP;
    std::vector<char> seen((size_t)tail, 0);
    int64_t total = 0;
    int32_t most = 0, most_prefix = 0;
    for (int32_t r = 0; r < R; ++r) {
        const int32_t pre = r < RP ? s.pre_each + (r < s.pre_more ? 1 : 0) : 0;
        int32_t t0, n;
        tail_share(s, RP, R, tail, r, t0, n);
        if (n < 0 || (n > 0 && (t0 < 0 || t0 + n > tail))) return false;
        for (int32_t t = t0; t < t0 + n; ++t)
            if (seen[t]++) return false;
        total += n;
        most = std::max(most, pre + n);
        most_prefix = std::max(most_prefix, pre);
    }
    return total == tail && most <= std::max(most_prefix, (PT + tail + R - 1) / R);
}

int main(int argc, char **argv)
{
    const int cases = argc > 1 ? std::atoi(argv[1]) : 2000;
    std::mt19937_64 rng(4243);
    long n = 0;
    for (int32_t PT = 0; PT <= 12; ++PT)
        for (int32_t R = 1; R <= 14; ++R)
            for (int32_t RP = 1; RP <= std::min(R, std::max(1, PT)); ++RP)
                for (int32_t tail = 0; tail <= 40; ++tail, ++n)
                    if (!share_ok(PT, RP, R, tail)) return std::printf("FAIL PT %d RP %d R %d tail %d\n", PT, RP, R, tail), 1;
    for (int c = 0; c < cases; ++c, ++n) {
        const int32_t PT = (int32_t)(rng() % 2050), R = 1 + (int32_t)(rng() % 256), tail = (int32_t)(rng() % (c % 2 ? 40 : 5000));
        const int32_t RP = 1 + (int32_t)(rng() % (uint64_t)std::min(R, std::max(1, PT)));
        if (!share_ok(PT, RP, R, tail)) return std::printf("FAIL PT %d RP %d R %d tail %d\n", PT, RP, R, tail), 1;
    }
    std::printf("ok %ld\n", n);
    return 0;
}
