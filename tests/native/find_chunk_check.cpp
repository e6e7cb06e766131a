// Host-side check of find_chunk (internal.h), by which the tiled prefill's tail finds a group's branch: with
// the lengths that the groups were counted from, every group is found in the chunk that holds it, once
// and in order; with lengths that changed after the count (all gone, shrunk, grown), every search ends
// within the chunks there are and never stands past the last branch.  Prints "ok <cases>" or the first failure.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "internal.h"

using namespace fka;

// groups of the chunk at branch b
static int chunk_total(const std::vector<int> &groups, int b)
{
    int t = 0;
    for (int i = b; i < b + 64 && i < (int)groups.size(); ++i) t += groups[i];
    return t;
}

int main(int argc, char **argv)
{
    const int cases = argc > 1 ? std::atoi(argv[1]) : 500;
    std::mt19937_64 rng(99);
    long n = 0;
    for (int c = 0; c < cases; ++c) {
        const int branches = 1 + (int)(rng() % 300), pre = (int)(rng() % 8), first0 = (int)(rng() % branches);
        std::vector<int> groups(branches), now;
        for (int &g : groups) g = (int)(rng() % 6);
        int n_groups = pre;
        for (int b = first0; b < branches; ++b) n_groups += groups[b];
        for (int how = 0; how < 4; ++how) {
            now = groups;
            for (int &g : now) g = how == 0 ? g : how == 1 ? 0 : how == 2 ? (int)(rng() % (g + 1)) : g + (int)(rng() % 3);
            int first = first0, base = pre, held = chunk_total(groups, first0), loads = 0;
            for (int idx = pre; idx < n_groups; ++idx, ++n) {
                const bool found = find_chunk(idx, branches - 1, first, base, [&] { return held; },
                                              [&](int b) { held = chunk_total(now, b), ++loads; });
                if (loads > branches / 64 + 1 || first >= branches) return std::printf("FAIL past the last chunk, case %d\n", c), 1;
                if (found && (idx < base || idx - base >= held)) return std::printf("FAIL group %d, case %d\n", idx, c), 1;
                if (how == 0) {
                    int before = pre;
                    for (int b = first0; b < first; ++b) before += groups[b];
                    if (!found || before != base) return std::printf("FAIL group %d not found, case %d\n", idx, c), 1;
                }
            }
        }
    }
    std::printf("ok %ld\n", n);
    return 0;
}
