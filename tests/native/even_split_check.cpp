// Host-side check of the reciprocal forms that a static split of whole blocks uses in place of the
// general split's divisions (internal.h): div_magic against x / d, and even_split against pre_split and
// suf_split for every worker, over random sizes up to the bounds they are used within (W <= 1024,
// slices x W < 2^31) and the small ones exhaustively; ExactDiv, whose
// bound stands at its definition, on both sides of quotients of some 200000 divisors.  Prints "ok <cases>" or the first failure.
#include <cstdio>
#include <cstdlib>
#include <random>

#include "internal.h"

using namespace fka;

static bool split_ok(int32_t W, int32_t P, int32_t S)
{
    const uint32_t m = magic_of((uint32_t)W);
    const int32_t b = S >= W ? P + S : S, bq = div_magic(b, W, m), br = b - bq * W;
    if (bq != b / W) return false;
    for (int32_t j = 0; j <= W; ++j) {
        const int32_t pre = even_split(j, P / W, P % W, m), joint = even_split(j, bq, br, m);
        if (pre != pre_split(j, W, P) || (S >= W ? joint - pre : joint) != suf_split(j, W, P, S)) return false;
    }
    return true;
}

int main(int argc, char **argv)
{
    const int cases = argc > 1 ? std::atoi(argv[1]) : 2000;
    std::mt19937_64 rng(4242);
    long n = 0;
    for (int32_t W = 1; W <= 24; ++W)
        for (int32_t P = 0; P <= 60; P += 1)
            for (int32_t S = 0; S <= 60; ++S, ++n)
                if (!split_ok(W, P, S)) return std::printf("FAIL W %d P %d S %d\n", W, P, S), 1;
    for (int c = 0; c < cases; ++c, ++n) {
        const int32_t W = 1 + (int32_t)(rng() % 1024);
        const int64_t most = (((int64_t)1 << 31) - 1) / W;
        const int32_t T = (int32_t)(rng() % (uint64_t)(c % 2 ? most : 5000) % (1 << 30)), P = T ? (int32_t)(rng() % T) : 0;
        if (!split_ok(W, P, T - P)) return std::printf("FAIL W %d P %d S %d\n", W, P, T - P), 1;
    }
    for (uint32_t d = 1; d <= 2048; ++d) {
        const uint32_t m = magic_of(d), last = 0xffffffffu / d;
        for (uint32_t x : {0u, 1u, d - 1, d, d + 1, last / d * d, last / d * d + d - 1, last - 1})
            if (x < 0x80000000u && (uint64_t)x * d < ((uint64_t)1 << 32) && div_magic((int32_t)x, (int32_t)d, m) != (int32_t)(x / d))
                return std::printf("FAIL %u / %u\n", x, d), 1;
        for (int k = 0; k < 200; ++k, ++n) {
            const uint32_t x = (uint32_t)(rng() % last) & 0x7fffffffu;
            if (div_magic((int32_t)x, (int32_t)d, m) != (int32_t)(x / d)) return std::printf("FAIL %u / %u\n", x, d), 1;
        }
    }
    for (int c = 0; c < 200000 + cases; ++c, ++n) {  // ExactDiv: any divisor, any 31-bit dividend
        const int64_t d = c < 4096 ? c + 1 : 1 + (int64_t)(rng() % ((uint64_t)1 << (1 + rng() % 31)));
        const ExactDiv e = exact_div(d);
        const int64_t top = 0x7fffffff, q = (int64_t)(rng() % (uint64_t)(top / d + 1)) * d;
        for (int64_t x : {(int64_t)0, d - 1, d, q - 1, q, q + d - 1, top / d * d - 1, top / d * d, top, (int64_t)(rng() & 0x7fffffff)})
            if (x >= 0 && x <= top && (int32_t)x / e != (int32_t)(x / d))
                return std::printf("FAIL %lld / %lld\n", (long long)x, (long long)d), 1;
    }
    std::printf("ok %ld\n", n);
    return 0;
}
