// The run's square root and quotients against sqrt and / of the host, from
// seeds as good as the hardware's (2^-22 off either way): random inputs, and
// quotients next to the middle between two doubles.
// Prints "<square roots off> <quotients off> <hard quotients off> <hard>".
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <random>

#include "bearing.h"

using namespace fmdp;

static bool planted;                                   // the iteration's own reciprocal, not refined

static double seed(double r2, std::mt19937_64 &rng) {
    const double d = std::ldexp(2.0 * (double)(rng() >> 11) * 0x1p-53 - 1.0, -22);
    return (double)((1.0L + d) / std::sqrt((long double)r2));
}

static Bearing from(double r2, double y) {
    Bearing v = bearing(r2, y);
    if (planted) {
        const double a = r2 * y, h = 0.5 * y, e = std::fma(-h, a, 0.5), h1 = std::fma(h, e, h);
        v.inv = h1 + h1;
    }
    return v;
}

int main(int argc, char **argv) {
    planted = argc > 1 && std::atoi(argv[1]) != 0;
    std::mt19937_64 rng(11);
    std::uniform_real_distribution<double> u(-1.0, 1.0);
    long root = 0, quot = 0, hard = 0, n_hard = 0;
    for (int i = 0; i < 500000; ++i) {
        const double s = std::ldexp(1.0, (int)(rng() % 40) - 20), bx = s * u(rng), by = 40.0 * s * u(rng);
        const double r2 = std::fma(bx, bx, by * by);
        const Bearing v = from(r2, seed(r2, rng));
        const double br = std::sqrt(r2);
        root += v.br != br;
        quot += bearing_quotient(bx, v) != bx / br;
        quot += bearing_quotient(by, v) != by / br;
    }
    // br = B 2^e, B odd of 53 bits; M B = b 2^54 + d, M odd of 54 bits and d
    // small: b / B lies d / B units of the 54th bit from the middle M
    const uint64_t mask = (1ull << 54) - 1;
    for (int i = 0; i < 200000; ++i) {
        const uint64_t B = (1ull << 52) | (rng() & ((1ull << 52) - 1)) | 1u;
        uint64_t inv = B;                              // 1 / B modulo 2^64 (Newton)
        for (int k = 0; k < 6; ++k) inv *= 2 - B * inv;
        for (int d = -5; d <= 5; d += 2) {
            const uint64_t M = (inv * (uint64_t)(int64_t)d) & mask;
            if (M < (1ull << 53)) continue;
            const __int128 p = (__int128)M * B - d;
            const double b = (double)(uint64_t)(p >> 54);
            const double br = std::ldexp((double)B, (int)(rng() % 40) - 60), x = b * (br / (double)B);
            const double r2 = br * br;                 // sqrt of it, rounded, is br again
            if (std::sqrt(r2) != br) continue;
            const Bearing v = from(r2, seed(r2, rng));
            root += v.br != br;
            hard += bearing_quotient(x, v) != x / br;
            ++n_hard;
        }
    }
    std::printf("%ld %ld %ld %ld\n", root, quot, hard, n_hard);
    return 0;
}
