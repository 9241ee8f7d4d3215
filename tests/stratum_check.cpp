// Host check of stratum_coordinate: against the exact quotient N / (g 2^33), N = digit 2^33 + 2 r + 1,
// rounded to nearest even in integers.  Random strata, those next to the ends, and every kind of tie:
// digit 0 and 2 r + 1 a multiple of g with a quotient below 2^-8.
#include <cstdint>
#include <cstdio>
#include <random>

#include "stratum.h"

typedef unsigned __int128 u128;

// N / (g 2^33) rounded to 24 bits, nearest even
static float exact(uint64_t N, uint32_t g) {
    int e = 0;  // the quotient times 2^e has 24 bits before the point
    u128 num = N, den = (u128)g << 33;
    while (num < den << 23) num <<= 1, ++e;
    uint64_t q = (uint64_t)(num / den);
    const u128 rest = num % den;
    if (2 * rest > den || (2 * rest == den && (q & 1))) ++q;
    return std::ldexp((float)q, -e);
}

int main() {
    std::mt19937_64 rng(7);
    long n = 0, ties = 0;
    auto check = [&](uint32_t digit, uint32_t r, uint32_t g) {
        const uint64_t N = ((uint64_t)digit << 33) + 2 * (uint64_t)r + 1;
        const float a = mcubes::stratum_coordinate(digit, r, g), b = exact(N, g);
        ++n;
        if (a == b) return true;
        printf("digit %u r %u g %u: %a, exactly %a\n", digit, r, g, a, b);
        return false;
    };
    for (uint32_t g = 1; g <= 200; ++g) {
        for (int i = 0; i < 2000; ++i)
            if (!check((uint32_t)(rng() % g), (uint32_t)rng(), g)) return 1;
        for (uint32_t digit : {0u, g - 1})
            for (uint32_t r : {0u, 1u, 0x7fffffffu, 0x80000000u, 0xfffffffeu, 0xffffffffu})
                if (!check(digit, r, g)) return 1;
        // 2 r + 1 = g m, m odd in [2^24, 2^25): halfway between floats below 2^-8
        for (int i = 0; i < 2000 && (g & 1); ++i) {
            const uint64_t m = (1u << 24) + 2 * (rng() % (1u << 23)) + 1, odd = g * m;
            if (odd >> 33) continue;
            ++ties;
            if (!check(0, (uint32_t)(odd >> 1), g)) return 1;
        }
    }
    printf("ok %ld, ties %ld\n", n, ties);
    return ties > 10000 ? 0 : 1;
}
