// Host-side check of the bitmap's arithmetic (pc_device.h: pc_w30_*, the integers
// prime to 30) and of the near quotients that place a prime's multiples in it,
// against plain remainders.
#include <cmath>
#include <cstdio>
#include <random>

#include "pc_device.h"

static int fails = 0;
#define CHECK(cond, ...)                                        \
    do {                                                        \
        if (!(cond) && fails++ < 20) {                          \
            std::printf("FAIL %s:%d ", __FILE__, __LINE__);     \
            std::printf(__VA_ARGS__);                           \
            std::printf("\n");                                  \
        }                                                       \
    } while (0)

static bool prime_to_30(uint32_t n) { return n % 2 && n % 3 && n % 5; }

int main()
{
    // every offset of the largest segment (2^19 bits span 1966080 integers) and past it
    uint32_t le = 0;
    for (uint32_t d = 0; d < 1u << 21; d++) {
        if (prime_to_30(d)) {
            CHECK(pc_w30_bit(d) == le, "bit of %u", d);
            CHECK(pc_w30_int(le) == d, "integer of bit %u", le);
            le++;
        }
        CHECK(pc_w30_le(d) == le, "count to %u", d);
    }
    for (uint32_t log2s : {15u, 16u, 18u, 19u})
        CHECK(pc_w30_le((uint32_t)pc_seg_span(log2s) - 1) == 1u << log2s, "span of 2^%u bits", log2s);
    for (uint32_t j = 0; j <= 30; j++) {
        uint32_t n = j;
        while (!prime_to_30(n))
            n++;
        CHECK(pc_w30_next(j) == n, "next from %u", j);
    }
    // pc_quot_near: a reciprocal one unit off on either side, exact multiples
    // and their neighbours, over p of every length and quotients to 2^17
    std::mt19937_64 rng(30);
    for (int i = 0; i < 4000000; i++) {
        const uint32_t p = std::max<uint32_t>(7, (uint32_t)(rng() >> (40 + rng() % 21)));
        const uint32_t q = (uint32_t)(rng() >> 32) % std::min<uint32_t>(1u << 17, (1u << 30) / p);
        const uint32_t r = i % 4 == 0 ? 0 : i % 4 == 1 ? p - 1 : i % 4 == 2 ? 1 : (uint32_t)(rng() % p);
        const float inv = 1.0f / (float)p;
        for (float rp : {inv, std::nextafterf(inv, 0.0f), std::nextafterf(inv, 1.0f)})
            CHECK(pc_quot_near(q * p + r, p, rp) == q, "%u / %u", q * p + r, p);
    }
    // pc_rem_near over n < 2^47
    for (int i = 0; i < 4000000; i++) {
        const uint32_t p = std::max<uint32_t>(7, (uint32_t)(rng() >> (33 + rng() % 28)));
        const uint64_t q = (rng() >> (17 + rng() % 40)) / p;
        const uint64_t n = q * p + (i % 4 == 0 ? 0 : i % 4 == 1 ? p - 1 : i % 4 == 2 ? p / 2 : rng() % p);
        if (n < 1ull << 47)
            CHECK(pc_rem_near(n, (double)n, p, 1.0 / p) == n % p, "%llu mod %u", (unsigned long long)n, p);
    }
    if (!fails)
        std::printf("OK\n");
    return fails != 0;
}
