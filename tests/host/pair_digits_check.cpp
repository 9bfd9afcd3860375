// Host-only model of the joint digit split of two limbs (csrc/pcmm_host.hpp: pair_ok, pair_const), operation by operation
// as split_pair_kernel performs it: the digits represent an integer that is x1 mod q1 and x2 mod q2, and fit nine bytes.
#include <math.h>
#include <stdint.h>
#include <stdio.h>

#include <initializer_list>

#include "pcmm_host.hpp"

using namespace pcmm_host;

static int failures = 0;
#define CHECK(cond)                                                              \
    do {                                                                         \
        if (!(cond)) {                                                           \
            printf("line %d: check failed: %s\n", __LINE__, #cond);              \
            ++failures;                                                          \
        }                                                                        \
    } while (0)

static uint64_t residue(__int128 x, uint64_t q)
{
    const __int128 r = x % (__int128)q;
    return (uint64_t)(r < 0 ? r + q : r);
}

static void check_value(const PairConst &c, uint64_t q1, uint64_t q2, uint64_t x1, uint64_t x2)
{
    const double magic = 6755399441055744.0;
    const double dx = (double)x2 - (double)x1;
    const double h = c.inv * dx, l = fma(c.inv, dx, -h), qh = fma(h, c.invq2, magic) - magic;
    const double v = fma(-qh, c.q2, h) + l + c.s;
    const double td = fma(-floor(fma(v, c.invq2, c.half_invq2)), c.q2, v);
    CHECK(td >= 0 && td < c.q2);
    const uint64_t t = (uint64_t)td;
    const uint32_t tl = (uint32_t)t, th = (uint32_t)(t >> 32) & 0xFu, ql = (uint32_t)q1, qhi = (uint32_t)(q1 >> 32);
    const uint64_t s = x1 + c.bias_mod_q1;
    const uint64_t p0 = (uint64_t)tl * ql + (uint32_t)s;
    const uint64_t p1 = (uint64_t)tl * qhi + (uint64_t)th * ql + (p0 >> 32) + (s >> 32);
    const uint32_t y2 = (uint32_t)(p1 >> 32) + th * qhi;
    CHECK(y2 <= 255);
    const uint32_t y[3] = {(uint32_t)p0, (uint32_t)p1, y2};
    __int128 X = 0;
    for (int d = kPairDigits - 1; d >= 0; --d) X = X * 256 + (int8_t)(((y[d / 4] >> (8 * (d % 4))) & 0xFF) ^ 0x80);
    CHECK(residue(X, q1) == x1 && residue(X, q2) == x2);
}

int main()
{
    // the largest odd pair below 2^36, numbers of 36, 35, 34, 33, 32 and 31 bits (31: the smallest that take five digits)
    const uint64_t qs[] = {68719476735ull, 68719476733ull, 68719476503ull, 68718428161ull, 34359738641ull, 34359738421ull,
                           17179869209ull, 8589934609ull, 4294967311ull, 4294967357ull,
                           4294967291ull, 4294967279ull, 2147483659ull, 2147483647ull, 2139062149ull, 2139062145ull};
    const int n = sizeof(qs) / sizeof(qs[0]);
    uint64_t r = 88172645463325252ull;
    int accepted = 0;
    for (int a = 0; a < n; ++a)
        for (int b = 0; b < n; ++b) {
            if (!pair_ok(qs[a], qs[b])) continue;
            ++accepted;
            const PairConst c = pair_const(qs[a], qs[b]);
            for (int i = 0; i < 20016 && !failures; ++i) {
                uint64_t x[2];
                for (int k = 0; k < 2; ++k) {
                    const uint64_t q = k ? qs[b] : qs[a];
                    r ^= r << 13; r ^= r >> 7; r ^= r << 17;
                    const int edge = (i >> (2 * k)) & 3;
                    x[k] = i >= 16 ? r % q : (edge == 0 ? 0 : (edge == 1 ? q - 1 : (edge == 2 ? q / 2 : 1)));
                }
                check_value(c, qs[a], qs[b], x[0], x[1]);
            }
        }
    CHECK(accepted >= 20);
    CHECK(!pair_ok(68718428161ull, 68718428161ull));                    // one modulus twice: not coprime
    CHECK(!pair_ok((1ull << 36) + 1, 68718428161ull));                  // 37 bits
    CHECK(!pair_ok(4294967291ull, 68718428161ull));                     // 32 and 36 bits
    CHECK(!pair_ok(68718428161ull, 8589934609ull));                     // q1 >= 2 q2
    // the plan pairs limbs only where nine digits replace ten, and its scratch covers both layouts
    const uint64_t q36[5] = {68719476733ull, 68718428161ull, 68719476503ull, 68719476731ull, 68719476735ull};
    Geometry g;
    for (int64_t nc : {1, 15, 16, 17, 31, 32, 33, 100, 8192})
        for (int32_t L = 1; L <= 5; ++L) {
            CHECK(plan_geometry(300, 129, nc, L, q36, 36, 8, 0, &g) == PCMM_OK);
            CHECK(g.pairs == (L % 2 ? 0 : L / 2) && g.pair_ntiles * 16 >= nc);   // small: an odd number of limbs stays single
            const size_t pair_bytes = (size_t)g.pairs * g.nkb * g.pair_ntiles * kPairDigits * kFragBytes;
            const size_t single_bytes = (size_t)(L - 2 * g.pairs) * g.nkb * g.ntiles * g.NT * g.D * kFragBytes;
            CHECK(pair_bytes + single_bytes <= g.ad_bytes);
        }
    CHECK(plan_geometry(300, 128, 100, 2, q36, 36, 8, 0, &g) == PCMM_OK && g.pairs == 0);      // short contraction
    CHECK(plan_geometry(300, 300, 100, 2, q36, 36, 16, 0, &g) == PCMM_OK && g.pairs == 0);     // two weight slices
    // an odd number of limbs pairs from 2.5 10^10 products a limb on (600 rows more than M), and the scratch covers the pairs and the single limb
    CHECK(plan_geometry(5000, 1000, 4464, 3, q36, 36, 8, 0, &g) == PCMM_OK && g.pairs == 0);
    CHECK(plan_geometry(5000, 1000, 4465, 1, q36, 36, 8, 0, &g) == PCMM_OK && g.pairs == 0);
    for (int64_t nc : {4465, 4480, 4481, 4497, 32768})
        for (int32_t L : {3, 5}) {
            CHECK(plan_geometry(5000, 1000, nc, L, q36, 36, 8, 0, &g) == PCMM_OK && g.pairs == L / 2);
            CHECK((size_t)g.nkb * kFragBytes * (g.pairs * g.pair_ntiles * kPairDigits + g.ntiles * g.NT * g.D) <= g.ad_bytes);
        }
    // pairs of short contractions: output rows of 2 KiB at a time as with single limbs, up to 16 m-tiles; beyond those no
    // pairs where the rows of C start inside a line
    CHECK(plan_geometry(4096, 2048, 8192, 2, q36, 36, 8, 0, &g) == PCMM_OK && g.pairs == 1 && g.pair_gn * 16 == g.gn * g.NT * 16);
    CHECK(plan_geometry(4096, 2049, 8192, 2, q36, 36, 8, 0, &g) == PCMM_OK && g.pair_gn == 8);
    CHECK(plan_geometry(4097, 2048, 8192, 2, q36, 36, 8, 0, &g) == PCMM_OK && g.pairs == 1 && g.pair_gn == 8);
    CHECK(plan_geometry(4097, 768, 8192, 2, q36, 36, 8, 0, &g) == PCMM_OK && g.pairs == 1);
    CHECK(plan_geometry(4097, 768, 8191, 2, q36, 36, 8, 0, &g) == PCMM_OK && g.pairs == 0);
    CHECK(plan_geometry(4096, 768, 8191, 2, q36, 36, 8, 0, &g) == PCMM_OK && g.pairs == 1);
    CHECK(plan_geometry(4097, 769, 8191, 2, q36, 36, 8, 0, &g) == PCMM_OK && g.pairs == 1);
    // every size of prime that takes five digits pairs, none that takes four or six
    for (int bits = 24; bits <= 41; ++bits) {
        const uint64_t top[2] = {((uint64_t)1 << bits) - 1, ((uint64_t)1 << bits) - 3};
        CHECK(plan_geometry(300, 300, 100, 2, top, bits, 8, 0, &g) == PCMM_OK);
        CHECK(g.pairs == (bits >= 31 && bits <= 36 ? 1 : 0) && (g.pairs == 0 || g.D == 5));
    }
    const uint64_t low31[2] = {2139062145ull - 2, 2139062145ull - 4}, edge31[2] = {2139062145ull, 2139062143ull};
    CHECK(plan_geometry(300, 300, 100, 2, low31, 31, 8, 0, &g) == PCMM_OK && g.D == 4 && g.pairs == 0);
    CHECK(plan_geometry(300, 300, 100, 2, edge31, 31, 8, 0, &g) == PCMM_OK && g.D == 5 && g.pairs == 1);
    const uint64_t same[2] = {68718428161ull, 68718428161ull};
    CHECK(plan_geometry(300, 300, 100, 2, same, 36, 8, 0, &g) == PCMM_OK && g.pairs == 0);
    CHECK(plan_geometry(128, 20000, 32768, 2, q36, 36, 8, 0, &g) == PCMM_OK && g.pairs == 0);  // nine planes beyond 4 GiB
    if (failures) {
        printf("%d checks failed\n", failures);
        return 1;
    }
    printf("limb pairs: all checks held\n");
    return 0;
}
