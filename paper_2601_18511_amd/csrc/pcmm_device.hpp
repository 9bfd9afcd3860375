// Device-side helpers shared by the PCMM kernels: vector types, modular arithmetic, the exact
// double-precision reduction of the epilogue, compile-time loops.  Included by every .hip file of the
// library; everything here is inline device code.
#ifndef PCMM_DEVICE_HPP
#define PCMM_DEVICE_HPP

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>
#include <utility>

#include "pcmm_host.hpp"

namespace pcmm_device {

using pcmm_host::LimbConst;
using namespace pcmm_host::epi;

typedef int v4i __attribute__((ext_vector_type(4)));
typedef unsigned int v2u __attribute__((ext_vector_type(2)));

constexpr int kFrag = pcmm_host::kFragBytes;   // bytes of one 16 x 64 int8 MFMA operand fragment
constexpr int kXcd = 8;       // accelerator complex dies, each with its own L2

// strip, part of the rows and limb of work-group `bid` (pcmm_host::StripRaster, whose counts fit 32 bits); false: none.  Divisions of 64 bits
// took 0.15 us of every launch (the smallest products 5.0 -> 5.15 us).
__device__ __forceinline__ bool strip_of(const pcmm_host::StripRaster &r, uint32_t bid, int &strip, int &mpart, int &limb)
{
    const uint32_t i = bid / kXcd, per = (uint32_t)r.per_xcd, n = (uint32_t)r.nstrips, m = (uint32_t)r.mparts;
    const uint32_t part = r.whole ? i / per : 0, t = (bid % kXcd) * per + (i - part * per);
    if (t >= (uint32_t)r.total) return false;
    const uint32_t row = t / n;                       // limb, or (limb, part)
    strip = (int)(t - row * n);
    limb = (int)(r.whole ? row : row / m);
    mpart = (int)(r.whole ? part : row - (uint32_t)limb * m);
    return true;
}

// ------------------------------------------------------------------------------------------------
// modular helpers (device)
// ------------------------------------------------------------------------------------------------
// u < 2^64, mu = floor(2^64/q).  qhat = floor(u*mu / 2^64) satisfies u/q - 2 < qhat <= u/q, hence
// u - qhat*q is in [0, 2q) and one conditional subtraction gives the canonical residue.
__device__ __forceinline__ uint64_t barrett_u64(uint64_t u, uint64_t q, uint64_t mu)
{
    uint64_t qhat = __umul64hi(u, mu);
    uint64_t r = u - qhat * q;
    return r >= q ? r - q : r;
}

// x < q < 2^63, c < q, cs = floor(c * 2^64 / q): returns x*c mod q (Shoup's constant multiplication).
__device__ __forceinline__ uint64_t mulmod_shoup(uint64_t x, uint64_t c, uint64_t cs, uint64_t q)
{
    uint64_t qhat = __umul64hi(x, cs);
    uint64_t r = x * c - qhat * q;
    return r >= q ? r - q : r;
}

template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
// f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>), fully unrolled
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f)
{
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// bytes of four words -> four words, word d of the result holding byte d of each
__device__ __forceinline__ void transpose_bytes(const uint32_t (&y)[4], uint32_t (&t)[4])
{
    const uint32_t a0 = __builtin_amdgcn_perm(y[1], y[0], 0x05010400u), a1 = __builtin_amdgcn_perm(y[1], y[0], 0x07030602u);
    const uint32_t b0 = __builtin_amdgcn_perm(y[3], y[2], 0x05010400u), b1 = __builtin_amdgcn_perm(y[3], y[2], 0x07030602u);
    t[0] = __builtin_amdgcn_perm(b0, a0, 0x05040100u);
    t[1] = __builtin_amdgcn_perm(b0, a0, 0x07060302u);
    t[2] = __builtin_amdgcn_perm(b1, a1, 0x05040100u);
    t[3] = __builtin_amdgcn_perm(b1, a1, 0x07060302u);
}

// Balanced base-256 digits of sixteen residues: byte j of out[d] (as sixteen int8) is digit d of x[j].
// With Bias = sum_{i<D} 128 * 256^i, the bytes of x + Bias, each xor 0x80, read as int8, are digits s_i in [-128,127]
// with x = sum_i s_i 256^i (valid while x + Bias < 256^D).
template <int D>
__device__ __forceinline__ void digits16(const uint64_t (&x)[16], v4i (&out)[D])
{
    static_assert(D >= 4 && D <= 8, "four to eight digits");
    constexpr uint64_t bias = 0x8080808080808080ull >> (8 * (8 - D));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t lo[4], hi[4], t[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint64_t y = x[4 * i + r] + bias;
            lo[r] = (uint32_t)y;
            hi[r] = (uint32_t)(y >> 32);
        }
        transpose_bytes(lo, t);
#pragma unroll
        for (int d = 0; d < 4; ++d) out[d][i] = (int)(t[d] ^ 0x80808080u);
        if constexpr (D > 4) {
            transpose_bytes(hi, t);
#pragma unroll
            for (int d = 4; d < D; ++d) out[d][i] = (int)(t[d - 4] ^ 0x80808080u);
        }
    }
}

// Rounding to the nearest integer without the (slower) rounding instruction: for |x| < 2^51 the sum
// x + 1.5 * 2^52 has unit spacing, so its rounding is the rounding of x to an integer (ties to even), and
// subtracting the constant again is exact.  round_fma(h, s) rounds the exact product h s once.
constexpr double kRoundMagic = 6755399441055744.0;   // 1.5 * 2^52
__device__ __forceinline__ double round_fma(double h, double s) { return __builtin_fma(h, s, kRoundMagic) - kRoundMagic; }

// a b mod q for integers held in doubles, |a| <= q/2 + 1, |b| <= 4 q, 2^23 < q < 2^50; returns r = a b (mod q) with
// |r| <= q, and |r| <= 0.75 q + 1 when |b| <= 2 q.
//   h = RN(a b), l = a b - h exactly (fma);  |a b| <= 2 q^2 < 2^101, so |l| <= 2^48 and l is an integer
//   qh = round(h invq) = a b / q + eta:  |h invq| <= 2 q (1 + 2^-51) < 2^51, the two roundings (of h and of
//        invq) shift it by at most 2^-52 |a b| / q <= 2^-51 q < 0.5 (0.25 for |b| <= 2 q), so |eta| <= 1 (0.75)
//   fma(-qh, q, h) = (a b - qh q) - l: an integer of magnitude < 2^50 + 2^48 < 2^53, so exact; adding l is exact
// The same function serves the transforms of primes below 2^36 that never reduce their sums: |a| <= q/2 + 1,
// |b| <= 2^13 q.  Then |h invq| < 2^49 (the rounding trick holds), qh = a b / q + eta with
// |eta| <= 1/2 + 2^-52 2^12 q <= 0.5625, h and qh q are integers whose difference is below 0.5625 q + |l|,
// |l| <= 2^30: fma(-qh, q, h) and the addition of l are exact and |r| <= 0.5625 q.  A value that is only ever added
// to others through the twelve stages grows to at most 2^12 0.5625 q < 2^12 q < 2^48, differences to 2^13 q.
__device__ __forceinline__ double mulmod(double a, double b, double q, double invq)
{
    const double h = a * b;
    const double l = __builtin_fma(a, b, -h);
    const double qh = round_fma(h, invq);
    return __builtin_fma(-qh, q, h) + l;
}

// The canonical residue in [0, q) of an integer v = k q + s, 0 <= s < q, for q (|k| + 1) < 2^50:
//   x = fma(v, invq, invq / 2) = (k + (s + 1/2) / q) (1 + eps), |eps| < 2^-51 (the rounding of invq and of the fma),
//   and (s + 1/2) / q lies in [1/(2q), 1 - 1/(2q)]: |x - (k + (s + 1/2)/q)| < (|k| + 1) 2^-51 < 1/(2q), so floor(x) = k
//   and fma(-k, q, v) = s exactly.
__device__ __forceinline__ double canonical(double v, double q, double invq, double half_invq)
{
    return __builtin_fma(-__builtin_floor(__builtin_fma(v, invq, half_invq)), q, v);
}

// Exact reduction in double precision.  `a` holds E int32 accumulators; returns (sum_e a[e] 256^e) mod q
// in [0, q) for 2^23 < q < 2^50.
//
// The accumulators are grouped from the bottom into G-digit numbers, G = 3 in general:
// c_g = a[3g] + 2^8 a[3g+1] + 2^16 a[3g+2] (|c_g| < 2^47.01, exact in a double).  Horner in base
// B = 2^(8G) from the top group, one step per group:
//   X  = r B                         exact (power-of-two scaling)
//   qh = rint((X + c_g) / q)         the sum and the quotient are rounded: qh = (X + c_g)/q + eta with
//                                    |eta| <= 0.5 + 3.01 * 2^-53 * |X + c_g|/q  <=  0.6
//                                    (G = 3: |X + c_g|/q < 2^48.01 in the first step, where r = c_top is not
//                                    yet reduced, and < 2^24 afterwards)
//   u  = fma(-qh, q, X)              = -c_g - eta q exactly: an integer of magnitude below 2^53
//   r  = u + c_g                     = -eta q exactly, so |r| <= 0.6 q
// After the last group a negative r is lifted by q, which lands in [0, q) because |r| <= 0.6 q.
// Every operation is exact or feeds the rint whose error the exact fma absorbs, so the result is the
// canonical residue bit for bit.
//
// MODE 1 (E = 7 or 8 accumulators of magnitude < 2^28, q > 2^37): G = 4, so that two groups and a single
// Horner step remain.  |c_g| < 2^28 (1 + 2^8 + 2^16 + 2^24) < 2^52.01 is still exact, |X + c_g| < 2^84.02
// in the one step gives |X + c_g|/q < 2^47.1 and |eta| <= 0.5 + 3.01 * 2^-5.9 < 0.56, and
// |u| <= |c_g| + 0.56 q < 2^53.
// MODE 2 (in addition 257 |acc| < 2^31): neighbouring accumulators are first joined in int32,
// p = a[2i] + 2^8 a[2i+1], which halves the conversions to double.
// R outputs are reduced side by side, stage by stage: R independent dependency chains in the order the
// scheduler should issue them.
constexpr int group_size(int mode) { return mode == 0 ? 3 : 4; }

// the group numbers c_g
template <int E, int MODE, int R, int G>
__device__ __forceinline__ void group_f64(const int (&a)[R][E], double (&c)[G][R])
{
    constexpr int GS = group_size(MODE);             // accumulators per group
    static_assert(G == (E + GS - 1) / GS, "one number per group");
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const int b0 = GS * g;
        if constexpr (MODE == 2) {
            int p0[R], p1[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                p0[r] = b0 + 1 < E ? a[r][b0] + (int)((unsigned)a[r][b0 + 1] << 8) : a[r][b0];
                if (b0 + 2 < E) p1[r] = b0 + 3 < E ? a[r][b0 + 2] + (int)((unsigned)a[r][b0 + 3] << 8) : a[r][b0 + 2];
            }
#pragma unroll
            for (int r = 0; r < R; ++r) c[g][r] = (double)p0[r];
            if (b0 + 2 < E) {
#pragma unroll
                for (int r = 0; r < R; ++r) c[g][r] = __builtin_fma((double)p1[r], 65536.0, c[g][r]);
            }
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) c[g][r] = (double)a[r][b0];
#pragma unroll
            for (int i = 1; i < GS; ++i)
                if (b0 + i < E) {
#pragma unroll
                    for (int r = 0; r < R; ++r)
                        c[g][r] = __builtin_fma((double)a[r][b0 + i], (double)(1 << (8 * i)), c[g][r]);
                }
        }
    }
}

// Horner over the groups, then the lift to [0, q)
template <int G, int MODE, int R>
__device__ __forceinline__ void horner_f64(const double (&c)[G][R], double q, double invq, uint64_t (&res)[R])
{
    static_assert(G >= 2, "at least one Horner step");
    static_assert(MODE == 0 || G == 2, "groups of four are proved for a single Horner step");
    constexpr double B = MODE == 0 ? 16777216.0 : 4294967296.0;
    double rr[R];
#pragma unroll
    for (int r = 0; r < R; ++r) rr[r] = c[G - 1][r];
#pragma unroll
    for (int g = G - 2; g >= 0; --g) {
        double X[R], qh[R];
#pragma unroll
        for (int r = 0; r < R; ++r) X[r] = rr[r] * B;
#pragma unroll
        for (int r = 0; r < R; ++r) qh[r] = __builtin_rint((X[r] + c[g][r]) * invq);
#pragma unroll
        for (int r = 0; r < R; ++r) rr[r] = __builtin_fma(-qh[r], q, X[r]) + c[g][r];
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        // lift a negative remainder by q without a compare and selects: |rr| <= 0.6 q, so rr / q lies in (-1, 1) and
        // its floor is -1 for every negative rr (the product cannot round to zero: |rr| >= 1) and 0 otherwise
        const double v = __builtin_fma(-__builtin_floor(rr[r] * invq), q, rr[r]);
        // v is an integer in [0, 2^52): adding 2^52 places it in the low mantissa bits
        res[r] = (uint64_t)__double_as_longlong(v + 4503599627370496.0) & 0x000FFFFFFFFFFFFFull;
    }
}

template <int E, int MODE, int R>
__device__ __forceinline__ void reduce_f64(const int (&a)[R][E], double q, double invq, uint64_t (&res)[R])
{
    constexpr int G = (E + group_size(MODE) - 1) / group_size(MODE);
    double c[G][R];
    group_f64<E, MODE, R>(a, c);
    horner_f64<G, MODE, R>(c, q, invq, res);
}

// (sum_e a[e] 256^e) modulo two primes from the same accumulators (groups of three)
template <int E, int R>
__device__ __forceinline__ void reduce_f64_pair(const int (&a)[R][E], double q1, double invq1, double q2, double invq2,
                                                uint64_t (&res1)[R], uint64_t (&res2)[R])
{
    constexpr int G = (E + 2) / 3;
    double c[G][R];
    group_f64<E, 0, R>(a, c);
    horner_f64<G, 0, R>(c, q1, invq1, res1);
    horner_f64<G, 0, R>(c, q2, invq2, res2);
}

// (sum_e a[e] 256^e) mod q for any q < 2^62 in integers: the value is vlo + 2^32 vhi (+ 2^64 vtop for a ninth
// accumulator), each part of magnitude < 2^56, made positive by lc.off, reduced and joined by Shoup multiplications.
template <int E, int R>
__device__ __forceinline__ void reduce_int(const int (&a)[R][E], const LimbConst &lc, uint64_t (&res)[R])
{
#pragma unroll
    for (int r = 0; r < R; ++r) {
        int64_t vlo = 0, vhi = 0;
#pragma unroll
        for (int e = 0; e < (E < 8 ? E : 8); ++e) {
            const int64_t v = (int64_t)a[r][e];
            if (e < 4) vlo += v << (8 * e);
            else vhi += v << (8 * (e - 4));
        }
        const uint64_t rlo = barrett_u64((uint64_t)vlo + lc.off, lc.q, lc.mu);
        const uint64_t rhi = barrett_u64((uint64_t)vhi + lc.off, lc.q, lc.mu);
        res[r] = rlo + mulmod_shoup(rhi, lc.c32, lc.c32s, lc.q);
        if (res[r] >= lc.q) res[r] -= lc.q;
        if constexpr (E == 9) {
            const uint64_t rtop = barrett_u64((uint64_t)(int64_t)a[r][8] + lc.off, lc.q, lc.mu);
            res[r] += mulmod_shoup(rtop, lc.c64, lc.c64s, lc.q);
            if (res[r] >= lc.q) res[r] -= lc.q;
        }
    }
}

}  // namespace pcmm_device

#endif  // PCMM_DEVICE_HPP
