// PCMv for MI355X (gfx950): the ring products of the decode-time plaintext-ciphertext matrix-vector
// multiplication,
//     out_j[m][c] = sum_{k<Kp} pt[m][k] * ct_j[k][c]   in  Z_{q_j}[X]/(X^N + 1),   c in {a, b},
// for every RNS limb j (Section 3.2: in decoding the matrix-matrix products become matrix-vector products;
// Table "he-operators": ring degree 4096, coefficient encoding; Section 5.3: the plaintext polynomials are
// kept in the NTT domain).  The packing of the weights into plaintext polynomials and the extraction of the
// useful coefficients afterwards belong to the algorithm the paper adopts by reference and are not here.
//
// Kernels:
//   ntt_kernel / ntt_blocked_kernel   forward negacyclic NTT of polynomials: the plaintexts once, at plan time ("model
//                     conversion"), and the 2 Kp L ciphertext polynomials of every run
//   mac_intt_kernel / mac_intt_blocked_kernel   per (limb, m): pointwise multiply-accumulate of the NTT-domain plaintexts
//                     with both ciphertext components, inverse NTT of the two sums, store as uint64 residues
// The *blocked* kernels serve the paper's ring degree, 4096, and 2048 and 1024: sixteen values per thread in registers, four stages per pass, two
// trips through LDS per transform; the multiply-accumulate kernel runs as persistent work-groups fed from a queue.
// The others serve every other power of two, one radix-2 stage per pass over LDS.
//
// Arithmetic.  MI355X runs double-precision vector arithmetic at full rate while 64-bit integer
// multiplication costs many quarter-rate 32-bit multiplies, so residues are held as balanced integers in
// doubles and multiplied exactly with fused multiply-adds (mulmod below); the bound q < 2^50 comes from
// there.  In the general kernels a polynomial lives in LDS as N doubles and each radix-2 stage is one pass over
// LDS (Gentleman-Sande inverse butterflies, bit-reversed order in, natural order out, twiddle inv[groups + group]).
//
// HBM traffic per run: the NTT-domain plaintexts are read once (8 Mp Kp N L bytes, the dominant term for
// long contractions) and the output written once (16 Mp N L bytes).
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <new>
#include <type_traits>
#include <vector>

#include "../../include/pcmm.h"
#include "pcmm_device.hpp"
#include "pcmm_hip_util.hpp"
#include "pcmv_host.hpp"

namespace {

using pcmm_device::canonical;
using pcmm_device::mulmod;
using pcmm_device::round_fma;

using pcmm_device::kXcd;

constexpr int kThreads = 256;
constexpr int kQueueStride = 32;   // words between the work queues' counters: each in a 128-byte line of its own

// the representative of an integer |v| < 2^52 modulo q (q > 2^23) with magnitude at most q/2 (+1 when the quotient
// rounds the other way)
__device__ __forceinline__ double reduce(double v, double q, double invq)
{
    return __builtin_fma(-round_fma(v, invq), q, v);
}

// Forward negacyclic NTT in place on N doubles in LDS (natural order in, bit-reversed order out).
// Cooley-Tukey butterflies with the powers of psi merged in: stage with m groups uses fwd[m + group].
// Inputs of magnitude <= q/2; outputs of magnitude <= 1.375 q.
__device__ __forceinline__ void ntt_forward(double *s, const double *__restrict__ fwd, int N, double q, double invq)
{
    int lt = 31 - __builtin_clz((unsigned)N);             // log2 of the butterfly span t
    for (int m = 1; m < N; m <<= 1) {
        --lt;
        const int t = 1 << lt;
        for (int bf = threadIdx.x; bf < N / 2; bf += kThreads) {
            const int i = bf >> lt, jj = bf & (t - 1);
            const int j = (i << (lt + 1)) + jj;
            const double S = fwd[m + i];
            const double U = reduce(s[j], q, invq);
            const double V = mulmod(S, s[j + t], q, invq);
            s[j] = U + V;
            s[j + t] = U - V;
        }
        __syncthreads();
    }
}

struct LimbDev {
    double q, invq, n_inv;
    double pad;
};

// Forward NTT of polynomials.  SRC = 0: uint64 residues in [0, q) (ciphertext polynomials, laid out
// [L][polys_per_limb][N]); SRC = 1: signed 32-bit plaintext coefficients shared by all limbs ([polys_per_limb][N]).
// Output: doubles [L][polys_per_limb][N], magnitudes <= q/2 + 1, bit-reversed order (plaintexts times 1/N mod q).
template <int SRC>
__global__ __launch_bounds__(kThreads) void ntt_kernel(const void *__restrict__ src, double *__restrict__ dst,
                                                       const double *__restrict__ fwd_tables, const LimbDev *__restrict__ lc,
                                                       int N, int64_t polys_per_limb)
{
    extern __shared__ double lds[];
    const int64_t p = blockIdx.x;
    const int limb = (int)(p / polys_per_limb);
    const int64_t within = p % polys_per_limb;
    const double q = lc[limb].q, invq = lc[limb].invq;
    for (int n = threadIdx.x; n < N; n += kThreads) {
        double v;
        if (SRC == 0) {
            const uint64_t x = static_cast<const uint64_t *>(src)[p * N + n];
            v = __builtin_fma((double)(uint32_t)(x >> 32), 4294967296.0, (double)(uint32_t)x);   // exact: x < 2^50
        } else {
            v = (double)static_cast<const int32_t *>(src)[within * N + n];
        }
        lds[n] = reduce(v, q, invq);
    }
    __syncthreads();
    ntt_forward(lds, fwd_tables + (int64_t)limb * N, N, q, invq);
    // the plaintexts carry the factor 1/N of the inverse transform that follows the pointwise products
    const double scale = lc[limb].n_inv;
    for (int n = threadIdx.x; n < N; n += kThreads) {
        double r = reduce(lds[n], q, invq);
        if (SRC == 1) r = reduce(mulmod(scale, r, q, invq), q, invq);
        dst[p * N + n] = r;
    }
}

// One work-group per (limb, m): acc_c = sum_k ptn[m][k] (.) ctn[k][c] for c = a, b, inverse NTT of both,
// times 1/N, canonical residues out.
//   ptn [L][Mp][Kp][N] doubles, ctn [L][Kp][2][N] doubles (both |.| <= q/2 + 1), out [L][Mp][2][N] uint64
__global__ __launch_bounds__(kThreads) void mac_intt_kernel(const double *__restrict__ ptn, const double *__restrict__ ctn,
                                                            uint64_t *__restrict__ out, const double *__restrict__ inv_tables,
                                                            const LimbDev *__restrict__ lc, int N, int64_t Mp, int Kp)
{
    extern __shared__ double lds[];          // two polynomials: [0, N) component a, [N, 2N) component b
    const int64_t blk = blockIdx.x;
    const int limb = (int)(blk / Mp);
    const int64_t m = blk % Mp;
    const double q = lc[limb].q, invq = lc[limb].invq;
    const double *pt = ptn + ((int64_t)limb * Mp + m) * Kp * N;
    const double *ct = ctn + (int64_t)limb * Kp * 2 * N;
    for (int n = threadIdx.x; n < N; n += kThreads) {
        double acc_a = 0.0, acc_b = 0.0;
        for (int k = 0; k < Kp; ++k) {
            const double w = pt[(int64_t)k * N + n];
            acc_a = reduce(acc_a + mulmod(w, ct[((int64_t)k * 2 + 0) * N + n], q, invq), q, invq);
            acc_b = reduce(acc_b + mulmod(w, ct[((int64_t)k * 2 + 1) * N + n], q, invq), q, invq);
        }
        lds[n] = acc_a;
        lds[N + n] = acc_b;
    }
    __syncthreads();
    const double *inv = inv_tables + (int64_t)limb * N;
    // the two transforms run stage by stage side by side (one barrier per stage for both)
    int lt = 0;                                            // log2 of the butterfly span t
    for (int mm = N; mm > 1; mm >>= 1) {
        const int h = mm >> 1, t = 1 << lt;
        for (int bf = threadIdx.x; bf < N; bf += kThreads) {          // N butterflies: N/2 per polynomial
            const int half = bf >= N / 2;
            const int b2 = bf - half * (N / 2);
            const int i = b2 >> lt, jj = b2 & (t - 1);
            double *s = lds + half * N;
            const int j = (i << (lt + 1)) + jj;
            const double S = inv[h + i];
            const double U = s[j], V = s[j + t];
            s[j] = reduce(U + V, q, invq);
            s[j + t] = mulmod(S, U - V, q, invq);
        }
        __syncthreads();
        ++lt;
    }
    uint64_t *o = out + ((int64_t)limb * Mp + m) * 2 * N;
    for (int n = threadIdx.x; n < 2 * N; n += kThreads) {
        double r = reduce(lds[n], q, invq);                          // |r| <= q/2 + 1 (1/N is folded into the plaintexts)
        r = r < 0.0 ? r + q : r;                                      // canonical: an integer in [0, q)
        o[n] = (uint64_t)__double_as_longlong(r + 4503599627370496.0) & 0x000FFFFFFFFFFFFFull;
    }
}


// ---- N = 4096 (the paper's PCMv ring degree): the inverse transform as three passes of four stages each,
// sixteen elements per thread in registers, two trips through LDS instead of twelve.
//
// NTT-domain polynomials are stored so that thread T reads its entries n = 16 T + e, e < 16, with 16-byte loads of
// consecutive threads: as doubles, entry n at word N/8 (e >> 1) + 2 T + (e & 1); the plaintexts of primes below 2^36
// packed (PtRaw below).
//   pass 1  stages t = 1, 2, 4, 8        thread T holds n = 16 T + e
//   pass 2  stages t = 16 .. 128         thread T = 16 A + B holds n = 256 A + B + 16 e
//   pass 3  stages t = 256 .. 2048       thread T holds n = T + 256 e
// Stage t pairs n with n + t and uses the twiddle inv[N/(2t) + (n >> (log2 t + 1))]: 8, 4, 2 and 1 distinct
// twiddles per thread in the four stages of a pass, contiguous in the table.
// LDS holds entry n at n + (n >> 4) (one word of padding per sixteen): the 16-word strides of pass 1's writes
// and the unit strides of the other accesses are then all free of bank conflicts for 8-byte accesses.
// Ring degrees 2048 and 1024 run the same way on 128 and 64 threads: passes 1 and 2 as they are, pass 3 with the three or two
// stages that are left, on two or four columns a thread
// (radix-2 kernels through LDS -> these: degree 2048, 8192 outputs of one ciphertext, two 36-bit limbs 578 -> 164 us; 4096 of four
// ciphertexts 484 -> 162; degree 1024, 8192 outputs, four limbs 413 -> 156; 4096 of four ciphertexts, two limbs 171 -> 75).
constexpr int kMinBlocked = 1024, kMaxBlocked = 4096;   // ring degrees of these kernels
template <int N>
struct Blocked {
    static constexpr int kT = N / 16;                // threads: sixteen values each
    static constexpr int kV = N / 256;               // values of a column of pass 3
    static constexpr int kLast = N == 4096 ? 4 : N == 2048 ? 3 : 2;   // stages of pass 3
    static constexpr int kLds = N + N / 16;          // words of one polynomial
    static constexpr uint32_t kQueues = N == 4096 ? 1 : 8;   // work queues of the multiply-accumulate kernel
    // entry i (= kV r + e) of thread T in pass 3: its index is n = T + at(i), its word in LDS T + (T >> 4) + word(i)
    static __host__ __device__ constexpr int at(int i) { return kT * (i / kV) + 256 * (i % kV); }
    static __host__ __device__ constexpr int word(int i) { return (kT + kT / 16) * (i / kV) + 272 * (i % kV); }
};

// four Gentleman-Sande stages on sixteen values; tw[0..7], tw[8..11], tw[12..13], tw[14]: the twiddles of the
// four stages (stage s pairs e with e + 2^s and uses twiddle number e >> (s + 1) of its run).
// Magnitudes, LAZY = false (q < 2^50): inputs <= q.  Stages 0 and 2 leave their sums unreduced (<= 2 q; differences
// <= 2 q give products <= 0.75 q + 1), stages 1 and 3 reduce the sums (<= 4 q < 2^52 in, <= q/2 + 1 out) and
// multiply differences <= 4 q (products <= q): outputs <= q again.
// LAZY = true (q < 2^36): no sum is reduced anywhere in the twelve stages of the transform (bounds in the comment of mulmod).
// STAGES < 4 (pass 3 of smaller degrees): the values are 16 >> STAGES independent columns, the twiddles those of the last
// STAGES runs.
template <bool LAZY, int STAGES = 4>
__device__ __forceinline__ void gs16(double (&v)[16], const double (&tw)[15], double q, double invq)
{
#pragma unroll
    for (int s = 0; s < STAGES; ++s) {
        const int half = 1 << s;
        const int run = s + 4 - STAGES;
        const int off = run == 0 ? 0 : (run == 1 ? 8 : (run == 2 ? 12 : 14));
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            if (e & half) continue;
            const double U = v[e], V = v[e + half];
            v[e] = (!LAZY && (s & 1)) ? reduce(U + V, q, invq) : U + V;
            v[e + half] = mulmod(tw[off + ((e & ((1 << STAGES) - 1)) >> (s + 1))], U - V, q, invq);
        }
    }
}

typedef unsigned int v2u __attribute__((ext_vector_type(2)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef double v2d __attribute__((ext_vector_type(2)));

// a range-checked view of n_bytes of device memory (reads outside it return 0)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t view(const void *base, uint32_t n_bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, n_bytes, 0x00020000);
}
// one double / two doubles at byte offset lane_off + uniform_off
__device__ __forceinline__ double ld1(__amdgpu_buffer_rsrc_t r, uint32_t lane_off, uint32_t uniform_off)
{
    return __builtin_bit_cast(double, (v2u)__builtin_amdgcn_raw_buffer_load_b64(r, lane_off, uniform_off, 0));
}
__device__ __forceinline__ v2d ld2(__amdgpu_buffer_rsrc_t r, uint32_t lane_off, uint32_t uniform_off)
{
    return __builtin_bit_cast(v2d, (v4u)__builtin_amdgcn_raw_buffer_load_b128(r, lane_off, uniform_off, 0));
}
// The sixteen NTT-domain values of a thread as they lie in memory.
// PACKED (primes below 2^36): a balanced residue r, |r| <= q/2 + 1 < 2^35, is kept as u = r + 2^35 < 2^36: the low 32 bits
// of entry e at byte N (e >> 2) + 16 T + 4 (e & 3), the top four bits of the sixteen entries as eight bytes at
// 4 N + 8 T, entry e in bits 4 e .. 4 e + 3.  At degree 4096 18 KiB a polynomial instead of the 32 KiB of doubles: the plaintexts are most
// of what the multiply-accumulate kernel reads, and it is bound by memory as much as by its arithmetic.  Unpacking
// places u in the low mantissa bits of 2^52 and subtracts: one v_perm and one addition a value, and the masks.
// Measured, doubles -> packed (4096 output polynomials, two 36-bit limbs): one input ciphertext 182 -> 175 us, four
// 416 -> 328 us (there also because every operand of a term is now requested one term ahead).
template <bool PACKED, int N>
struct PtRaw;
template <int N>
struct PtRaw<true, N> {
    static constexpr uint32_t kBytes = N * 4 + N / 2;   // of one polynomial
    static constexpr uint32_t kRow = N;                 // bytes of four entries of every thread (16 bytes each)
    v4u lo[4];
    v2u hi;
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t T, uint32_t uniform_off)
    {
#pragma unroll
        for (int c = 0; c < 4; ++c) lo[c] = (v4u)__builtin_amdgcn_raw_buffer_load_b128(r, 16u * T + kRow * c, uniform_off, 0);
        hi = (v2u)__builtin_amdgcn_raw_buffer_load_b64(r, 8u * T + 4 * kRow, uniform_off, 0);
    }
    __device__ __forceinline__ void unpack(double (&w)[16]) const
    {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t nib[2] = {hi[h] & 0x0F0F0F0Fu, (hi[h] >> 4) & 0x0F0F0F0Fu};   // even and odd entries, a byte each
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int e = 8 * h + i;
                const uint32_t top = __builtin_amdgcn_perm(0x43300000u, nib[i & 1], 0x07060500u | (uint32_t)(i >> 1));
                w[e] = __builtin_bit_cast(double, (v2u){lo[e >> 2][e & 3], top}) - (4503599627370496.0 + 34359738368.0);
            }
        }
    }
    // r[16] -> memory
    static __device__ __forceinline__ void store(const double (&r)[16], char *poly, uint32_t T)
    {
        v2u h = {0, 0};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            v4u l;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int e = 4 * c + i;
                const v2u u = __builtin_bit_cast(v2u, r[e] + (4503599627370496.0 + 34359738368.0));
                l[i] = u[0];
                h[e >> 3] |= (u[1] & 0xFu) << (4 * (e & 7));
            }
            *reinterpret_cast<v4u *>(poly + 16u * T + kRow * c) = l;
        }
        *reinterpret_cast<v2u *>(poly + 8u * T + 4 * kRow) = h;
    }
};
template <int N>
struct PtRaw<false, N> {
    static constexpr uint32_t kBytes = N * 8;
    static constexpr uint32_t kRow = N;                 // bytes of two entries of every thread (16 bytes each)
    v2d x[8];
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t T, uint32_t uniform_off)
    {
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = ld2(r, 16u * T + kRow * i, uniform_off);
    }
    __device__ __forceinline__ void unpack(double (&w)[16]) const
    {
#pragma unroll
        for (int e = 0; e < 16; ++e) w[e] = x[e >> 1][e & 1];
    }
    static __device__ __forceinline__ void store(const double (&r)[16], char *poly, uint32_t T)
    {
#pragma unroll
        for (int i = 0; i < 8; ++i) *reinterpret_cast<v2d *>(poly + 16u * T + kRow * i) = (v2d){r[2 * i], r[2 * i + 1]};
    }
};

// the fifteen twiddles of four stages: eight consecutive table entries from 8 (base + i0), four from 4 (base + i0),
// two from 2 (base + i0), one at base + i0
__device__ __forceinline__ void load_tw(double (&tw)[15], __amdgpu_buffer_rsrc_t irs, uint32_t base, uint32_t i0)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const v2d t = ld2(irs, (8 * base + 8 * i0) * 8u, 16u * i);
        tw[2 * i] = t[0];
        tw[2 * i + 1] = t[1];
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const v2d t = ld2(irs, (4 * base + 4 * i0) * 8u, 16u * i);
        tw[8 + 2 * i] = t[0];
        tw[9 + 2 * i] = t[1];
    }
    const v2d t = ld2(irs, (2 * base + 2 * i0) * 8u, 0);
    tw[12] = t[0];
    tw[13] = t[1];
    tw[14] = ld1(irs, (base + i0) * 8u, 0);
}

// four Cooley-Tukey stages on sixteen values (stage s pairs e with e + (8 >> s); its 2^s twiddles are the run of
// that length in tw, in the layout load_tw produces: tw[14], tw[12..13], tw[8..11], tw[0..7]).
// Magnitudes, LAZY = false: inputs <= 1.5 q + 1.  Stages 0 and 2 add a product (<= 0.75 q + 1, its operand being
// <= 2 q) to an unreduced value: <= 2.25 q + 2; stages 1 and 3 reduce that value first (<= q/2 + 1) and multiply
// operands <= 2.25 q + 2 <= 4 q (products <= q): outputs <= 1.5 q + 1 again.
// LAZY = true (q < 2^36): nothing is reduced; a value grows by at most 0.5625 q per stage, to less than 8 q in twelve.
// STAGES < 4 (pass A of smaller degrees): 16 >> STAGES independent columns.  Three stages end without a reduction: outputs
// <= 2.25 q + 2, so that the next pass's first stage leaves <= 3.25 q + 3 <= 4 q and its second reduces as above.
template <bool LAZY, int STAGES = 4>
__device__ __forceinline__ void ct16(double (&v)[16], const double (&tw)[15], double q, double invq)
{
#pragma unroll
    for (int s = 0; s < STAGES; ++s) {
        const int half = (1 << STAGES) >> (s + 1);
        const int off = s == 0 ? 14 : (s == 1 ? 12 : (s == 2 ? 8 : 0));
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            if (e & half) continue;
            const double U = (!LAZY && (s & 1)) ? reduce(v[e], q, invq) : v[e];
            const double V = mulmod(tw[off + ((e & ((1 << STAGES) - 1)) >> (STAGES - s))], v[e + half], q, invq);
            v[e] = U + V;
            v[e + half] = U - V;
        }
    }
}

// Forward negacyclic NTT of polynomials, one per work-group: the mirror image of the inverse
// transform below -- three passes of four Cooley-Tukey stages on sixteen values per thread, two trips through LDS.
//   pass A  stages t = 2048 .. 256       thread T holds n = T + 256 e     (read from memory, coalesced)
//   pass B  stages t = 128 .. 16         thread T = 16 A + B holds n = 256 A + B + 16 e
//   pass C  stages t = 8 .. 1            thread T holds n = 16 T + e      (entries of the bit-reversed order, stored in
//                                        the layout the multiply-accumulate reads: PtRaw)
// Stage t = N/(2m) uses the twiddle fwd[m + (n >> (log2 t + 1))].  Sources and the scaling of the plaintexts as in ntt_kernel.
template <int N, int SRC, bool LAZY>
__global__ __launch_bounds__(N / 16) void ntt_blocked_kernel(const void *__restrict__ src, void *__restrict__ dst,
                                                           const double *__restrict__ fwd_tables, const LimbDev *__restrict__ lc,
                                                           int64_t polys_per_limb, uint32_t *__restrict__ queue, uint32_t queue_start)
{
    using G = Blocked<N>;
    __shared__ double lds[G::kLds];
    const int64_t p = blockIdx.x;
    if (queue && p == 0 && threadIdx.x < G::kQueues)                     // the work queues of the kernel that follows
        queue[threadIdx.x * kQueueStride] = queue_start;
    const int limb = (int)(p / polys_per_limb);
    const int64_t within = p % polys_per_limb;
    const double q = lc[limb].q, invq = lc[limb].invq;
    const __amdgpu_buffer_rsrc_t frs = view(fwd_tables + (int64_t)limb * N, N * 8);
    const int T = threadIdx.x, A = T >> 4, B = T & 15;
    double v[16], tw[15];
    load_tw(tw, frs, 1, 0);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        if (SRC == 0) {
            const uint64_t x = static_cast<const uint64_t *>(src)[p * N + T + G::at(e)];
            v[e] = __builtin_fma((double)(uint32_t)(x >> 32), 4294967296.0, (double)(uint32_t)x);   // exact: x < 2^50
        } else {
            v[e] = (double)static_cast<const int32_t *>(src)[within * N + T + G::at(e)];
        }
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) v[e] = reduce(v[e], q, invq);
    ct16<LAZY, G::kLast>(v, tw, q, invq);
#pragma unroll
    for (int e = 0; e < 16; ++e) lds[T + (T >> 4) + G::word(e)] = v[e];
    load_tw(tw, frs, N / 256, A);
    __syncthreads();
    {
        double *s = lds + 272 * A + B;
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = s[17 * e];
        ct16<LAZY>(v, tw, q, invq);
#pragma unroll
        for (int e = 0; e < 16; ++e) s[17 * e] = v[e];
    }
    load_tw(tw, frs, N / 16, T);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 16; ++e) v[e] = lds[17 * T + e];
    ct16<LAZY>(v, tw, q, invq);
    // the plaintexts carry the factor 1/N of the inverse transform that follows the pointwise products
    const double scale = lc[limb].n_inv;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        v[e] = reduce(v[e], q, invq);
        if (SRC == 1) v[e] = reduce(mulmod(scale, v[e], q, invq), q, invq);
    }
    using Raw = PtRaw<SRC == 1 && LAZY, N>;               // plaintexts packed where the prime allows it, ciphertexts as doubles
    Raw::store(v, static_cast<char *>(dst) + p * (int64_t)Raw::kBytes, T);
}

// Persistent work-groups (eight waves per compute unit), so that what depends only on the limb stays in registers from one
// polynomial to the next -- the twiddles of passes 1 and 2 and, for KP1 (one input ciphertext, the shape of every decode projection
// whose input fits one polynomial), the thread's 32 values of the transformed ciphertext -- and the plaintext values of the
// next polynomial are requested while the present one is transformed.  total = L Mp polynomials: the first two of a work-group
// are fixed, the rest come from a queue in order of asking; the loop ends for every wave when its index passes the last.
// Degrees 2048 and 1024 have a queue for each XCD (work-group b runs on XCD b % 8) with an eighth of the polynomials: one counter hands
// out a polynomial every 12 ns at most, and the 8192 of degree 1024 (4096 outputs, two 50-bit limbs) took 114 us with one queue, 55
// with eight.  Degree 4096 needs a polynomial every 20 ns and keeps one: with eight it is no faster.
//
// LAZY (every prime below 2^36): no intermediate reduction of sums, neither in the transform nor between the
// terms of the multiply-accumulate (Kp <= 4096 products of magnitude <= 0.5625 q: below 2^12 q; one reduction
// after the last term).
//
// All global reads are buffer loads (uniform base and offset in scalar registers, one 32-bit lane offset): no vector
// registers go into addresses, and the loads of a term are all issued before the first is used (left to itself the
// compiler starts the arithmetic on the first values early, which splits the loads into two dependent round trips).
template <int N, bool LAZY, bool KP1>
__global__ __launch_bounds__(N / 16, 2) void mac_intt_blocked_kernel(const void *__restrict__ ptn, const double *__restrict__ ctn,
                                                                   uint64_t *__restrict__ out, const double *__restrict__ inv_tables,
                                                                   const LimbDev *__restrict__ lc, uint32_t Mp, int Kp, uint32_t total,
                                                                   uint32_t *__restrict__ queue)
{
    using G = Blocked<N>;
    constexpr uint32_t PB = N * 8;                    // bytes of one polynomial of doubles
    __shared__ double lds[2 * G::kLds];          // component a, component b
    __shared__ uint32_t queue_word;
    const int T = threadIdx.x;
    using Raw = PtRaw<LAZY, N>;
    constexpr uint32_t Q = G::kQueues;
    const uint32_t own = blockIdx.x % Q, per_queue = (total + Q - 1) / Q, lo = own * per_queue;
    const uint32_t hi = min(lo + per_queue, total);   // this queue's polynomials (none where lo >= hi); total + 3 grid + 8 < 2^32
    uint32_t blk = lo + blockIdx.x / Q;
    if (blk >= hi) return;
    uint32_t next = blk + gridDim.x / Q;              // the first two polynomials of a work-group are fixed
    const uint32_t kpb = (uint32_t)Kp * Raw::kBytes;  // bytes of the plaintexts of one output polynomial (Kp <= 4096)
    auto plaintexts = [&](uint32_t poly) { return view(static_cast<const char *>(ptn) + (int64_t)poly * kpb, kpb); };

    double tw1[15], tw2[15];
    PtRaw<false, N> xa, xb;                              // transformed ciphertext values
    Raw wv;                                           // plaintext values, requested one term ahead
    double q = 0.0, invq = 0.0;
    uint32_t limb_loaded = 0xFFFFFFFFu;
    wv.load(plaintexts(blk), T, 0);
    for (;;) {
        const uint32_t limb = blk / Mp;
        // the polynomial after the next one comes from the queue (one lane asks; the answer is passed on through LDS
        // behind the first barrier below)
        uint32_t asked = 0;
        if (T == 0) asked = lo + atomicAdd(&queue[own * kQueueStride], 1u);
        // the LDS addresses below are recomputed from the thread index in every round (the asm hides that it is the same
        // index): kept across the loop they cost more registers than the kernel has
        int Ti = T;
        asm volatile("" : "+v"(Ti));
        const int Ai = Ti >> 4, Bi = Ti & 15;
        const __amdgpu_buffer_rsrc_t crs = view(ctn + (int64_t)limb * Kp * 2 * N, (uint32_t)Kp * 2 * PB);
        const __amdgpu_buffer_rsrc_t irs = view(inv_tables + (int64_t)limb * N, PB);
        if (limb != limb_loaded) {                    // uniform: first polynomial of a limb for this work-group
            limb_loaded = limb;
            q = lc[limb].q;
            invq = lc[limb].invq;
            if constexpr (KP1) {
                load_tw(tw1, irs, N / 16, T);         // pass 1: table entries N/2 + 8 T .., N/4 + 4 T .., N/8 + 2 T .., N/16 + T
                load_tw(tw2, irs, N / 256, T >> 4);   // pass 2, A = T / 16: N/32 + 8 A .., N/64 + 4 A .., N/128 + 2 A .., N/256 + A
                xa.load(crs, T, 0);
                xb.load(crs, T, PB);
            }
        }

        // ---- pass 1: pointwise multiply-accumulate of both components straight into registers (each plaintext
        // value is loaded once and used for a and b), then stages t = 1 .. 8
        double va[16], vb[16];
        if constexpr (KP1) {
            __builtin_amdgcn_sched_barrier(0);
            double w[16];
            wv.unpack(w);
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                va[e] = mulmod(w[e], xa.x[e >> 1][e & 1], q, invq);
                vb[e] = mulmod(w[e], xb.x[e >> 1][e & 1], q, invq);
            }
        } else {
            const __amdgpu_buffer_rsrc_t prs = plaintexts(blk);
            xa.load(crs, T, 0);
            xb.load(crs, T, PB);
#pragma unroll
            for (int e = 0; e < 16; ++e) va[e] = vb[e] = 0.0;
            // One term.  Each set of operands is requested for the next term as soon as the present one has used it: the
            // plaintexts once unpacked, component a's values behind the products of a, component b's behind those of b.
            auto products = [&](double (&v)[16], const double (&w)[16], const PtRaw<false, N> &x) {
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const double y = mulmod(w[e], x.x[e >> 1][e & 1], q, invq);
                    v[e] = LAZY ? v[e] + y : reduce(v[e] + y, q, invq);
                }
            };
            auto term = [&](int k, auto last_c) {
                constexpr bool LAST = decltype(last_c)::value;
                double w[16];
                wv.unpack(w);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (!LAST) wv.load(prs, T, (uint32_t)(k + 1) * Raw::kBytes);
                products(va, w, xa);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (!LAST) xa.load(crs, T, (uint32_t)(k + 1) * 2 * PB);
                products(vb, w, xb);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (!LAST) xb.load(crs, T, (uint32_t)(k + 1) * 2 * PB + PB);
            };
            for (int k = 0; k < Kp - 1; ++k) term(k, std::false_type{});
            term(Kp - 1, std::true_type{});
        }
        // The products are complete here: the empty asm uses them and orders memory accesses, so that the compiler can
        // neither sink the arithmetic below the loads that follow nor lift those loads above it (either way the registers
        // would have to hold the operands of both).
#pragma unroll
        for (int e = 0; e < 16; e += 4)
            asm volatile("" ::"v"(va[e]), "v"(va[e + 1]), "v"(va[e + 2]), "v"(va[e + 3]), "v"(vb[e]), "v"(vb[e + 1]), "v"(vb[e + 2]),
                         "v"(vb[e + 3])
                         : "memory");
        // the first plaintext values of the next polynomial are requested now and used in the next round
        if (next < hi) wv.load(plaintexts(next), T, 0);
        if constexpr (!KP1) {
            // with several terms the registers do not hold the twiddles from one polynomial to the next
            load_tw(tw1, irs, N / 16, Ti);
            load_tw(tw2, irs, N / 256, Ai);
            if constexpr (LAZY) {
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    va[e] = reduce(va[e], q, invq);
                    vb[e] = reduce(vb[e], q, invq);
                }
            }
        }
        gs16<LAZY>(va, tw1, q, invq);
        if (T == 0) queue_word = asked;
        __syncthreads();                                               // every wave has read the previous polynomial from LDS
        const uint32_t after_next = __builtin_amdgcn_readfirstlane(queue_word);
#pragma unroll
        for (int e = 0; e < 16; ++e) lds[17 * Ti + e] = va[e];          // n = 16 T + e at n + (n >> 4)
        gs16<LAZY>(vb, tw1, q, invq);
#pragma unroll
        for (int e = 0; e < 16; ++e) lds[G::kLds + 17 * Ti + e] = vb[e];
        __syncthreads();

        // ---- pass 2: stages t = 16 .. 128 on n = 256 A + B + 16 e, i.e. LDS word 272 A + B + 17 e
        for (int c = 0; c < 2; ++c) {
            double *s = lds + c * G::kLds + 272 * Ai + Bi;
            double v[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) v[e] = s[17 * e];
            gs16<LAZY>(v, tw2, q, invq);
#pragma unroll
            for (int e = 0; e < 16; ++e) s[17 * e] = v[e];
        }
        __syncthreads();

        // ---- pass 3: stages t = 256 .. N / 2 on n = T + 256 e (and further columns of smaller degrees); then out
        // (the fifteen twiddles are the same for every thread: table entries 1 .. 15)
        const double *inv = inv_tables + (int64_t)limb * N;
        double tw3[15];
#pragma unroll
        for (int i = 0; i < 8; ++i) tw3[i] = inv[8 + i];
#pragma unroll
        for (int i = 0; i < 4; ++i) tw3[8 + i] = inv[4 + i];
        tw3[12] = inv[2];
        tw3[13] = inv[3];
        tw3[14] = inv[1];
        const double half_invq = 0.5 * invq;
        uint64_t *o = out + (int64_t)blk * 2 * N;
        for (int c = 0; c < 2; ++c) {
            const double *s = lds + c * G::kLds + Ti + (Ti >> 4);
            double v[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) v[e] = s[G::word(e)];
            gs16<LAZY, G::kLast>(v, tw3, q, invq);
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                double r;                                              // canonical: an integer in [0, q) (1/N is folded into the plaintexts)
                if constexpr (LAZY) {
                    r = canonical(v[e], q, invq, half_invq);          // |v| < 2^12 q, q < 2^36
                } else {
                    r = reduce(v[e], q, invq);                        // |r| <= q/2 + 1
                    r = r < 0.0 ? r + q : r;
                }
                // non-temporal: written once and not read here, so that the caches keep what is read (177 -> 174 us for
                // 4096 outputs of one ciphertext and two limbs, 329 -> 323 us for four; the same hint on the plaintext
                // loads costs 2 % where they fit the last-level cache)
                __builtin_nontemporal_store((uint64_t)__double_as_longlong(r + 4503599627370496.0) & 0x000FFFFFFFFFFFFFull,
                                            &o[c * N + Ti + G::at(e)]);
            }
        }
        if (next >= hi) break;
        blk = next;
        next = after_next;
    }
}

bool blocked(int64_t N) { return N >= kMinBlocked && N <= kMaxBlocked; }

// f(integral_constant<int, N>) for a ring degree of the blocked kernels
template <class F>
void with_degree(int N, F &&f)
{
    if (N == 4096) f(std::integral_constant<int, 4096>{});
    else if (N == 2048) f(std::integral_constant<int, 2048>{});
    else f(std::integral_constant<int, 1024>{});
}

}  // namespace

struct pcmv_plan {
    int64_t Mp, Kp, N;
    int L, device;
    uint32_t grid;     // work-groups of the persistent kernel: eight waves per compute unit
    uint32_t *queue;   // device: its work queues' counters
    bool lazy;         // every prime is below 2^36: the blocked transforms run without intermediate reductions
    void *ptn;         // device [L][Mp][Kp]: plaintexts in the NTT domain (N doubles, or PtRaw<true> for blocked degrees and lazy)
    double *ctn;       // device [L][Kp][2][N]: scratch, the ciphertexts of one run in the NTT domain
    double *fwd, *inv; // device [L][N] twiddle tables
    LimbDev *lc;       // device [L]
    size_t bytes;
};

extern "C" {

pcmm_status pcmv_plan_create(pcmv_plan **out, int64_t Mp, int64_t Kp, int64_t N, int32_t L, const uint64_t *primes_host,
                             int32_t prime_bits, const int32_t *pt_dev, int32_t device, void *stream)
{
    if (!out) return PCMM_EINVAL;
    *out = nullptr;
    if (!pt_dev) return PCMM_EINVAL;
    const pcmm_status arc = pcmv_host::check_args(Mp, Kp, N, L, primes_host, prime_bits, device);
    if (arc != PCMM_OK) return arc;

    std::vector<double> fwd, inv;
    std::vector<LimbDev> lc((size_t)L);
    try {
        fwd.resize((size_t)L * N);
        inv.resize((size_t)L * N);
        for (int j = 0; j < L; ++j) {
            pcmv_host::LimbTables t;
            const pcmm_status trc = pcmv_host::limb_tables(primes_host[j], N, &t);
            if (trc != PCMM_OK) return trc;          // no primitive 2N-th root: not a prime of the form 1 mod 2N
            for (int64_t i = 0; i < N; ++i) {
                fwd[(size_t)j * N + i] = t.fwd[(size_t)i];
                inv[(size_t)j * N + i] = t.inv[(size_t)i];
            }
            lc[(size_t)j].q = t.qd;
            lc[(size_t)j].invq = t.invq;
            lc[(size_t)j].n_inv = t.n_inv;
            lc[(size_t)j].pad = 0.0;
        }
    } catch (const std::bad_alloc &) {
        return PCMM_ENOMEM;
    }

    pcmv_plan *p = new (std::nothrow) pcmv_plan();
    if (!p) return PCMM_ENOMEM;
    p->Mp = Mp; p->Kp = Kp; p->N = N; p->L = L; p->device = device;
    p->lazy = prime_bits <= 36;      // check_args: every prime has exactly prime_bits bits
    p->ptn = nullptr; p->ctn = nullptr; p->fwd = nullptr; p->inv = nullptr; p->lc = nullptr; p->queue = nullptr;
    p->grid = 0;
    pcmm_hip_util::DevGuard dg(device);
    if (!dg.ok) { delete p; return PCMM_EDEVICE; }
    hipStream_t st = (hipStream_t)stream;
    // 8 bytes a value, the documented size of a plan, whether the values are packed or not (PtRaw<true> uses 4.5)
    const size_t ptn_bytes = (size_t)L * Mp * Kp * N * sizeof(double);
    const size_t ctn_bytes = (size_t)L * Kp * 2 * N * sizeof(double);
    const size_t tab_bytes = (size_t)L * N * sizeof(double);
    const size_t lc_bytes = (size_t)L * sizeof(LimbDev);
    const size_t queue_bytes = kXcd * kQueueStride * sizeof(uint32_t);
    pcmm_status rc = PCMM_OK;
    if (hipMalloc((void **)&p->ptn, ptn_bytes) != hipSuccess || hipMalloc((void **)&p->ctn, ctn_bytes) != hipSuccess ||
        hipMalloc((void **)&p->fwd, tab_bytes) != hipSuccess || hipMalloc((void **)&p->inv, tab_bytes) != hipSuccess ||
        hipMalloc((void **)&p->lc, lc_bytes) != hipSuccess || hipMalloc((void **)&p->queue, queue_bytes) != hipSuccess) {
        (void)hipGetLastError();
        rc = PCMM_ENOMEM;
    }
    p->bytes = ptn_bytes + ctn_bytes + 2 * tab_bytes + lc_bytes + queue_bytes;
    if (rc == PCMM_OK) {
        // the persistent kernel runs two waves per SIMD: two work-groups of four waves per compute unit at degree 4096
        int cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || cus <= 0) rc = PCMM_EDEVICE;
        const int64_t total = (int64_t)L * Mp;
        const int64_t most = 2 * (int64_t)cus * (kMaxBlocked / N);
        p->grid = (uint32_t)((total < most ? total : most) + kXcd - 1) / kXcd * kXcd;   // whole rounds over the XCDs
    }
    if (rc == PCMM_OK) {
        if (hipMemcpyAsync(p->fwd, fwd.data(), tab_bytes, hipMemcpyHostToDevice, st) != hipSuccess ||
            hipMemcpyAsync(p->inv, inv.data(), tab_bytes, hipMemcpyHostToDevice, st) != hipSuccess ||
            hipMemcpyAsync(p->lc, lc.data(), lc_bytes, hipMemcpyHostToDevice, st) != hipSuccess)
            rc = PCMM_EDEVICE;
    }
    if (rc == PCMM_OK) {
        // the plaintexts into the NTT domain, once (the paper's model conversion for PCMv, Section 5.3)
        const int64_t polys = (int64_t)L * Mp * Kp;
        if (blocked(N))
            with_degree((int)N, [&](auto n) {
                constexpr int NN = decltype(n)::value;
                hipLaunchKernelGGL((p->lazy ? ntt_blocked_kernel<NN, 1, true> : ntt_blocked_kernel<NN, 1, false>), dim3((unsigned)polys),
                                   dim3(NN / 16), 0, st, (const void *)pt_dev, p->ptn, p->fwd, p->lc, Mp * Kp, (uint32_t *)nullptr, 0u);
            });
        else
            hipLaunchKernelGGL((ntt_kernel<1>), dim3((unsigned)polys), dim3(kThreads), (size_t)N * sizeof(double), st,
                               (const void *)pt_dev, (double *)p->ptn, p->fwd, p->lc, (int)N, Mp * Kp);
        if (hipGetLastError() != hipSuccess) rc = PCMM_EDEVICE;
    }
    if (hipStreamSynchronize(st) != hipSuccess) rc = rc == PCMM_OK ? PCMM_EDEVICE : rc;   // the host tables live on this frame
    if (rc != PCMM_OK) {
        pcmv_plan_destroy(p);
        return rc;
    }
    *out = p;
    return PCMM_OK;
}

size_t pcmv_plan_workspace_bytes(const pcmv_plan *plan) { return plan ? plan->bytes : 0; }

pcmm_status pcmv_run(const pcmv_plan *plan, const uint64_t *ct_dev, uint64_t *out_dev, void *stream)
{
    if (!plan || !ct_dev || !out_dev) return PCMM_EINVAL;
    pcmm_hip_util::DevGuard dg(plan->device);
    if (!dg.ok) return PCMM_EDEVICE;
    hipStream_t st = (hipStream_t)stream;
    const int N = (int)plan->N;
    const int64_t ct_polys = (int64_t)plan->L * plan->Kp * 2;
    if (blocked(N)) {
        hipError_t rc = hipSuccess;
        with_degree(N, [&](auto n) {
            constexpr int NN = decltype(n)::value;
            hipLaunchKernelGGL((plan->lazy ? ntt_blocked_kernel<NN, 0, true> : ntt_blocked_kernel<NN, 0, false>), dim3((unsigned)ct_polys),
                               dim3(NN / 16), 0, st, (const void *)ct_dev, plan->ctn, plan->fwd, plan->lc, plan->Kp * 2, plan->queue,
                               2u * plan->grid / Blocked<NN>::kQueues);
            rc = hipGetLastError();
            if (rc != hipSuccess) return;
            auto kern = plan->Kp == 1 ? (plan->lazy ? mac_intt_blocked_kernel<NN, true, true> : mac_intt_blocked_kernel<NN, false, true>)
                                      : (plan->lazy ? mac_intt_blocked_kernel<NN, true, false> : mac_intt_blocked_kernel<NN, false, false>);
            hipLaunchKernelGGL(kern, dim3(plan->grid), dim3(NN / 16), 0, st, plan->ptn, plan->ctn, out_dev, plan->inv, plan->lc,
                               (uint32_t)plan->Mp, (int)plan->Kp, (uint32_t)(plan->L * plan->Mp), plan->queue);
        });
        if (rc != hipSuccess) return PCMM_EDEVICE;
    } else {
        hipLaunchKernelGGL((ntt_kernel<0>), dim3((unsigned)ct_polys), dim3(kThreads), (size_t)N * sizeof(double), st,
                           (const void *)ct_dev, plan->ctn, plan->fwd, plan->lc, N, plan->Kp * 2);
        if (hipGetLastError() != hipSuccess) return PCMM_EDEVICE;
        hipLaunchKernelGGL(mac_intt_kernel, dim3((unsigned)((int64_t)plan->L * plan->Mp)), dim3(kThreads),
                           (size_t)2 * N * sizeof(double), st, (const double *)plan->ptn, plan->ctn, out_dev, plan->inv, plan->lc, N, plan->Mp,
                           (int)plan->Kp);
    }
    return hipGetLastError() == hipSuccess ? PCMM_OK : PCMM_EDEVICE;
}

void pcmv_plan_destroy(pcmv_plan *plan)
{
    if (!plan) return;
    pcmm_hip_util::DevGuard dg(plan->device);
    if (plan->ptn) (void)hipFree(plan->ptn);
    if (plan->ctn) (void)hipFree(plan->ctn);
    if (plan->fwd) (void)hipFree(plan->fwd);
    if (plan->inv) (void)hipFree(plan->inv);
    if (plan->lc) (void)hipFree(plan->lc);
    if (plan->queue) (void)hipFree(plan->queue);
    delete plan;
}

}  // extern "C"
