// PCMM for MI355X (gfx950): C_j = W . A_j mod q_j, batched over RNS limbs and both ciphertext
// components (the clear matrix product that the paper's linear-layer PCMM reduces to, Sections 2.2,
// 3.2 and 5.1; ciphertexts as pairs in R_Q^2 with component-wise addition, Appendix A).
//
// Kernels of the PCMM path:
//   pack_w_kernel   (plan time)  W -> int8 slices in MFMA A-operand fragment order
//   split_kernel    (every run)  uint64 residues -> D signed base-256 digit planes in MFMA
//                                B-operand fragment order (split_pair_kernel: two limbs joined into one
//                                integer of nine digits)
//   gemm_kernel     (every run)  v_mfma_i32_16x16x64_i8 main loop, then recombination of the digit
//                                accumulators and reduction modulo q_j
//   (contractions of at most 128 values of k run as one kernel, pcmm_shortk.hip, and so do those whose digits fit LDS,
//   pcmm_resident.hip)
// Beside it:
//   transpose_u64_kernel         the coefficient permutation of ring switching (Section 3.3)
//   mfma_probe_kernel            measurement aid: what the matrix cores sustain without memory traffic
//
// Fragment order.  One v_mfma_i32_16x16x64_i8 operand is 16 (rows or columns) x 64 (k) int8: lane l
// of the wave holds the 16 bytes with index (l % 16) and k = 16*(l/16) .. 16*(l/16)+15.  Both
// operands use the same k mapping, so an integer dot product does not depend on the order of k
// inside a lane.  A "fragment" is the 1 KiB such an operand takes, stored [lane][16 bytes], so that
// a wave fetches it with one 16-byte load per lane from contiguous memory.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <algorithm>
#include <mutex>
#include <new>
#include <type_traits>
#include <utility>
#include "../../include/pcmm.h"
#include "pcmm_host.hpp"
#include "pcmm_device.hpp"
#include "pcmm_resident.hpp"
#include "pcmm_shortk.hpp"
#include "pcmm_hip_util.hpp"

using namespace pcmm_device;

namespace {

// The MFMA accumulators live in fixed accumulation registers a[0 : 4*MT*NT*E) that only the asm
// statements below name; the compiler never sees them as values, so it can neither migrate them
// between register files nor copy them at a point where the hardware would return a stale value.
// (An MFMA result may not be read by a non-MFMA instruction for up to 18 cycles after issue, and the
// hardware does not interlock; mfma_drain() provides the wait.)  Compiler-generated code never
// allocates accumulation registers in these kernels: they are used only when the 256 ordinary
// registers run out, and tests/test_build_asm.py checks that none appears outside the asm.
//
// acc[BASE : BASE+4) += A x B on one 16 x 16 x 64 int8 tile
template <int BASE>
__device__ __forceinline__ void mfma_i8(const v4i &a, const v4i &b)
{
    asm volatile("v_mfma_i32_16x16x64_i8 a[%0:%1], %2, %3, a[%0:%1]" ::"n"(BASE), "n"(BASE + 3), "v"(a), "v"(b));
}
template <int IDX>
__device__ __forceinline__ void acc_zero()
{
    asm volatile("v_accvgpr_write_b32 a[%0], 0" ::"n"(IDX));
}
template <int IDX>
__device__ __forceinline__ int acc_read()
{
    int x;
    asm volatile("v_accvgpr_read_b32 %0, a[%1]" : "=v"(x) : "n"(IDX));
    return x;
}
// tells the compiler which accumulation registers the kernel uses (it sizes the register file from this)
template <int NACC>
__device__ __forceinline__ void acc_declare()
{
    static_assert(NACC == 96 || NACC == 112 || NACC == 128 || NACC == 144 || NACC == 160, "add a clobber for this count");
    if constexpr (NACC == 96) asm volatile("" ::: "a95");
    if constexpr (NACC == 112) asm volatile("" ::: "a111");
    if constexpr (NACC == 128) asm volatile("" ::: "a127");
    if constexpr (NACC == 144) asm volatile("" ::: "a143");
    if constexpr (NACC == 160) asm volatile("" ::: "a159");
}

// wait states between the last MFMA (or accumulator write) and the next different kind of access
__device__ __forceinline__ void mfma_drain()
{
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
}

// the constants of every limb pair, passed to the split kernel by value
struct PairConsts {
    pcmm_host::PairConst c[pcmm_host::kMaxLimbs / 2];
};

// ------------------------------------------------------------------------------------------------
// plan-time kernel: pack W
// ------------------------------------------------------------------------------------------------
// Output Wp[s][kb][mb][lane][16]: slice s of W[mb*16 + lane%16][kb*64 + (lane/16)*16 + 0..15],
// zero outside M x K.  int16 entries are split as w = lo + 256*hi with lo = sign-extended low byte;
// err is set to 1 if some hi does not fit int8.
template <typename WT, int S>
__global__ __launch_bounds__(256) void pack_w_kernel(const WT *__restrict__ W, int8_t *__restrict__ Wp,
                                                     int64_t M, int64_t K, int64_t MB, int64_t nkb,
                                                     int *__restrict__ err)
{
    int64_t unit = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;   // one 16-byte lane slot
    int64_t total = MB * nkb * 64;
    if (unit >= total) return;
    int lane = (int)(unit % 64);
    int64_t kb = (unit / 64) % nkb;
    int64_t mb = unit / (64 * nkb);
    int64_t m = mb * 16 + (lane % 16);
    int64_t k0 = kb * 64 + (lane / 16) * 16;
    int8_t lo[16], hi[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        int64_t k = k0 + j;
        int w = (m < M && k < K) ? (int)W[m * K + k] : 0;
        int l = (int)(int8_t)(w & 0xFF);
        int h = (w - l) >> 8;
        lo[j] = (int8_t)l;
        hi[j] = (int8_t)h;
        if (S == 2 && (h < -128 || h > 127)) atomicExch(err, 1);
    }
    int8_t *dst = Wp + ((kb * MB + mb) * 64 + lane) * 16;
#pragma unroll
    for (int j = 0; j < 16; ++j) dst[j] = lo[j];
    if (S == 2) {
        int8_t *dst2 = dst + MB * nkb * kFrag;
#pragma unroll
        for (int j = 0; j < 16; ++j) dst2[j] = hi[j];
    }
}

// ------------------------------------------------------------------------------------------------
// run-time kernel 1: digit split
// ------------------------------------------------------------------------------------------------
// Balanced base-256 digits: with Bias = sum_{i<D} 128 * 256^i, the bytes of x + Bias, each xor 0x80,
// read as int8, are digits s_i in [-128,127] with x = sum_i s_i 256^i (valid while x + Bias < 256^D).
//
// Output layout Ad[limb][kb][ntile][nt][d][lane][16]; fragment (nt, d) of chunk (limb, kb, ntile)
// holds digit d of A[limb][kb*64 + (lane/16)*16 + 0..15][(ntile*NT + nt)*16 + lane%16], zero outside
// K x Ncols.  One block = 4 waves = 64 columns x 64 k; wave g takes k-group g, lane = column.
//
// NT_ACCESS (pcmm_host::SplitNt): what streams past the caches.
template <int NT_ACCESS>
__device__ __forceinline__ uint64_t residue(const uint64_t *word)
{
    return NT_ACCESS == pcmm_host::kNtBoth ? __builtin_nontemporal_load(word) : *word;
}
template <int NT_ACCESS>
__device__ __forceinline__ void store_digits(const v4i &v, int8_t *at)
{
    if constexpr (NT_ACCESS != pcmm_host::kNtNone) __builtin_nontemporal_store(v, reinterpret_cast<v4i *>(at));
    else *reinterpret_cast<v4i *>(at) = v;
}
template <int D, int NT_ACCESS>
__global__ __launch_bounds__(256) void split_kernel(const uint64_t *__restrict__ A, int8_t *__restrict__ Ad,
                                                    int64_t K, int64_t Ncols, int64_t nkb, int64_t ntiles,
                                                    int NT)
{
    const int lane = threadIdx.x & 63;
    const int g = threadIdx.x >> 6;
    const int64_t kb = blockIdx.y;
    const int64_t limb = blockIdx.z;
    const int64_t n = (int64_t)blockIdx.x * 64 + lane;
    const int64_t nb = n >> 4;
    if (nb >= ntiles * NT) return;

    uint64_t bias = 0;
#pragma unroll
    for (int i = 0; i < D; ++i) bias |= (uint64_t)0x80 << (8 * i);

    const int64_t k0 = kb * 64 + g * 16;
    const uint64_t *src = A + (limb * K + k0) * Ncols + n;
    uint32_t out[D][4];
#pragma unroll
    for (int d = 0; d < D; ++d)
#pragma unroll
        for (int i = 0; i < 4; ++i) out[d][i] = 0;

#pragma unroll
    for (int j = 0; j < 16; ++j) {
        uint64_t x = (k0 + j < K && n < Ncols) ? residue<NT_ACCESS>(&src[(int64_t)j * Ncols]) : 0;
        uint64_t y = x + bias;
#pragma unroll
        for (int d = 0; d < D; ++d) out[d][j >> 2] |= (uint32_t)((y >> (8 * d)) & 0xFF) << (8 * (j & 3));
    }

    const int64_t ntile = nb / NT;
    const int nt = (int)(nb % NT);
    int8_t *chunk = Ad + ((limb * nkb + kb) * ntiles + ntile) * ((int64_t)NT * D * kFrag);
#pragma unroll
    for (int d = 0; d < D; ++d) {
        v4i v;
        v.x = (int)(out[d][0] ^ 0x80808080u);
        v.y = (int)(out[d][1] ^ 0x80808080u);
        v.z = (int)(out[d][2] ^ 0x80808080u);
        v.w = (int)(out[d][3] ^ 0x80808080u);
        store_digits<NT_ACCESS>(v, chunk + (nt * D + d) * kFrag + (g * 16 + (int)(n & 15)) * 16);
    }
}

// Digit split of TWO limbs at once (S = 1, five digits a limb, primes below 2^36).  One residue x_i < q_i < 2^36 takes five
// base-256 digits, so two limbs cost ten digit products although they hold only 72 bits, nine bytes.  The two
// residues are therefore joined by the Chinese remainder theorem into one integer X with X = x1 mod q1 and
// X = x2 mod q2, and X is cut into nine balanced digits; the product sum W X reduced modulo q1 and modulo q2 gives both
// outputs.  One digit product in ten is saved: in the matrix products, in the digit planes and in every copy of them.
//   t = ((x2 - x1) q1^-1 + s) mod q2,   s = floor(Bias / q1) mod q2,   Y = q1 t + x1 + (Bias mod q1)
// is X + Bias for X = q1 (t - floor(Bias / q1)) + x1, and 0 <= Y < q1 q2 + q1 <= 256^9, so the bytes of Y, each xor 0x80, are the
// balanced digits of X (pcmm_host.hpp decides which primes qualify and derives the constants).
// Bound: HBM, 16 bytes read and 9 written per pair of residues; about 45 vector instructions per pair, a third of what
// the memory time hides.  Layout as in split_kernel with one 16-column fragment per tile (NT = 1) and nine digits.
template <int NT_ACCESS>
__global__ __launch_bounds__(256) void split_pair_kernel(const uint64_t *__restrict__ A, int8_t *__restrict__ Ad,
                                                         int64_t K, int64_t Ncols, int64_t nkb, int64_t ntiles,
                                                         PairConsts pcs)
{
    constexpr int D = pcmm_host::kPairDigits;
    const int lane = threadIdx.x & 63;
    const int g = threadIdx.x >> 6;
    const int64_t kb = blockIdx.y;
    const int64_t pair = blockIdx.z;
    const int64_t n = (int64_t)blockIdx.x * 64 + lane;
    const int64_t ntile = n >> 4;
    if (ntile >= ntiles) return;
    const pcmm_host::PairConst pc = pcs.c[pair];

    const int64_t k0 = kb * 64 + g * 16;
    const uint64_t *src1 = A + (2 * pair * K + k0) * Ncols + n;
    const uint64_t *src2 = src1 + K * Ncols;
    uint64_t x1[16], x2[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const bool in = k0 + j < K && n < Ncols;
        x1[j] = in ? residue<NT_ACCESS>(&src1[(int64_t)j * Ncols]) : 0;
        x2[j] = in ? residue<NT_ACCESS>(&src2[(int64_t)j * Ncols]) : 0;
    }
    uint32_t out[D][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t y0[4], y1[4], y2[4];               // Y = y0 + 2^32 y1 + 2^64 y2
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint64_t u1 = x1[4 * i + r], u2 = x2[4 * i + r];
            // residues as doubles: placed in the low mantissa bits of 2^52 + x, whose difference is exact
            constexpr uint64_t kMagic = 0x4330000000000000ull;
            const double dx = __longlong_as_double(u2 | kMagic) - __longlong_as_double(u1 | kMagic);
            // -q1 < dx < q2 and q1 < 2 q2, so |mulmod| <= 0.75 q2 + 1; 0 <= s < q2: -0.75 q2 - 1 <= v < 1.75 q2 + 1, which
            // is within one q2 of [0, q2), and canonical takes far more
            const double v = mulmod(pc.inv, dx, pc.q2, pc.invq2) + pc.s;
            const uint64_t t = (uint64_t)__double_as_longlong(canonical(v, pc.q2, pc.invq2, pc.half_invq2) + 4503599627370496.0);
            const uint32_t tl = (uint32_t)t, th = (uint32_t)(t >> 32) & 0xFu;
            const uint64_t c = u1 + pc.bias_mod_q1;
            const uint32_t ql = (uint32_t)pc.q1, qh = (uint32_t)(pc.q1 >> 32);
            const uint64_t p0 = (uint64_t)tl * ql + (uint32_t)c;
            const uint64_t p1 = (uint64_t)tl * qh + (uint64_t)th * ql + (p0 >> 32) + (c >> 32);
            y0[r] = (uint32_t)p0;
            y1[r] = (uint32_t)p1;
            y2[r] = (uint32_t)(p1 >> 32) + th * qh;
        }
        uint32_t t0[4], t1[4];                      // four digits of four values each
        transpose_bytes(y0, t0);
        transpose_bytes(y1, t1);
#pragma unroll
        for (int d = 0; d < 4; ++d) { out[d][i] = t0[d]; out[4 + d][i] = t1[d]; }
        out[8][i] = y2[0] | (y2[1] << 8) | (y2[2] << 16) | (y2[3] << 24);
    }
    int8_t *chunk = Ad + ((pair * nkb + kb) * ntiles + ntile) * (D * kFrag);
#pragma unroll
    for (int d = 0; d < D; ++d) {
        v4i v;
        v.x = (int)(out[d][0] ^ 0x80808080u);
        v.y = (int)(out[d][1] ^ 0x80808080u);
        v.z = (int)(out[d][2] ^ 0x80808080u);
        v.w = (int)(out[d][3] ^ 0x80808080u);
        store_digits<NT_ACCESS>(v, chunk + d * kFrag + (g * 16 + (int)(n & 15)) * 16);
    }
}

// ------------------------------------------------------------------------------------------------
// run-time kernel 2: int8 MFMA main loop + recombination + Barrett
// ------------------------------------------------------------------------------------------------
struct GemmArgs {
    const int8_t *Wp;       // [S][nkb][MB][64][16]
    const int8_t *Ad;       // [L][nkb][ntiles][NT][D][64][16]
    uint64_t *C;            // [L][M][Ncols]
    const LimbConst *lc;    // [L]
    int64_t M, Ncols;
    int64_t MB;             // padded M / 16
    int nkb;                // padded K / 64: k-steps in the layouts of Wp and Ad
    int kb0, nkbc;          // this launch contracts k-steps [kb0, kb0 + nkbc), nkbc >= 2
    int nt_stores;          // C is stored non-temporally (pcmm_host::gemm_nt_stores)
    int accumulate;         // 0: C = result;  1: C = (C + result) mod q  (later slices of a long K)
    int mtiles, ntiles, L;
    int gn;                 // n-tiles per raster group
    int64_t per_xcd;        // work items per XCD
    int64_t total;          // L * mtiles * ntiles
};

// Work-group tile: (WM waves x MT fragments x 16) rows by (NT x 16) columns, all D digit planes.
// Each wave owns MT*16 rows and keeps E = D+S-1 int32 accumulators per output: accumulator e sums
// the products W_slice_s x digit_d with s + d = e, which all carry the weight 256^e.
// W fragments go global -> registers (each wave reads only its own rows); digit fragments are shared
// by all waves and staged through LDS.
//
// EPI_F64_PAIR: the digits are those of limb pairs (split_pair_kernel), "limb" below counts pairs, and the epilogue
// reduces every sum modulo both primes of the pair.  Nine accumulators per output then leave room for one 16-column
// fragment (NT = 1): the wave tile is 64 x 16, four W fragments and nine digit fragments feed 36 MFMAs per k-step.
// Measured (whole pcmm_run, single limbs -> pairs): 4096 x 4096 by 4096 x 32768, four 36-bit limbs 9.25 -> 8.81 ms;
// 14336 rows 29.66 -> 28.16 ms; 14336 values of k, three limbs (a pair and a single) 23.80 -> 22.59 ms.
//
// Work done for padding: a contraction of an odd number of k-steps runs its first k-step in the second phase of the pipeline
// instead of taking a k-step of zeros along, and a wave whose rows all lie beyond M only moves its share of the digit chunks.
// (A three-step tail of its own for odd counts took 20 to 40 registers more and the two-wave kernels past 256, one wave on
// a SIMD instead of two: 128 x 4096 by 4096 x 16384, two 38-bit limbs 444 us without, 459 with, 442 this way; 64 x 1024 by
// 1024 x 16384, int16 W, two 62-bit limbs 158, 162 and 159 us.)
// Measured (pcmm_run, before -> after): 1000 x 777 by 777 x 12300, three 45-bit limbs 333 -> 319 us; 2100 x 160 by
// 160 x 16384, four 36-bit limbs 377 -> 334 us; 300 x 4160 by 4160 x 16384, two limbs 553 -> 526 us; 3000 x 320 by
// 320 x 16384, int16 W, two 55-bit limbs 729 -> 687 us; whole tiles and even counts equal (4096 x 4096: 8.69 and 8.70 ms).
//
// ALONE: one wave on a SIMD (the descriptor asks for more than 256 registers; the code is the same).  A second two-wave
// work-group of a compute unit otherwise lands on the SIMDs of the first while the two others idle.  Launches of at most two
// work-groups a compute unit take this variant (shared -> alone: 64 x 96 by 96 x 4332, int16 W, two 60-bit limbs, 272
// work-groups 22.1 -> 18.7 us; 64 x 300 by 300 x 8192, two 56-bit limbs, 512 work-groups 29.3 -> 27.2; 1024 work-groups,
// 64 x 96 by 96 x 16384 31.6 -> 34.6, hence the line).
template <int WM, int MT, int NT, int D, int S, int EPI, bool ALONE = false>
__global__ __launch_bounds__(WM * 64) __attribute__((amdgpu_waves_per_eu(1, ALONE ? 1 : 8))) void gemm_kernel(GemmArgs a)
{
    constexpr int E = D + S - 1;
    constexpr int T = WM * 64;
    constexpr int CH = NT * D * kFrag;            // bytes of one digit chunk (one k-step)
    // a chunk is moved by all threads: NFULL 16-byte units each and a rest of TAIL = 4, 8 or 0 bytes each, so that no
    // byte is fetched or written to LDS twice
    constexpr int NFULL = CH / (16 * T), TAIL = (CH - NFULL * 16 * T) / T;
    constexpr int NLD = NFULL + (TAIL ? 1 : 0);
    static_assert(NFULL * 16 * T + TAIL * T == CH && (TAIL == 0 || TAIL == 4 || TAIL == 8), "a chunk is cut evenly");
    constexpr int LP = EPI == EPI_F64_PAIR ? 2 : 1;   // limbs that share a set of digits
    static_assert(NT == 2 || (NT == 1 && LP == 2), "a k-step is processed in 16-column parts");

    __shared__ __attribute__((aligned(16))) int8_t lds[2][CH];

    // ---- which tile: XCD-aware raster.  Work-groups are dealt round-robin to the 8 XCDs, so
    // bid % 8 names the XCD; each XCD walks its own contiguous range of tiles in groups of gn n-tiles
    // x all m-tiles, n fastest inside a group, so that the tiles resident on one XCD (an 8 x 8 block
    // for gn = 8) share W rows and digit columns in that XCD's L2.
    const int64_t bid = blockIdx.x;
    const int64_t t = (bid % kXcd) * a.per_xcd + bid / kXcd;
    if (bid / kXcd >= a.per_xcd || t >= a.total) return;
    const int64_t per_limb = (int64_t)a.mtiles * a.ntiles;
    const int limb = (int)(t / per_limb);
    const int64_t rem = t % per_limb;
    const int64_t grp = rem / ((int64_t)a.gn * a.mtiles);
    const int64_t within = rem % ((int64_t)a.gn * a.mtiles);
    const int gcount = (int)min((int64_t)a.gn, a.ntiles - grp * a.gn);
    const int tm = (int)(within / gcount);
    const int tn = (int)(grp * a.gn + within % gcount);

    const int lane = threadIdx.x & 63;
    // the wave index is the same in all lanes: say so, so that addresses derived from it stay in
    // scalar registers and loads take the (scalar base + 32-bit lane offset) form
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nkb = a.nkbc;                                   // k-steps of this launch, numbered from 0 below
    const int64_t kleft = a.nkb - a.kb0;                      // k-steps from kb0 to the end of the layouts

    // chunk kb0 of this tile; k-step stride ntiles*CH
    const int8_t *Adc = a.Ad + (((int64_t)limb * a.nkb + a.kb0) * a.ntiles + tn) * CH;
    const int64_t mb0 = ((int64_t)tm * WM + wave) * MT;       // first 16-row block of this wave
    // Both operands are fetched with buffer loads: a scalar descriptor (base + size, out-of-range reads
    // return 0), a scalar byte offset for the k-step and a 32-bit lane offset, so that no vector ALU
    // work goes into addresses.  One descriptor per W slice and one for this limb's digit chunks.
    // Both arrays are k-step major, so that the work-groups running the same k-step at the same time read
    // one contiguous region (spread over all L2 channels) rather than addresses a power of two apart.
    const uint32_t loff = (uint32_t)lane * 16u;
    __amdgpu_buffer_rsrc_t wrs[S];
#pragma unroll
    for (int sl = 0; sl < S; ++sl)
        wrs[sl] = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<int8_t *>(a.Wp + (((int64_t)sl * a.nkb + a.kb0) * a.MB + mb0) * kFrag), 0,
            (uint32_t)((kleft * a.MB - mb0) * kFrag), 0x00020000);
    const __amdgpu_buffer_rsrc_t ars =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t *>(Adc), 0,
                                          (uint32_t)((kleft * a.ntiles - tn) * CH), 0x00020000);
    // byte offsets of a k-step: unsigned 32-bit products (one limb of digit chunks may take up to 4 GiB)
    const uint32_t w_kstride = (uint32_t)a.MB * (uint32_t)kFrag;     // bytes between k-steps of W
    const uint32_t a_kstride = (uint32_t)a.ntiles * (uint32_t)CH;    // bytes between k-steps of the digit chunks
    auto ld_w = [&](int sl, int wi, int kk) -> v4i {   // fragment (slice sl, row block wi, k-step kk)
        return (v4i)__builtin_amdgcn_raw_buffer_load_b128(
            wrs[sl], loff, (int)((uint32_t)kk * w_kstride + (uint32_t)(wi * kFrag)), 0);
    };
    // byte offsets of this thread's units inside a chunk (the same in global memory and in LDS)
    const uint32_t uoff = (uint32_t)threadIdx.x * 16u;
    const uint32_t toff = (uint32_t)(NFULL * 16 * T) + (uint32_t)threadIdx.x * (uint32_t)TAIL;
    struct Staged {
        v4i full[NFULL];
        v2u tail;
    };
    auto ld_a = [&](Staged &x, auto ic, int kk) {      // unit ic of digit chunk kk: global -> registers
        constexpr int i = decltype(ic)::value;
        const int off = (int)((uint32_t)kk * a_kstride);
        if constexpr (i < NFULL) x.full[i] = (v4i)__builtin_amdgcn_raw_buffer_load_b128(ars, uoff + (uint32_t)(i * 16 * T), off, 0);
        else if constexpr (TAIL == 8) x.tail = (v2u)__builtin_amdgcn_raw_buffer_load_b64(ars, toff, off, 0);
        else x.tail[0] = __builtin_amdgcn_raw_buffer_load_b32(ars, toff, off, 0);
    };
    auto st_a = [&](const Staged &x, auto ic, int buf) {   // registers -> LDS
        constexpr int i = decltype(ic)::value;
        if constexpr (i < NFULL) *reinterpret_cast<v4i *>(&lds[buf][uoff + (uint32_t)(i * 16 * T)]) = x.full[i];
        else if constexpr (TAIL == 8) *reinterpret_cast<v2u *>(&lds[buf][toff]) = x.tail;
        else *reinterpret_cast<uint32_t *>(&lds[buf][toff]) = x.tail[0];
    };

    // 1: an odd number of k-steps, the two-phase pipeline below is entered in phase 1 (k-step kb in phase (kb + odd) & 1,
    // its digit chunk in that LDS buffer)
    int odd = 0;
    if constexpr (pcmm_host::odd_ksteps(S, MT)) odd = nkb & 1;

    // A wave whose rows all lie in the padding of the last m-tile: the same copies and barriers as below, no products.
    if (mb0 * 16 >= a.M) {
        Staged x, y;
        static_for<NLD>([&](auto ic) { ld_a(x, ic, 0); });
        static_for<NLD>([&](auto ic) { ld_a(y, ic, 1); });
        static_for<NLD>([&](auto ic) { st_a(x, ic, odd); });
        __syncthreads();
        for (int kb = 0; kb < nkb - 1; ++kb) {
            static_for<NLD>([&](auto ic) { st_a(y, ic, (kb + 1 + odd) & 1); });
            if (kb + 2 < nkb) static_for<NLD>([&](auto ic) { ld_a(y, ic, kb + 2); });
            __syncthreads();
        }
        return;
    }

    // accumulator (i, j, e) = registers a[4*((i*NT + j)*E + e) ...+4)
    constexpr int NACC = 4 * MT * NT * E;
    acc_declare<NACC>();
    static_for<NACC>([&](auto ic) { acc_zero<decltype(ic)::value>(); });
    mfma_drain();

    // Software pipeline, one k-step = 64 k, LDS double-buffered, one barrier per k-step:
    //   W fragments   global -> wreg[2], loaded one k-step ahead of use
    //   digit chunk   global -> areg (second half of k-step kb-1) -> LDS[(kb+1+odd)&1] (first half of kb)
    //   digit operand LDS -> b, read at the start of each 16-column half
    // The kernel is sized to at most 256 registers per lane so that two work-groups share a CU:
    // the second wave on each SIMD issues MFMAs while the first waits on LDS, memory or the barrier.
    // Memory instructions are spread between the MFMAs, because a wave issues in order and a burst
    // of LDS writes (about 64 B/clk per CU) would hold back the MFMAs queued behind it.
    // The last two k-steps run without the loads that would reach past the contraction.
    v4i wreg[2][S][MT];
    Staged areg;
    v4i b[D];
    constexpr int CNT = D * S * MT;                  // MFMAs per 16-column part of a k-step
    constexpr int NW = S * MT;                       // W fragments per k-step
    // MFMA order within a k-step: digit by digit, the W fragments forwards for one digit and backwards
    // for the next, so that every MFMA shares one operand with the one before it (less switching at the
    // matrix cores' inputs: the kernel is power-limited, and this order measures 0.7 % faster)
    auto snake = [](int digit, int f) constexpr { return (digit & 1) ? NW - 1 - f : f; };

    // prologue: everything the first k-step and the LDS fill of the second need is requested at once,
    // so that a tile start pays one memory latency, not two (nkb >= 2).  The limb's constants come
    // first and are moved to scalar registers: a vector load still in flight when the epilogue
    // branches around padding blocks would make the compiler wait for it behind the first stores.
    LimbConst lc, lc2;                               // lc2: the second limb of a pair
    {
        constexpr int LCW = sizeof(LimbConst) / 4;
        static_assert(sizeof(LimbConst) % 4 == 0, "LimbConst is read word by word");
        const uint32_t *src = reinterpret_cast<const uint32_t *>(a.lc + LP * limb);
        uint32_t w[LP * LCW];
#pragma unroll
        for (int i = 0; i < LP * LCW; ++i) w[i] = src[i];
        Staged first;
        static_for<NLD>([&](auto ic) { ld_a(first, ic, 0); });
#pragma unroll
        for (int f = 0; f < NW; ++f) {
            if (odd) wreg[1][f / MT][f % MT] = ld_w(f / MT, f % MT, 0);
            else wreg[0][f / MT][f % MT] = ld_w(f / MT, f % MT, 0);
        }
        static_for<NLD>([&](auto ic) { ld_a(areg, ic, 1); });
#pragma unroll
        for (int i = 0; i < LP * LCW; ++i) w[i] = __builtin_amdgcn_readfirstlane(w[i]);
        __builtin_memcpy(&lc, w, sizeof(lc));
        __builtin_memcpy(&lc2, w + (LP - 1) * LCW, sizeof(lc2));
        static_for<NLD>([&](auto ic) { st_a(first, ic, odd); });
    }
    __syncthreads();

    // One k-step.  FILL: k-step kb+1 exists (fetch its W fragments, move its digit chunk to LDS);
    // AHEAD: k-step kb+2 exists (request its digit chunk).  The last two k-steps run without the
    // loads that would have nowhere to go, so that no load is in flight when the epilogue starts: a
    // wait for one placed behind the first stores would, the counter being in order, wait for those
    // stores to complete.
    auto step = [&](auto phase, auto fill, auto ahead, int kb) {
        constexpr int CUR = decltype(phase)::value, NXT = CUR ^ 1;
        constexpr bool FILL = decltype(fill)::value, AHEAD = decltype(ahead)::value;
        const int kw = kb + 1;
        const int ka = kb + 2;
        // Memory instructions of the k-step, in order: the W loads of k-step kb+1, the LDS writes of chunk kb+1 (which
        // free the staging registers), the loads of digit chunk kb+2.  With two column parts the first part takes the
        // first two groups and the second part the third; with one part all three are spread over it.
        constexpr int OPS_FILL = FILL ? NW + NLD : 0, OPS_AHEAD = AHEAD ? NLD : 0;
        auto memory_op = [&](auto nc) {
            constexpr int n = decltype(nc)::value;
            if constexpr (n < OPS_FILL) {
                if constexpr (n < NW) wreg[NXT][n / MT][n % MT] = ld_w(n / MT, n % MT, kw);
                else st_a(areg, std::integral_constant<int, n - NW>{}, NXT);
            } else {
                ld_a(areg, std::integral_constant<int, n - OPS_FILL>{}, ka);
            }
        };
        static_for<NT>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            constexpr int FIRST = j == 0 ? 0 : OPS_FILL;
            constexpr int OPS = (j == NT - 1 ? OPS_FILL + OPS_AHEAD : OPS_FILL) - FIRST;
#pragma unroll
            for (int d = 0; d < D; ++d)
                b[d] = *reinterpret_cast<const v4i *>(&lds[CUR][(j * D + d) * kFrag + lane * 16]);
            static_for<CNT>([&](auto mc) {
                constexpr int m = decltype(mc)::value;
                constexpr int n_lo = (m * OPS + CNT - 1) / CNT, n_hi = ((m + 1) * OPS + CNT - 1) / CNT;
                static_for<n_hi - n_lo>([&](auto oc) {
                    memory_op(std::integral_constant<int, FIRST + n_lo + decltype(oc)::value>{});
                });
                constexpr int d = m / NW, f = snake(j * D + d, m % NW), ws = f / MT, wi = f % MT;
                mfma_i8<4 * ((wi * NT + j) * E + d + ws)>(wreg[CUR][ws][wi], b[d]);
            });
        });
        if constexpr (FILL) __syncthreads();   // chunk kb+1 is in LDS; buffer CUR may be refilled
    };
    {
        using P0 = std::integral_constant<int, 0>;
        using P1 = std::integral_constant<int, 1>;
        int kb = odd;                     // the last two k-steps always run in phases 0 and 1
        if (odd) step(P1{}, std::true_type{}, std::true_type{}, 0);
        for (; kb + 2 < nkb; kb += 2) {
            step(P0{}, std::true_type{}, std::true_type{}, kb);
            step(P1{}, std::true_type{}, std::true_type{}, kb + 1);
        }
        step(P0{}, std::true_type{}, std::false_type{}, kb);
        step(P1{}, std::false_type{}, std::false_type{}, kb + 1);
    }

    // volatile asm statements keep their order: last MFMA, drain, accumulator reads
    mfma_drain();
    // Every load has been consumed by now.  Saying so with a wait the compiler sees keeps it from
    // placing one of its own (for a load it cannot prove finished on some path) behind the first stores.
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)

    // ---- epilogue.  Accumulator register r of lane l is output row 4*(l/16)+r, column l%16 of its
    // 16 x 16 block.
    // Stores go through a buffer descriptor that covers exactly the valid rows of the 16-row block:
    // rows at or beyond M fall outside it and are dropped by the range check, and lanes whose column
    // is at or beyond Ncols get an offset that is out of range for every row; no address arithmetic
    // or branching per output.
    uint64_t *Cl = a.C + (int64_t)(LP * limb) * a.M * a.Ncols;
    const uint32_t c_rowbytes = (uint32_t)a.Ncols * 8u;
    // The whole epilogue exists three times, with the read-add of the previous contents of C and without it for both kinds of stores,
    // chosen once per wave: a branch per output would stop the scheduler from overlapping outputs.
    auto store_block = [&](__amdgpu_buffer_rsrc_t crs, uint32_t c_lane, uint64_t (&res)[4], uint64_t q, auto accumulate_c, auto nt_c) {
        if constexpr (decltype(accumulate_c)::value) {   // rows and columns outside C read as 0
            v2u old[4];
#pragma unroll
            for (int r = 0; r < 4; ++r)
                old[r] = __builtin_amdgcn_raw_buffer_load_b64(crs, c_lane + (uint32_t)r * c_rowbytes, 0, 0);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                res[r] += (uint64_t)old[r][0] | ((uint64_t)old[r][1] << 32);
                if (res[r] >= q) res[r] -= q;
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
            __builtin_amdgcn_raw_buffer_store_b64((v2u){(uint32_t)res[r], (uint32_t)(res[r] >> 32)}, crs,
                                                  c_lane + (uint32_t)r * c_rowbytes, 0, decltype(nt_c)::value ? 2 : 0);
    };
    auto epilogue = [&](auto accumulate_c, auto nt_c) {
    static_for<MT * NT>([&](auto ijc) {
        constexpr int i = decltype(ijc)::value / NT, j = decltype(ijc)::value % NT;
        // 16 x 16 blocks that lie wholly in the padding are skipped (wave-uniform)
        if ((mb0 + i) * 16 < a.M && ((int64_t)tn * NT + j) * 16 < a.Ncols) {
            const int64_t m0 = (mb0 + i) * 16;
            const uint32_t rows_valid = (uint32_t)min((int64_t)16, a.M - m0);
            const __amdgpu_buffer_rsrc_t crs =
                __builtin_amdgcn_make_buffer_rsrc(Cl + m0 * a.Ncols, 0, rows_valid * c_rowbytes, 0x00020000);
            const int64_t n = ((int64_t)tn * NT + j) * 16 + (lane & 15);
            const uint32_t c_lane = n < a.Ncols ? (uint32_t)((lane >> 4) * 4) * c_rowbytes + (uint32_t)n * 8u
                                                : 0x80000000u;
            // all accumulators of the block's four outputs first (the reads are volatile and keep their
            // order), so that the four reductions are independent chains the scheduler can interleave
            int avs[4][E];
            static_for<4 * E>([&](auto rec) {
                constexpr int r = decltype(rec)::value / E, e = decltype(rec)::value % E;
                avs[r][e] = acc_read<4 * ((i * NT + j) * E + e) + r>();
            });
            if constexpr (LP == 2) {              // one residue of each limb from the same accumulators
                uint64_t res1[4], res2[4];
                reduce_f64_pair<E, 4>(avs, lc.qd, lc.invq, lc2.qd, lc2.invq, res1, res2);
                const __amdgpu_buffer_rsrc_t crs2 = __builtin_amdgcn_make_buffer_rsrc(
                    Cl + (a.M + m0) * a.Ncols, 0, rows_valid * c_rowbytes, 0x00020000);
                store_block(crs, c_lane, res1, lc.q, accumulate_c, nt_c);
                store_block(crs2, c_lane, res2, lc2.q, accumulate_c, nt_c);
                return;
            }
            uint64_t res[4];
            if constexpr (EPI == EPI_F64) {
                reduce_f64<E, 0, 4>(avs, lc.qd, lc.invq, res);
            } else if constexpr (EPI == EPI_F64_G4) {
                reduce_f64<E, 1, 4>(avs, lc.qd, lc.invq, res);
            } else if constexpr (EPI == EPI_F64_G4P) {
                reduce_f64<E, 2, 4>(avs, lc.qd, lc.invq, res);
            } else {
                reduce_int<E, 4>(avs, lc, res);
            }
            store_block(crs, c_lane, res, lc.q, accumulate_c, nt_c);
        }
    });
    };
    if (a.accumulate) epilogue(std::true_type{}, std::false_type{});
    else if (a.nt_stores) epilogue(std::false_type{}, std::true_type{});
    else epilogue(std::false_type{}, std::false_type{});
}

// ------------------------------------------------------------------------------------------------
// ring switching: coefficient permutation either side of the PCMM (HBM-bound)
// ------------------------------------------------------------------------------------------------
// out[p][c][r] = in[p][r][c] for npoly matrices of R x C 64-bit words, R and C powers of two.
// Decomposition p(X) = sum_j p_j(X^k) X^j is the case R = N/k, C = k (coefficient i*k + j of p becomes
// coefficient i of p_j); composition is R = k, C = N/k.  One block moves a TR x TC tile (TR*TC = 4096
// words unless the matrix is smaller) through LDS, so that both the reads (along c) and the writes
// (along r) are contiguous runs of at least 128 bytes whenever the matrix allows it.  The row pitch
// TC + 1 keeps the column-wise LDS reads off a single bank.
constexpr int kTransposeWords = 4096;   // words per tile
constexpr int kTransposeMaxTR = 512;    // most rows per tile (tiles of narrow matrices)
// Stores are non-temporal: the output is written once and not read here (2^16-coefficient polynomials, k = 16: 816 ->
// 721 us for 2 GiB in, 93 -> 76 us for 256 MiB in, equal from 8 MiB down).  The call that reads the parts next pays for it
// where cached stores would have left them in the last-level cache, and gains where they would have pushed out what it reads
// (cached -> non-temporal, four sets of buffers in turn: decompose 32 MiB and a product of 128 rows 29.9 -> 31.3 us, 64 MiB
// and 512 rows 81.6 -> 84.6, 128 MiB and 512 rows 173 -> 171; decompose, product and compose 32 MiB 46.2 -> 46.5, 64 MiB 105
// and 105, 128 MiB 221 -> 205; the permutation of 64 MiB by itself 24.9 -> 20.2): no line on the size was better over all.
// Loads are non-temporal (NT_LOADS) for inputs larger than the 256 MiB last-level cache, where no later pass can find the
// input there (2 GiB in: 721 -> 685 us; 512 MiB: 175 -> 166 us; 256 MiB: 76 -> 82 us, hence the line).
constexpr int64_t kLastLevelCacheBytes = (int64_t)256 << 20;
template <bool NT_LOADS>
__global__ __launch_bounds__(256) void transpose_u64_kernel(const uint64_t *__restrict__ in, uint64_t *__restrict__ out,
                                                            int64_t R, int64_t C, int lTR, int lTC, int64_t tiles_r,
                                                            int64_t tiles_c)
{
    __shared__ uint64_t tile[kTransposeWords + kTransposeMaxTR];     // TR * (TC + 1) words at most
    const int TR = 1 << lTR, TC = 1 << lTC;
    const int64_t b = blockIdx.x;
    const int64_t tc = b % tiles_c, tr = (b / tiles_c) % tiles_r, poly = b / (tiles_c * tiles_r);
    const uint64_t *src = in + poly * R * C + (tr << lTR) * C + (tc << lTC);
    uint64_t *dst = out + poly * R * C + (tc << lTC) * R + (tr << lTR);
    const int n = TR * TC;
    const int pitch = TC + 1;
    if (n == kTransposeWords) {   // full tile: 16 words per thread, all loads in flight before the first use
        uint64_t v[16];
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            const int idx = threadIdx.x + 256 * s;
            const uint64_t *word = &src[(int64_t)(idx >> lTC) * C + (idx & (TC - 1))];
            v[s] = NT_LOADS ? __builtin_nontemporal_load(word) : *word;
        }
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            const int idx = threadIdx.x + 256 * s;
            tile[(idx >> lTC) * pitch + (idx & (TC - 1))] = v[s];
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            const int idx = threadIdx.x + 256 * s;
            const int c = idx >> lTR, r = idx & (TR - 1);
            __builtin_nontemporal_store(tile[r * pitch + c], &dst[(int64_t)c * R + r]);
        }
        return;
    }
    for (int idx = threadIdx.x; idx < n; idx += 256) {
        const int r = idx >> lTC, c = idx & (TC - 1);
        tile[r * pitch + c] = src[(int64_t)r * C + c];
    }
    __syncthreads();
    for (int idx = threadIdx.x; idx < n; idx += 256) {
        const int c = idx >> lTR, r = idx & (TR - 1);
        dst[(int64_t)c * R + r] = tile[r * pitch + c];
    }
}

// ------------------------------------------------------------------------------------------------
// measurement: register-resident MFMA-only probe
// ------------------------------------------------------------------------------------------------
// 40 independent accumulators per wave (the footprint of the D = 5 main loop), four W-like and ten
// digit-like operand registers, no memory traffic in the loop.  Operands are pseudo-random bytes or
// zeros: the rate the matrix cores sustain depends on how much the data toggles (power).  One lane
// also reports shader-clock and wall-clock ticks.
__global__ __launch_bounds__(256) void mfma_probe_kernel(long long *out, int iters, int random_operands)
{
    const long long c0 = clock64(), w0 = wall_clock64();
    unsigned x = threadIdx.x * 2654435761u + blockIdx.x * 40503u + 12345u;
    v4i wa[4], bd[10];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            x ^= x << 13; x ^= x >> 17; x ^= x << 5;
            wa[i][j] = random_operands ? (int)x : 0;
        }
#pragma unroll
    for (int i = 0; i < 10; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            x ^= x << 13; x ^= x >> 17; x ^= x << 5;
            bd[i][j] = random_operands ? (int)x : 0;
        }
    acc_declare<160>();
    static_for<160>([&](auto ic) { acc_zero<decltype(ic)::value>(); });
    mfma_drain();
    for (int it = 0; it < iters; ++it)
        static_for<40>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            mfma_i8<4 * m>(wa[m % 4], bd[m / 4]);
        });
    mfma_drain();
    int sum = 0;
    static_for<160>([&](auto ic) { sum += acc_read<decltype(ic)::value>(); });
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        out[0] = clock64() - c0;
        out[1] = wall_clock64() - w0;
        out[2] = sum;
    }
}

}  // namespace

// ------------------------------------------------------------------------------------------------
// static digit scratch for pcmm_run_noalloc
// ------------------------------------------------------------------------------------------------
// Every GPU the library runs on holds its own copy of this array until the process ends.  Host code
// never passes the array's name to a kernel or a HIP call: it asks HIP for the device address once per
// device (static_scratch_ptr) and uses that pointer from then on.
static __device__ __align__(256) unsigned char scratch[PCMM_NOALLOC_SCRATCH_BYTES];

// ------------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------------
struct pcmm_plan {
    int64_t M, K, Ncols;
    int L, prime_bits, w_bits, device;
    int D, S;
    int WM, MT, NT;          // tile configuration
    int epi;                 // Epi: how the epilogue reduces
    int64_t MB, nkb, mtiles, ntiles;
    int64_t nkb_launch;      // most k-steps one GEMM launch may contract (int32 accumulator headroom)
    int64_t ksteps;          // k-steps that are split and contracted (the layouts hold nkb)
    int8_t *Wp;              // device
    int8_t *Ad;              // device digit scratch
    LimbConst *lc;           // device
    size_t bytes;
    size_t ad_bytes;         // size of the digit planes of one run (pcmm_run_noalloc's limit)
    bool shortk;             // at most 128 values of k: pcmm_shortk runs, which needs no digit scratch
    pcmm_host::ResidentTile resident;   // NT > 0: pcmm_resident runs, which needs none either
    int pairs;               // limb pairs whose digits are split jointly; limbs from 2 * pairs on run singly
    int64_t pair_ntiles;     // n-tiles (16 columns) of a pair
    int gn, pair_gn;         // n-tiles per raster group
    PairConsts pcs;
    hipEvent_t ev[4];
    bool have_ev;
};

namespace {

using pcmm_host::tile_mt;
using pcmm_hip_util::DevGuard;

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices];   // device address of `scratch` on each device, nullptr until asked for

// Device address of this device's copy of `scratch`; `device` must be the current device.
// nullptr if HIP cannot tell.
int8_t *static_scratch_ptr(int device)
{
    if (device < 0 || device >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[device]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) {
            (void)hipGetLastError();
            return nullptr;
        }
        g_scratch_ptr[device] = ptr;
    }
    return static_cast<int8_t *>(g_scratch_ptr[device]);
}

// bytes of the digit planes of all limb pairs
int64_t pair_digit_bytes(const pcmm_plan *p)
{
    return p->pairs * p->nkb * p->pair_ntiles * (int64_t)(pcmm_host::kPairDigits * kFrag);
}

template <int WM, int MT, int NT, int D, int S, int EPI>
void launch_alone_or_not(const GemmArgs &ga, dim3 g, hipStream_t st)
{
    if constexpr (WM == 2) {
        if (ga.total <= 2 * 256) {               // two for each of 256 compute units
            hipLaunchKernelGGL((gemm_kernel<WM, MT, NT, D, S, EPI, true>), g, dim3(WM * 64), 0, st, ga);
            return;
        }
    }
    hipLaunchKernelGGL((gemm_kernel<WM, MT, NT, D, S, EPI>), g, dim3(WM * 64), 0, st, ga);
}

template <int WM, int MT, int NT, int D, int S>
hipError_t launch_gemm_ds(const pcmm_plan *p, const GemmArgs &ga, int64_t grid, hipStream_t st)
{
    const dim3 g((unsigned)grid);
    // 50-bit primes need at least 7 digits and 7-digit primes can be below 2^50: D <= 6 always takes
    // the double-precision epilogue, D = 8 never does
    if (p->epi == EPI_F64) {
        if constexpr (D <= 7) launch_alone_or_not<WM, MT, NT, D, S, EPI_F64>(ga, g, st);
        else return hipErrorInvalidValue;
    } else if (p->epi == EPI_F64_G4 || p->epi == EPI_F64_G4P) {
        if constexpr (D <= 7 && D + S - 1 >= 7) {
            // the grouping of short contractions (G4P) only for four waves: those of few rows, if they come here at all, have
            // accumulators small enough for either grouping
            if constexpr (WM == 4) {
                if (p->epi == EPI_F64_G4P) launch_alone_or_not<WM, MT, NT, D, S, EPI_F64_G4P>(ga, g, st);
                else launch_alone_or_not<WM, MT, NT, D, S, EPI_F64_G4>(ga, g, st);
            } else launch_alone_or_not<WM, MT, NT, D, S, EPI_F64_G4>(ga, g, st);
        } else return hipErrorInvalidValue;
    } else {
        if constexpr (D >= 7) {
            launch_alone_or_not<WM, MT, NT, D, S, EPI_INT>(ga, g, st);
        } else return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int D, int S>
hipError_t launch_gemm_tile(const pcmm_plan *p, const GemmArgs &ga, int64_t grid, hipStream_t st)
{
    constexpr int MT = tile_mt(D + S - 1);
    if (p->MT != MT || p->NT != 2) return hipErrorInvalidValue;
    if (p->WM == 4) return launch_gemm_ds<4, MT, 2, D, S>(p, ga, grid, st);
    if (p->WM == 2) return launch_gemm_ds<2, MT, 2, D, S>(p, ga, grid, st);
    return hipErrorInvalidValue;
}

hipError_t launch_gemm(const pcmm_plan *p, const GemmArgs &ga, int64_t grid, hipStream_t st)
{
    if (p->S == 1) {
        switch (p->D) {
        case 4: return launch_gemm_tile<4, 1>(p, ga, grid, st);
        case 5: return launch_gemm_tile<5, 1>(p, ga, grid, st);
        case 6: return launch_gemm_tile<6, 1>(p, ga, grid, st);
        case 7: return launch_gemm_tile<7, 1>(p, ga, grid, st);
        case 8: return launch_gemm_tile<8, 1>(p, ga, grid, st);
        }
    } else {
        switch (p->D) {
        case 4: return launch_gemm_tile<4, 2>(p, ga, grid, st);
        case 5: return launch_gemm_tile<5, 2>(p, ga, grid, st);
        case 6: return launch_gemm_tile<6, 2>(p, ga, grid, st);
        case 7: return launch_gemm_tile<7, 2>(p, ga, grid, st);
        case 8: return launch_gemm_tile<8, 2>(p, ga, grid, st);
        }
    }
    return hipErrorInvalidValue;
}

// digit split of all limbs: pairs first (their digit planes come first in the scratch), then the rest
hipError_t launch_split(const pcmm_plan *p, int8_t *Ad, const uint64_t *A, hipStream_t st)
{
    const dim3 block(256);
    const pcmm_host::SplitNt nt = pcmm_host::split_nt(p->L, p->K, p->Ncols, (uint64_t)(uintptr_t)A);
    using pcmm_host::kNtBoth;
    using pcmm_host::kNtNone;
    using pcmm_host::kNtStores;
    if (p->pairs) {
        const dim3 grid((unsigned)((p->pair_ntiles * 16 + 63) / 64), (unsigned)p->ksteps, (unsigned)p->pairs);
        const auto kern = nt == kNtBoth ? split_pair_kernel<kNtBoth> : nt == kNtStores ? split_pair_kernel<kNtStores> : split_pair_kernel<kNtNone>;
        hipLaunchKernelGGL(kern, grid, block, 0, st, A, Ad, p->K, p->Ncols, p->nkb, p->pair_ntiles, p->pcs);
        const hipError_t rc = hipGetLastError();
        if (rc != hipSuccess) return rc;
    }
    const int single = p->L - 2 * p->pairs;
    if (!single) return hipSuccess;
    A += (int64_t)2 * p->pairs * p->K * p->Ncols;
    Ad += pair_digit_bytes(p);
    int64_t colblocks = (p->ntiles * p->NT * 16 + 63) / 64;
    dim3 grid((unsigned)colblocks, (unsigned)p->ksteps, (unsigned)single);
#define PCMM_SPLIT_CASE(DD)                                                                              \
    case DD:                                                                                             \
        hipLaunchKernelGGL((nt == kNtBoth ? split_kernel<DD, kNtBoth> : nt == kNtStores ? split_kernel<DD, kNtStores>   \
                                                                                        : split_kernel<DD, kNtNone>),  \
                           grid, block, 0, st, A, Ad, p->K, p->Ncols, p->nkb, p->ntiles, p->NT);         \
        break;
    switch (p->D) {
        PCMM_SPLIT_CASE(4)
        PCMM_SPLIT_CASE(5)
        PCMM_SPLIT_CASE(6)
        PCMM_SPLIT_CASE(7)
        PCMM_SPLIT_CASE(8)
    default: return hipErrorInvalidValue;
    }
#undef PCMM_SPLIT_CASE
    return hipGetLastError();
}

// one launch of the general MFMA kernel over the k-steps that ga names, for all limb pairs or for the single limbs
hipError_t launch_products(const pcmm_plan *p, GemmArgs ga, bool pair, hipStream_t st)
{
    const int limb0 = pair ? 0 : 2 * p->pairs;
    ga.L = pair ? p->pairs : p->L - limb0;
    if (!ga.L) return hipSuccess;
    ga.ntiles = (int)(pair ? p->pair_ntiles : p->ntiles);
    ga.gn = pair ? p->pair_gn : p->gn;
    ga.Ad += pair ? 0 : pair_digit_bytes(p);
    ga.C += (int64_t)limb0 * p->M * p->Ncols;
    ga.lc += limb0;
    ga.total = (int64_t)ga.L * p->mtiles * ga.ntiles;
    ga.per_xcd = (ga.total + kXcd - 1) / kXcd;
    const int64_t grid = ga.per_xcd * kXcd;
    if (!pair) return launch_gemm(p, ga, grid, st);
    if (p->MT != 4 || p->S != 1) return hipErrorInvalidValue;
    constexpr int PD = pcmm_host::kPairDigits;
    if (p->WM == 4) hipLaunchKernelGGL((gemm_kernel<4, 4, 1, PD, 1, EPI_F64_PAIR>), dim3((unsigned)grid), dim3(256), 0, st, ga);
    else launch_alone_or_not<2, 4, 1, PD, 1, EPI_F64_PAIR>(ga, dim3((unsigned)grid), st);
    return hipGetLastError();
}

// Ad: the digit scratch of this run (the plan's own, or the library's static one)
pcmm_status run_impl(const pcmm_plan *p, int8_t *Ad, const uint64_t *A, uint64_t *C, hipStream_t st, float *ms)
{
    DevGuard dg(p->device);
    if (!dg.ok) return PCMM_EDEVICE;

    if (ms && hipEventRecord(p->ev[0], st) != hipSuccess) return PCMM_EDEVICE;
    if (!p->shortk && !p->resident.NT && launch_split(p, Ad, A, st) != hipSuccess) return PCMM_EDEVICE;
    if (ms && (hipEventRecord(p->ev[1], st) != hipSuccess || hipEventRecord(p->ev[2], st) != hipSuccess))
        return PCMM_EDEVICE;
    if (p->shortk) {
        // at most 128 values of k: the kernel that cuts the digits itself, keeps them in registers and walks down W
        pcmm_shortk::Args sa;
        sa.Wp = p->Wp; sa.A = A; sa.C = C; sa.lc = p->lc;
        sa.M = p->M; sa.K = p->K; sa.Ncols = p->Ncols; sa.MB = p->MB;
        sa.L = p->L;
        if (pcmm_shortk::launch(sa, p->D, p->S, p->epi, st) != hipSuccess) return PCMM_EDEVICE;
    } else if (p->resident.NT) {
        // the digits of the whole contraction fit LDS
        pcmm_resident::Args ra;
        ra.Wp = p->Wp; ra.A = A; ra.C = C; ra.lc = p->lc;
        ra.M = p->M; ra.K = p->K; ra.Ncols = p->Ncols; ra.MB = p->MB;
        ra.nkb = (int)p->nkb;
        ra.L = p->L;
        if (pcmm_resident::launch(ra, p->resident, p->D, p->S, p->epi, st) != hipSuccess) return PCMM_EDEVICE;
    } else {
        GemmArgs ga = {};
        ga.Wp = p->Wp;
        ga.Ad = Ad;
        ga.C = C;
        ga.lc = p->lc;
        ga.M = p->M;
        ga.Ncols = p->Ncols;
        ga.MB = p->MB;
        ga.nkb = (int)p->nkb;
        ga.nt_stores = pcmm_host::gemm_nt_stores(p->M, p->K, p->S, p->Ncols, (uint64_t)(uintptr_t)C);
        ga.mtiles = (int)p->mtiles;
        // A contraction longer than the int32 accumulators can hold runs as several launches over
        // consecutive ranges of k; every launch after the first adds its result to C modulo q_j.
        for (int64_t kb0 = 0; kb0 < p->ksteps; kb0 += p->nkb_launch) {
            ga.kb0 = (int)kb0;
            ga.nkbc = (int)std::min(p->nkb_launch, p->ksteps - kb0);
            ga.accumulate = kb0 > 0;
            for (bool pair : {true, false})
                if (launch_products(p, ga, pair, st) != hipSuccess) return PCMM_EDEVICE;
        }
    }
    if (ms) {
        if (hipEventRecord(p->ev[3], st) != hipSuccess) return PCMM_EDEVICE;
        if (hipEventSynchronize(p->ev[3]) != hipSuccess) return PCMM_EDEVICE;
        if (hipEventElapsedTime(&ms[0], p->ev[0], p->ev[1]) != hipSuccess) return PCMM_EDEVICE;
        if (hipEventElapsedTime(&ms[1], p->ev[2], p->ev[3]) != hipSuccess) return PCMM_EDEVICE;
    }
    return PCMM_OK;
}

}  // namespace

extern "C" {

const char *pcmm_status_str(pcmm_status s)
{
    switch (s) {
    case PCMM_OK: return "PCMM_OK";
    case PCMM_EINVAL: return "PCMM_EINVAL: invalid argument";
    case PCMM_EUNSUPPORTED: return "PCMM_EUNSUPPORTED: request outside the supported range";
    case PCMM_ENOMEM: return "PCMM_ENOMEM: allocation failed";
    case PCMM_EDEVICE: return "PCMM_EDEVICE: HIP call or kernel launch failed";
    }
    return "PCMM: unknown status";
}

pcmm_status pcmm_plan_create(pcmm_plan **out, int64_t M, int64_t K, int64_t Ncols, int32_t L,
                             const uint64_t *primes_host, int32_t prime_bits, int32_t w_bits,
                             const void *W_dev, int32_t device, void *stream)
{
    if (!out) return PCMM_EINVAL;
    *out = nullptr;
    if (!primes_host || !W_dev) return PCMM_EINVAL;
    pcmm_host::Geometry g;
    const pcmm_status grc = pcmm_host::plan_geometry(M, K, Ncols, L, primes_host, prime_bits, w_bits, device, &g);
    if (grc != PCMM_OK) return grc;
    const int D = g.D, S = g.S;

    pcmm_plan *p = new (std::nothrow) pcmm_plan();
    if (!p) return PCMM_ENOMEM;
    p->M = M; p->K = K; p->Ncols = Ncols; p->L = L;
    p->prime_bits = prime_bits; p->w_bits = w_bits; p->device = device;
    p->D = D; p->S = S;
    p->WM = g.WM; p->MT = g.MT; p->NT = g.NT;
    p->epi = g.epi;
    p->shortk = pcmm_shortk::covers(g.D, g.S, g.epi, g.nkb);
    p->resident = g.resident;
    p->MB = g.MB; p->nkb = g.nkb; p->mtiles = g.mtiles; p->ntiles = g.ntiles;
    p->nkb_launch = g.nkb_launch;
    p->ksteps = g.ksteps;
    p->pairs = g.pairs;
    p->pair_ntiles = g.pair_ntiles;
    p->gn = g.gn; p->pair_gn = g.pair_gn;
    for (int j = 0; j < g.pairs; ++j) p->pcs.c[j] = pcmm_host::pair_const(primes_host[2 * j], primes_host[2 * j + 1]);
    p->Wp = nullptr; p->Ad = nullptr; p->lc = nullptr; p->bytes = 0; p->have_ev = false;

    DevGuard dg(device);
    if (!dg.ok) { delete p; return PCMM_EDEVICE; }
    hipStream_t st = (hipStream_t)stream;
    // set-up for pcmm_run_noalloc: this device's address of the static digit scratch, asked for once
    if (!static_scratch_ptr(device)) { delete p; return PCMM_EDEVICE; }

    const size_t wp_bytes = g.wp_bytes + pcmm_host::kWpSlack, ad_bytes = p->shortk || p->resident.NT ? 0 : g.ad_bytes;   // scratch the plan owns
    const size_t lc_bytes = (size_t)L * sizeof(LimbConst);
    int *err_dev = nullptr;
    pcmm_status rc = PCMM_OK;
    if (hipMalloc((void **)&p->Wp, wp_bytes) != hipSuccess ||
        (ad_bytes && hipMalloc((void **)&p->Ad, ad_bytes) != hipSuccess) ||
        hipMalloc((void **)&p->lc, lc_bytes) != hipSuccess || hipMalloc((void **)&err_dev, sizeof(int)) != hipSuccess) {
        (void)hipGetLastError();
        rc = PCMM_ENOMEM;
    }
    p->bytes = wp_bytes + ad_bytes + lc_bytes;
    p->ad_bytes = g.ad_bytes;

    if (rc == PCMM_OK) {
        LimbConst h[pcmm_host::kMaxLimbs];
        for (int j = 0; j < L; ++j) h[j] = pcmm_host::limb_const(primes_host[j]);
        if (hipMemcpyAsync(p->lc, h, lc_bytes, hipMemcpyHostToDevice, st) != hipSuccess ||
            hipMemsetAsync(err_dev, 0, sizeof(int), st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess)   // h lives on this stack frame
            rc = PCMM_EDEVICE;
    }
    if (rc == PCMM_OK) {
        int64_t units = p->MB * p->nkb * 64;
        dim3 grid((unsigned)((units + 255) / 256)), block(256);
        if (w_bits == 8)
            hipLaunchKernelGGL((pack_w_kernel<int8_t, 1>), grid, block, 0, st, (const int8_t *)W_dev, p->Wp, M, K,
                               p->MB, p->nkb, err_dev);
        else
            hipLaunchKernelGGL((pack_w_kernel<int16_t, 2>), grid, block, 0, st, (const int16_t *)W_dev, p->Wp, M, K,
                               p->MB, p->nkb, err_dev);
        int err_host = 0;
        if (hipGetLastError() != hipSuccess ||
            hipMemcpyAsync(&err_host, err_dev, sizeof(int), hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess)
            rc = PCMM_EDEVICE;
        else if (err_host)
            rc = PCMM_EINVAL;   // an int16 entry above 32639
    }
    if (rc == PCMM_OK) {
        p->have_ev = true;
        for (int i = 0; i < 4; ++i)
            if (hipEventCreate(&p->ev[i]) != hipSuccess) {
                for (int k = 0; k < i; ++k) (void)hipEventDestroy(p->ev[k]);
                p->have_ev = false;
                rc = PCMM_EDEVICE;
                break;
            }
    }
    if (err_dev) (void)hipFree(err_dev);
    if (rc != PCMM_OK) {
        if (p->Wp) (void)hipFree(p->Wp);
        if (p->Ad) (void)hipFree(p->Ad);
        if (p->lc) (void)hipFree(p->lc);
        delete p;
        return rc;
    }
    *out = p;
    return PCMM_OK;
}

size_t pcmm_plan_workspace_bytes(const pcmm_plan *plan) { return plan ? plan->bytes : 0; }

int32_t pcmm_plan_digits(const pcmm_plan *plan) { return plan ? plan->D : 0; }

pcmm_status pcmm_run(const pcmm_plan *plan, const uint64_t *A_dev, uint64_t *C_dev, void *stream)
{
    if (!plan || !A_dev || !C_dev) return PCMM_EINVAL;
    return run_impl(plan, plan->Ad, A_dev, C_dev, (hipStream_t)stream, nullptr);
}

pcmm_status pcmm_run_profiled(const pcmm_plan *plan, const uint64_t *A_dev, uint64_t *C_dev, void *stream,
                              float *ms_out)
{
    if (!plan || !A_dev || !C_dev || !ms_out) return PCMM_EINVAL;
    return run_impl(plan, plan->Ad, A_dev, C_dev, (hipStream_t)stream, ms_out);
}

pcmm_status pcmm_run_noalloc(const pcmm_plan *plan, const uint64_t *A_dev, uint64_t *C_dev, void *stream)
{
    if (!plan || !A_dev || !C_dev) return PCMM_EINVAL;
    if (plan->ad_bytes > (size_t)PCMM_NOALLOC_SCRATCH_BYTES) return PCMM_EUNSUPPORTED;
    int8_t *ptr;
    {
        DevGuard dg(plan->device);
        if (!dg.ok) return PCMM_EDEVICE;
        ptr = static_scratch_ptr(plan->device);   // resolved by pcmm_plan_create; a table look-up here
    }
    if (!ptr) return PCMM_EDEVICE;
    // the digit split rewrites every byte of the scratch that the MFMA kernel reads, so nothing has to
    // start at zero
    return run_impl(plan, ptr, A_dev, C_dev, (hipStream_t)stream, nullptr);
}

pcmm_status pcmm_mfma_probe(int32_t device, int32_t iters, int32_t random_operands, double *tops_out,
                            double *shader_mhz_out)
{
    if (device < 0 || iters <= 0 || !tops_out || !shader_mhz_out) return PCMM_EINVAL;
    DevGuard dg(device);
    if (!dg.ok) return PCMM_EDEVICE;
    long long *dev = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    pcmm_status rc = PCMM_OK;
    const int wgs = 512;   // two work-groups of four waves per CU on 256 CUs
    float ms = 0.f;
    long long h[3] = {0, 0, 0};
    if (hipMalloc((void **)&dev, sizeof(h)) != hipSuccess) return PCMM_ENOMEM;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) rc = PCMM_EDEVICE;
    if (rc == PCMM_OK) {
        hipLaunchKernelGGL(mfma_probe_kernel, dim3(wgs), dim3(256), 0, nullptr, dev, 64, random_operands);   // warm-up
        (void)hipEventRecord(e0, nullptr);
        hipLaunchKernelGGL(mfma_probe_kernel, dim3(wgs), dim3(256), 0, nullptr, dev, iters, random_operands);
        if (hipGetLastError() != hipSuccess || hipEventRecord(e1, nullptr) != hipSuccess ||
            hipEventSynchronize(e1) != hipSuccess || hipEventElapsedTime(&ms, e0, e1) != hipSuccess ||
            hipMemcpy(h, dev, sizeof(h), hipMemcpyDeviceToHost) != hipSuccess)
            rc = PCMM_EDEVICE;
    }
    if (rc == PCMM_OK && ms > 0.f && h[1] > 0) {
        *tops_out = 2.0 * 16 * 16 * 64 * 40.0 * (double)iters * 4.0 * wgs / (ms * 1e-3) / 1e12;
        *shader_mhz_out = (double)h[0] / (double)h[1] * 100.0;   // the wall clock ticks at 100 MHz
    } else if (rc == PCMM_OK) {
        rc = PCMM_EDEVICE;
    }
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    (void)hipFree(dev);
    return rc;
}

namespace {

int log2_exact(int64_t v)   // -1 unless v is a power of two
{
    if (v <= 0 || (v & (v - 1))) return -1;
    int l = 0;
    while (((int64_t)1 << l) < v) ++l;
    return l;
}

// out[p][c][r] = in[p][r][c], R x C words, both powers of two
pcmm_status launch_transpose(const uint64_t *in, uint64_t *out, int64_t npoly, int64_t R, int64_t C, int32_t device,
                             hipStream_t st)
{
    const int lR = log2_exact(R), lC = log2_exact(C);
    if (lR < 0 || lC < 0) return PCMM_EINVAL;
    int lTC = std::min(lC, 6);
    int lTR = std::min(lR, std::min(12 - lTC, 9));       // TR * TC <= 4096, TR <= 512
    lTC = std::min(lC, 12 - lTR);                         // a short matrix gets wider tiles
    const int64_t tiles_r = R >> lTR, tiles_c = C >> lTC;
    const int64_t blocks = npoly * tiles_r * tiles_c;
    if (blocks > 0x7fffffff) return PCMM_EUNSUPPORTED;
    DevGuard dg(device);
    if (!dg.ok) return PCMM_EDEVICE;
    const auto kern = npoly * R * C * 8 > kLastLevelCacheBytes ? transpose_u64_kernel<true> : transpose_u64_kernel<false>;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), 0, st, in, out, R, C, lTR, lTC, tiles_r,
                       tiles_c);
    return hipGetLastError() == hipSuccess ? PCMM_OK : PCMM_EDEVICE;
}

pcmm_status ring_args_ok(const void *in, const void *out, int64_t npoly, int64_t N, int64_t k, int32_t device)
{
    if (!in || !out || in == out || npoly <= 0 || device < 0) return PCMM_EINVAL;
    if (log2_exact(N) < 0 || log2_exact(k) < 0 || k > N || N > ((int64_t)1 << 24)) return PCMM_EINVAL;
    if (npoly > ((int64_t)1 << 40) / N) return PCMM_EUNSUPPORTED;
    return PCMM_OK;
}

}  // namespace

pcmm_status pcmm_ring_decompose(const uint64_t *in_dev, uint64_t *out_dev, int64_t npoly, int64_t N, int64_t k,
                                int32_t device, void *stream)
{
    const pcmm_status rc = ring_args_ok(in_dev, out_dev, npoly, N, k, device);
    if (rc != PCMM_OK) return rc;
    return launch_transpose(in_dev, out_dev, npoly, N / k, k, device, (hipStream_t)stream);
}

pcmm_status pcmm_ring_compose(const uint64_t *in_dev, uint64_t *out_dev, int64_t npoly, int64_t N, int64_t k,
                              int32_t device, void *stream)
{
    const pcmm_status rc = ring_args_ok(in_dev, out_dev, npoly, N, k, device);
    if (rc != PCMM_OK) return rc;
    return launch_transpose(in_dev, out_dev, npoly, k, N / k, device, (hipStream_t)stream);
}

void pcmm_plan_destroy(pcmm_plan *plan)
{
    if (!plan) return;
    DevGuard dg(plan->device);
    if (plan->have_ev)
        for (int i = 0; i < 4; ++i) (void)hipEventDestroy(plan->ev[i]);
    if (plan->Wp) (void)hipFree(plan->Wp);
    if (plan->Ad) (void)hipFree(plan->Ad);
    if (plan->lc) (void)hipFree(plan->lc);
    delete plan;
}

}  // extern "C"
