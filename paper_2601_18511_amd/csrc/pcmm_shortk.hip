// PCMM for short contractions (K <= 128) on MI355X (gfx950): C_j = W . A_j mod q_j where W is tall and
// A_j is very wide -- the shape of the plaintext-ciphertext attention products of Section 4.2, whose
// contraction runs over the head dimension.  Such a product writes far more than it reads (24 GiB of
// residues for the 4096 x 128 by 128 x 131072 case with six limbs), so it is bound by the stores and by
// the vector-ALU work of the modular reduction, not by the matrix cores.
//
// Design.  A work-group of four waves owns a strip of 64 columns of one limb; wave w owns columns
// 16w .. 16w+15, reads their residues, cuts them into digits and keeps the digit fragments (both k-steps, all D
// digits: 2 D operand registers of 16 bytes) in registers for the whole kernel.  No digit plane goes through memory
// and no split kernel runs before this one (with one: 128 x 128 by 128 x 8192, two 36-bit limbs 17.5 us against 8.4;
// 300 x 100 by 100 x 131072, six 50-bit limbs 756 us against 511; 4096 x 128 by 128 x 131072, six limbs 6.27 ms
// against 6.12).
// The work-group then walks down the rows of W.  W is shared by the four waves, so it is staged through
// LDS, four 16-row blocks at a time, double-buffered: the global loads of stage s+2 are issued before
// the results of stage s+1 are stored.  Per 16 x 16 output block a wave issues 2 D S MFMAs into
// E = D+S-1 accumulators (ordinary vector registers here: the compiler tracks the MFMA hazards, and the
// epilogue reads them without accumulator-register moves), reduces them and stores the block.  The
// kernel fits 128 registers per lane for most digit counts, so four waves share a SIMD: while one reduces and stores its
// block, the others keep the matrix cores busy.  (A variant that kept two accumulator sets per wave and
// interleaved the reduction of one block with the MFMAs of the next, at two waves per SIMD, measured
// 6 % slower; a fifth wave per work-group that does nothing but the W loads, 15 % slower.)
// Measured on the 4096 x 128 by 128 x 131072 case: the chip is power-limited here (shader clock about
// 1.5 GHz with matrix cores, double-precision vector work and 4 TB/s of stores all active); the output
// stores alone, in this pattern or any other, take 4.6 ms of the 6.0 ms.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <algorithm>

#include "pcmm_device.hpp"
#include "pcmm_shortk.hpp"

using namespace pcmm_device;

namespace {

constexpr int RS = 4;   // 16-row blocks of W per LDS stage

struct KArgs {
    pcmm_shortk::Args a;
    int stages_per_part;  // LDS stages (RS row blocks each) per part
    pcmm_host::StripRaster raster;   // of 64-column strips
};

// MODE: the grouping reduce_f64 uses (0: groups of three accumulators; 2: groups of four, pairs joined in int32)
// ONCE: one work-group covers all rows of its strip, so every residue is read once: non-temporal loads (64 rows,
//       131072 columns, four limbs 152 -> 145 us).  With several parts the later ones find the residues in the caches;
//       non-temporal loads would keep them out (4096 x 128 by 128 x 8192: 74 -> 121 us).
// NT_STORES: shortk_nt_stores in pcmm_host.hpp says when and what both sides measured.
template <int D, int S, int MODE, bool ONCE, bool NT_STORES>
__global__ __launch_bounds__(256, D == 7 && S == 2 ? 3 : 4) void gemm_shortk_kernel(KArgs ka)
{
    constexpr int E = D + S - 1;
    constexpr int NF = RS * S * 2;                // W fragments per stage: [row block][slice][k-step]
    constexpr int STAGE = NF * kFrag;
    constexpr int NLD = NF / 4;                   // fragments each wave moves per stage (one 16-byte unit per lane)
    static_assert(NF % 4 == 0, "a stage is moved by four waves, whole fragments each");
    const pcmm_shortk::Args &a = ka.a;

    __shared__ __attribute__((aligned(16))) int8_t lds[2][STAGE];

    // which strip (strips side by side at a time against the parts of a strip next to each other: 8192 x 64 by 64 x 8192 132 ->
    // 101 us; 777 x 96 by 96 x 20001, four limbs 202 -> 183 us; equal where a strip has one part)
    int strip, mpart, limb;
    if (!strip_of(ka.raster, blockIdx.x, strip, mpart, limb)) return;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t loff = (uint32_t)lane * 16u;

    // ---- this wave's digit fragments, cut from the residues of its 16 columns: lane l holds column l % 16 and, of each
    // k-step, the values 16 (l / 16) .. 16 (l / 16) + 15 of k.  All sixteen loads of a k-step are in flight before the
    // first use; rows and columns beyond the matrix load its last one instead and count as zero.
    const int nb = strip * 4 + wave;
    const int64_t n = (int64_t)nb * 16 + (lane & 15);
    v4i b[2][D];
    {
        const uint64_t *src = a.A + (int64_t)limb * a.K * a.Ncols + min(n, a.Ncols - 1);
        const int k0 = (lane >> 4) * 16, klast = (int)a.K - 1;
        uint64_t x[2][16];
        auto load = [&](int kb) {
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const uint64_t *word = &src[(int64_t)min(kb * 64 + k0 + j, klast) * a.Ncols];
                x[kb][j] = ONCE ? __builtin_nontemporal_load(word) : *word;
            }
        };
        auto cut = [&](int kb) {
#pragma unroll
            for (int j = 0; j < 16; ++j)
                if (kb * 64 + k0 + j > klast || n >= a.Ncols) x[kb][j] = 0;
            digits16<D>(x[kb], b[kb]);
        };
        load(0);
        if constexpr (D < 6) load(1);
        cut(0);
        if constexpr (D >= 6) {              // both at once would not fit the 128 registers
            __builtin_amdgcn_sched_barrier(0);
            load(1);
        }
        cut(1);
        // The digits are final values here: without this the compiler carries parts of their making into the loop and
        // needs 132 registers for seven digits of two slices instead of 124 (three waves on a SIMD instead of four).
        if constexpr (MODE == 2) {
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int d = 0; d < D; ++d) asm volatile("" : "+v"(b[kb][d]));
        }
        __builtin_amdgcn_sched_barrier(0);   // the loads of W below stay below
    }

    // ---- W stages.  Fragment f = wave + 4 i of a stage is (row block f / (2S), slice (f / 2) % S, k-step f % 2)
    // and lies at byte f * 1024 of the stage in LDS.
    const uint32_t wp_bytes = (uint32_t)((int64_t)S * 2 * a.MB * kFrag);
    const __amdgpu_buffer_rsrc_t wrs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t *>(a.Wp), 0, wp_bytes, 0x00020000);
    const int mb_first = mpart * ka.stages_per_part * RS;
    const int mb_last = (int)a.MB - 1;
    v4i wst[NLD];
    auto stage_load = [&](int s) {           // stage s of this part: global -> registers
        const int mb0 = mb_first + s * RS;
#pragma unroll
        for (int i = 0; i < NLD; ++i) {
            const int f = wave + 4 * i;
            const int r = f / (2 * S), sl = (f / 2) % S, kb = f % 2;
            const int mb = min(mb0 + r, mb_last);   // blocks beyond the packed matrix are not stored: any data will do
            const uint32_t off = (uint32_t)((sl * 2 + kb) * (int)a.MB + mb) * (uint32_t)kFrag;
            wst[i] = (v4i)__builtin_amdgcn_raw_buffer_load_b128(wrs, loff, (int)off, 0);
        }
    };
    auto stage_store = [&](int buf) {        // registers -> LDS
#pragma unroll
        for (int i = 0; i < NLD; ++i)
            *reinterpret_cast<v4i *>(&lds[buf][(wave + 4 * i) * kFrag + lane * 16]) = wst[i];
    };

    // the limb's constants, in scalar registers
    LimbConst lc;
    {
        constexpr int LCW = sizeof(LimbConst) / 4;
        const uint32_t *src = reinterpret_cast<const uint32_t *>(a.lc + limb);
        uint32_t w[LCW];
#pragma unroll
        for (int i = 0; i < LCW; ++i) w[i] = __builtin_amdgcn_readfirstlane(src[i]);
        __builtin_memcpy(&lc, w, sizeof(lc));
    }

    uint64_t *Cl = a.C + (int64_t)limb * a.M * a.Ncols;
    const uint32_t c_rowbytes = (uint32_t)a.Ncols * 8u;
    // lanes whose column lies beyond Ncols get an offset that is out of range for every row
    const uint32_t c_lane = n < a.Ncols ? (uint32_t)((lane >> 4) * 4) * c_rowbytes + (uint32_t)n * 8u : 0x80000000u;

    // one 16 x 16 block: acc[e] = sum over slices, k-steps and digits with d + slice = e
    auto compute = [&](v4i (&acc)[E], int buf, int r) {
        v4i wf[S][2];
#pragma unroll
        for (int sl = 0; sl < S; ++sl)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
                wf[sl][kb] = *reinterpret_cast<const v4i *>(&lds[buf][((r * S + sl) * 2 + kb) * kFrag + lane * 16]);
        // consecutive MFMAs go to different accumulators; the first one of each starts from zero
#pragma unroll
        for (int sl = 0; sl < S; ++sl)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    const int e = d + sl;
                    const bool first = kb == 0 && (sl == 0 || d == D - 1);
                    acc[e] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wf[sl][kb], b[kb][d], first ? (v4i){0, 0, 0, 0} : acc[e], 0, 0, 0);
                }
    };
    // reduce and store one block.  Accumulator register r of lane l is output row 4*(l/16)+r, column l%16.
    // Rows at or beyond M fall outside the buffer descriptor and are dropped by its range check.
    auto emit = [&](const v4i (&acc)[E], int mb) {
        // no branch here: a block beyond M gets an empty descriptor, which drops its stores
        const int64_t m0 = min((int64_t)mb * 16, a.M);
        const uint32_t rows_valid = (uint32_t)min((int64_t)16, a.M - m0);
        const __amdgpu_buffer_rsrc_t crs =
            __builtin_amdgcn_make_buffer_rsrc(Cl + m0 * a.Ncols, 0, rows_valid * c_rowbytes, 0x00020000);
        int avs[4][E];
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int e = 0; e < E; ++e) avs[r][e] = acc[e][r];
        uint64_t res[4];
        reduce_f64<E, MODE, 4>(avs, lc.qd, lc.invq, res);
#pragma unroll
        for (int r = 0; r < 4; ++r)
            __builtin_amdgcn_raw_buffer_store_b64((v2u){(uint32_t)res[r], (uint32_t)(res[r] >> 32)}, crs,
                                                  c_lane + (uint32_t)r * c_rowbytes, 0, NT_STORES ? 2 : 0);
    };

    // ---- stage s is in LDS[s & 1] while stage s+1 travels global -> registers
    const int nst = ka.stages_per_part;
    v4i acc[E];
    stage_load(0);
    stage_store(0);
    __syncthreads();
    if (nst > 1) stage_load(1);
    for (int s = 0; s < nst; ++s) {
        const int cur = s & 1;
        const int mb0 = mb_first + s * RS;
#pragma unroll
        for (int r = 0; r < RS; ++r) {
            compute(acc, cur, r);
            emit(acc, mb0 + r);
        }
        if (s + 1 < nst) {
            stage_store(cur ^ 1);            // every wave has left that buffer (barrier of stage s-1)
            __syncthreads();
            if (s + 2 < nst) stage_load(s + 2);
        }
    }
}

template <int D, int S, int MODE>
void launch_mode(const KArgs &ka, int64_t grid, hipStream_t st)
{
    const dim3 g((unsigned)grid), b(256);
    const bool once = ka.raster.mparts == 1;
    const bool nt = pcmm_host::shortk_nt_stores(ka.a.Ncols, (uint64_t)(uintptr_t)ka.a.C, (int64_t)ka.a.L * ka.a.M * ka.a.Ncols * 8,
                                                (int64_t)ka.a.L * ka.raster.nstrips, ka.raster.mparts);
    const auto kern = once ? (nt ? gemm_shortk_kernel<D, S, MODE, true, true> : gemm_shortk_kernel<D, S, MODE, true, false>)
                           : (nt ? gemm_shortk_kernel<D, S, MODE, false, true> : gemm_shortk_kernel<D, S, MODE, false, false>);
    hipLaunchKernelGGL(kern, g, b, 0, st, ka);
}

template <int D, int S>
hipError_t launch_ds(const KArgs &ka, int epi, int64_t grid, hipStream_t st)
{
    constexpr int E = D + S - 1;
    if (epi == EPI_F64) {
        launch_mode<D, S, 0>(ka, grid, st);
    } else if (epi == EPI_F64_G4P) {
        if constexpr (E >= 7) launch_mode<D, S, 2>(ka, grid, st);
        else return hipErrorInvalidValue;
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

namespace pcmm_shortk {

bool covers(int D, int S, int epi, int64_t nkb)
{
    return nkb == 2 && D >= 4 && D <= 7 && (S == 1 || S == 2) && (epi == EPI_F64 || epi == EPI_F64_G4P);
}

hipError_t launch(const Args &a, int D, int S, int epi, hipStream_t st)
{
    if (!covers(D, S, epi, 2)) return hipErrorInvalidValue;
    KArgs ka;
    ka.a = a;
    const int64_t nstrips = (a.Ncols + 63) / 64;
    const int64_t stages = ((a.M + 15) / 16 + RS - 1) / RS;        // stages that hold a row of W
    // Enough work-groups to balance the 1024 resident ones, as few as possible otherwise: every part of a strip reads
    // and cuts the strip's residues again.  Up to 512 strips, where that repeats most, 1536 work-groups, else 3072.
    // Measured with 1536 / 3072 / 6144: 128 strips (4096 x 128 by 128 x 8192) 56 / 69 / 82 us; 256 strips (1024 x 128
    // by 128 x 8192, two limbs) 36 / 41 / 60 us; 626 strips (4096 x 128 by 128 x 20000, two limbs) 273 / 261 / 277 us;
    // 2048 strips (1000 x 80 by 80 x 65536, two limbs) 249 / 210 / 223 us.  With the present raster, over 160 shapes, against these
    // targets: 768 work-groups 0.99 to 1.05 of the time by the number of strips, 1536 0.99 to 1.04, 3072 0.99 to 1.02, 6144 1.01 to 1.06.
    const int64_t strips = (int64_t)a.L * nstrips;
    const int64_t target = strips <= 512 ? 1536 : 3072;
    const int64_t mparts = std::min<int64_t>(stages, std::max<int64_t>(1, (target + strips - 1) / strips));
    ka.stages_per_part = (int)((stages + mparts - 1) / mparts);
    const int64_t slots = D == 7 && S == 2 ? 96 : 128;            // of an XCD: three or four waves on a SIMD
    ka.raster = pcmm_host::strip_raster(a.L, nstrips, (stages + ka.stages_per_part - 1) / ka.stages_per_part,
                                        pcmm_host::whole_strips(a.M, a.K, a.Ncols, a.L, S), slots);
    const int64_t grid = ka.raster.grid;
    if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
#define PCMM_SHORTK_CASE(DD, SS) \
    if (D == DD && S == SS) return launch_ds<DD, SS>(ka, epi, grid, st);
    PCMM_SHORTK_CASE(4, 1)
    PCMM_SHORTK_CASE(5, 1)
    PCMM_SHORTK_CASE(6, 1)
    PCMM_SHORTK_CASE(7, 1)
    PCMM_SHORTK_CASE(4, 2)
    PCMM_SHORTK_CASE(5, 2)
    PCMM_SHORTK_CASE(6, 2)
    PCMM_SHORTK_CASE(7, 2)
#undef PCMM_SHORTK_CASE
    return hipErrorInvalidValue;
}

}  // namespace pcmm_shortk
