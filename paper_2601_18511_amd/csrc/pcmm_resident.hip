// PCMM for contractions whose digits fit LDS (at most 64 floor(160 / D) values of k, 1280 for eight digits to 2560 for
// four, where pcmm_shortk.hip does not run and an estimate says that this is the faster way) on MI355X (gfx950): C_j = W . A_j mod q_j.
//
// Design.  A work-group owns a strip of 16 NT columns of one limb.  It reads the strip's residues, cuts them into
// balanced digits and keeps the MFMA operand fragments of ALL k-steps in LDS (NT D KiB a k-step); then its waves walk down the
// rows of W, each wave by itself, MT 16-row blocks at a time: W fragments come from L2 straight into registers up to three
// k-steps ahead, digit fragments from LDS one 16-column part ahead.  Against the digit split and the GEMM kernel of pcmm.hip no
// digit plane goes through memory (5 to 8 bytes a residue written once and read once per 256 rows), one launch goes, and
// there is no barrier after the digits are cut: waves drift apart, so that one wave's reduction and stores run beside the
// MFMAs of the other wave of its SIMD.
//
// Tile.  A k-step of a wave takes MT S fragments of W through the vector L1 (64 bytes a clock) and NT D digit fragments from
// LDS (128 bytes a clock) for MT NT D S MFMAs of 16 clocks; accumulators (E a block), two to four sets of W fragments and one of
// digits have to fit 256 registers, so that two waves share a SIMD.  Two column fragments for up to six accumulators (W
// traffic counts most), one beyond.  Accumulators are ordinary registers written by the MFMA builtin: the epilogue needs no
// moves, and the first k-step starts them from an inline zero (144 moves a row group otherwise, 4 to 8 % at 13 k-steps).
//
// Measured (whole pcmm_run in rows of calls, split and GEMM kernel -> this one): 1000 x 777 by 777 x 12300, three 45-bit limbs
// 328 -> 215 us (on other buffers each call 315 -> 230); 1000 x 300 by 300 x 8192, four 36-bit limbs 116 -> 72; 4096 x 1024 by
// 1024 x 16384, four 36-bit limbs 1360 -> 1160; 128 x 384 by 384 x 4096, two 36-bit limbs 21 -> 8.  Of the first one the stores' bytes and residues take
// 97 us at 5.5 TB/s and the MFMAs 94 us; what is left is the cutting at the start of a work-group, during which its waves run no
// MFMAs, and the last, partial round of work-groups.  What the stores cost beside the MFMAs decides more than either: cached
// ones of whole lines take 234 us where non-temporal ones take 202 (12288 columns).
// Built, measured and dropped: W fragments one k-step ahead only (three: 5 % faster); non-temporal loads of
// the residues (4 to 10 % slower: neighbouring strips share lines and parts of a strip re-read them); digits kept in
// registers across the epilogue (spills, and 10 to 40 % slower).
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <algorithm>
#include <type_traits>

#include "pcmm_device.hpp"
#include "pcmm_resident.hpp"

using namespace pcmm_device;

namespace {

using pcmm_host::ResidentTile;

struct KArgs {
    pcmm_resident::Args a;
    int ksteps;           // k-steps of 64 that are cut and contracted
    int groups;           // groups of MT row blocks in all
    int groups_per_part;
    pcmm_host::StripRaster raster;
};

template <int D, int S, int NT, int MT, int EPI, bool NT_STORES>
__global__ __launch_bounds__(512, 2) void gemm_resident_kernel(KArgs ka)
{
    constexpr int E = D + S - 1;
    constexpr int NW = S * MT;                        // W fragments per k-step
    constexpr int PF = pcmm_host::resident_ahead(D, S, NT, MT), U = PF + 1;
    const pcmm_resident::Args &a = ka.a;
    extern __shared__ __attribute__((aligned(16))) int8_t dig[];   // [k-step][NT][D][lane][16]

    int strip, mpart, limb;
    if (!strip_of(ka.raster, blockIdx.x, strip, mpart, limb)) return;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nw = blockDim.x >> 6;
    const int nks = ka.ksteps;
    const int64_t n0 = (int64_t)strip * (16 * NT);
    const uint32_t rowbytes = (uint32_t)a.Ncols * 8u;

    // ---- digits of the strip.  One unit of work is one k-step of 16 columns: lane l holds column l % 16 and the values
    // 16 (l / 16) .. + 15 of k.  The loads go through a descriptor of the k-step's rows: rows beyond K and (by their
    // offset) columns beyond Ncols read as 0, whose digits are 0.
    {
        auto load = [&](uint64_t (&x)[16], int u) {
            const int kb = u / NT, nt = u % NT;
            const int64_t n = n0 + nt * 16 + (lane & 15);
            const uint32_t rows = (uint32_t)pcmm_host::resident_rows(a.K, kb);   // 0: a k-step of padding
            const uint32_t off = n < a.Ncols ? (uint32_t)((lane >> 4) * 16) * rowbytes + (uint32_t)n * 8u : 0x80000000u;
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<uint64_t *>(a.A + ((int64_t)limb * a.K + (int64_t)kb * 64) * a.Ncols), 0, rows * rowbytes, 0x00020000);
            auto word = [&](int j, uint32_t lane_off, uint32_t uniform_off) {
                const v2u w = (v2u)__builtin_amdgcn_raw_buffer_load_b64(rs, lane_off, (int)uniform_off, 0);
                x[j] = (uint64_t)w[0] | ((uint64_t)w[1] << 32);
            };
            // The range check counts the lane's offset; whether it counts the uniform one too is not the same in all documents.
            // So that one stays inside the descriptor, and a last k-step with fewer rows has its row offsets in the lanes.
            if (rows == 64) {
#pragma unroll
                for (int j = 0; j < 16; ++j) word(j, off, (uint32_t)j * rowbytes);
            } else {
#pragma unroll
                for (int j = 0; j < 16; ++j) word(j, off + (uint32_t)j * rowbytes, 0);
            }
        };
        auto cut = [&](const uint64_t (&x)[16], int u) {
            v4i out[D];
            digits16<D>(x, out);
#pragma unroll
            for (int d = 0; d < D; ++d) *reinterpret_cast<v4i *>(&dig[(u * D + d) * kFrag + lane * 16]) = out[d];
        };
        const int nu = nks * NT;
        uint64_t x0[16], x1[16];
        if (wave < nu) load(x0, wave);
        for (int u = wave; u < nu; u += 2 * nw) {
            if (u + nw < nu) load(x1, u + nw);
            cut(x0, u);
            if (u + nw < nu) {
                if (u + 2 * nw < nu) load(x0, u + 2 * nw);
                cut(x1, u + nw);
            }
        }
    }
    __syncthreads();

    const int g_end = min(ka.groups_per_part, ka.groups - mpart * ka.groups_per_part);
    int g = wave;
    if (g >= g_end) return;

    // ---- W: one descriptor per slice, a scalar byte offset for row group and k-step.  A group's blocks beyond MB read the next
    // k-step's first ones, behind the last k-step the slack of the packed array (pcmm_host::kWpSlack): their rows are dropped below.
    const uint32_t slice_bytes = (uint32_t)(a.nkb * a.MB * kFrag);
    const uint32_t kstride = (uint32_t)a.MB * (uint32_t)kFrag;
    const uint32_t loff = (uint32_t)lane * 16u;
    __amdgpu_buffer_rsrc_t wrs[S];
#pragma unroll
    for (int sl = 0; sl < S; ++sl)
        wrs[sl] = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t *>(a.Wp + (int64_t)sl * slice_bytes), 0, slice_bytes, 0x00020000);
    auto first_offset = [&](int gg) { return (uint32_t)((mpart * ka.groups_per_part + gg) * MT) * (uint32_t)kFrag; };

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

    v4i wreg[U][S][MT];
    v4i b[D];
    v4i acc[MT][NT][E];
    uint32_t woff = first_offset(g);
    static_for<PF>([&](auto kc) {                     // at least PF k-steps
        constexpr int k = decltype(kc)::value;
#pragma unroll
        for (int f = 0; f < NW; ++f)
            wreg[k][f / MT][f % MT] =
                (v4i)__builtin_amdgcn_raw_buffer_load_b128(wrs[f / MT], loff, (int)(woff + k * kstride + (f % MT) * kFrag), 0);
    });

    // One k-step in NT parts of 16 columns.  wnext.x: byte offset of the W fragments to request (a later k-step's, or one of the
    // next row group); wnext.y: 0, or an offset out of range for every lane where there is no next group (nothing is fetched).
    auto step = [&](auto phase, auto first, int kb, uint2 wnext) {
        constexpr int CUR = decltype(phase)::value, NXT = (CUR + PF) % U;
        constexpr bool FIRST = decltype(first)::value;
        constexpr int CNT = D * NW * NT;              // MFMAs
        const int kb_next = kb + 1 < nks ? kb + 1 : 0;
        static_for<NT>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            const int8_t *next = &dig[(j + 1 < NT ? kb * NT + j + 1 : kb_next * NT) * (D * kFrag) + lane * 16];
            static_for<D>([&](auto dc) {
                constexpr int d = decltype(dc)::value;
                static_for<NW>([&](auto fc) {
                    constexpr int m = (j * D + d) * NW + decltype(fc)::value;
                    constexpr int n_lo = (m * NW + CNT - 1) / CNT, n_hi = ((m + 1) * NW + CNT - 1) / CNT;
                    static_for<n_hi - n_lo>([&](auto oc) {
                        constexpr int n = n_lo + decltype(oc)::value;
                        wreg[NXT][n / MT][n % MT] =
                            (v4i)__builtin_amdgcn_raw_buffer_load_b128(wrs[n / MT], loff + wnext.y, (int)(wnext.x + (n % MT) * kFrag), 0);
                    });
                    // W fragments forwards for one digit and backwards for the next: consecutive MFMAs share an operand
                    constexpr int f = ((j * D + d) & 1) ? NW - 1 - decltype(fc)::value : decltype(fc)::value;
                    constexpr int ws = f / MT, wi = f % MT;
                    constexpr bool zero = FIRST && (S == 1 || ws == 1 || d == 0);   // the first product of its accumulator
                    acc[wi][j][d + ws] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wreg[CUR][ws][wi], b[d],
                                                                              zero ? (v4i){0, 0, 0, 0} : acc[wi][j][d + ws], 0, 0, 0);
                });
                b[d] = *reinterpret_cast<const v4i *>(next + d * kFrag);
                __builtin_amdgcn_sched_barrier(0);
            });
        });
    };
    for (;;) {
        const int g_next = g + nw;
        const uint32_t wfirst = first_offset(g_next < g_end ? g_next : g);
        const uint32_t none = g_next < g_end ? 0u : 0x80000000u;      // a slice is smaller
        auto wahead = [&](int kb) {                   // the k-step PF after kb, perhaps of the next group
            const int k = kb + PF;
            return k < nks ? make_uint2(woff + (uint32_t)k * kstride, 0u) : make_uint2(wfirst + (uint32_t)(k - nks) * kstride, none);
        };
#pragma unroll
        for (int d = 0; d < D; ++d) b[d] = *reinterpret_cast<const v4i *>(&dig[d * kFrag + lane * 16]);
        // k-step kb runs in phase kb % U; the first one starts the accumulators
        step(std::integral_constant<int, 0>{}, std::true_type{}, 0, wahead(0));
        int kb = 1;
        for (; kb + U <= nks; kb += U)
            static_for<U>([&](auto uc) {
                constexpr int u = decltype(uc)::value;
                step(std::integral_constant<int, (u + 1) % U>{}, std::false_type{}, kb + u, wahead(kb + u));
            });
        static_for<U - 1>([&](auto uc) {
            constexpr int u = decltype(uc)::value;
            if (kb + u < nks) step(std::integral_constant<int, (u + 1) % U>{}, std::false_type{}, kb + u, wahead(kb + u));
        });
        const int rest = (nks - kb + 1) % U;
        static_for<U - 1>([&](auto rc) {              // the next group starts with register set 0 again
            constexpr int r = decltype(rc)::value + 1;
            if (rest == r) {
                v4i tmp[PF][S][MT];
#pragma unroll
                for (int i = 0; i < PF; ++i)
#pragma unroll
                    for (int f = 0; f < NW; ++f) tmp[i][f / MT][f % MT] = wreg[(i + r) % U][f / MT][f % MT];
#pragma unroll
                for (int i = 0; i < PF; ++i)
#pragma unroll
                    for (int f = 0; f < NW; ++f) wreg[i][f / MT][f % MT] = tmp[i][f / MT][f % MT];
            }
        });
        // The next W fragments have to be here before the first store is issued: a wait for them behind the stores would,
        // the counter being in order, wait for those to complete.
#pragma unroll
        for (int f = 0; f < PF * NW; ++f) asm volatile("" : "+v"(wreg[f / NW][f % NW / MT][f % MT]));
        __builtin_amdgcn_sched_barrier(0);

        // ---- epilogue: accumulator register r of lane l is output row 4 (l / 16) + r, column l % 16 of its 16 x 16 block
        const int mb0 = (mpart * ka.groups_per_part + g) * MT;
        static_for<MT * NT>([&](auto ijc) {
            constexpr int i = decltype(ijc)::value / NT, j = decltype(ijc)::value % NT;
            // rows at or beyond M and columns at or beyond Ncols are dropped by the range check
            const int64_t m0 = min((int64_t)(mb0 + i) * 16, a.M);
            const uint32_t rows_valid = (uint32_t)min((int64_t)16, a.M - m0);
            const int64_t n = n0 + j * 16 + (lane & 15);
            const uint32_t c_lane = n < a.Ncols ? (uint32_t)((lane >> 4) * 4) * rowbytes + (uint32_t)n * 8u : 0x80000000u;
            int avs[4][E];
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int e = 0; e < E; ++e) avs[r][e] = acc[i][j][e][r];
            uint64_t res[4];
            if constexpr (EPI == EPI_F64) reduce_f64<E, 0, 4>(avs, lc.qd, lc.invq, res);
            else if constexpr (EPI == EPI_F64_G4) reduce_f64<E, 1, 4>(avs, lc.qd, lc.invq, res);
            else reduce_int<E, 4>(avs, lc, res);
            const __amdgpu_buffer_rsrc_t crs =
                __builtin_amdgcn_make_buffer_rsrc(Cl + m0 * a.Ncols, 0, rows_valid * rowbytes, 0x00020000);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                __builtin_amdgcn_raw_buffer_store_b64((v2u){(uint32_t)res[r], (uint32_t)(res[r] >> 32)}, crs,
                                                      c_lane + (uint32_t)r * rowbytes, 0, NT_STORES ? 2 : 0);
            __builtin_amdgcn_sched_barrier(0);
        });
        if (g_next >= g_end) break;
        g = g_next;
        woff = wfirst;
    }
}

template <int D, int S, int NT, int EPI>
hipError_t launch_tile(const KArgs &ka, const ResidentTile &tile, hipStream_t st)
{
    constexpr int MT = pcmm_host::resident_mt(D, S, NT);
    // the pipeline holds the W fragments of resident_ahead k-steps of one row group
    if (tile.MT != MT || ka.ksteps < pcmm_host::resident_ahead(D, S, NT, MT)) return hipErrorInvalidValue;
    const int64_t lds = (int64_t)ka.ksteps * NT * D * kFrag;
    if (lds > pcmm_host::kLdsBytes) return hipErrorInvalidValue;
    const bool nt = pcmm_host::resident_nt_stores(ka.a.K, ka.a.Ncols, (uint64_t)(uintptr_t)ka.a.C, D, S);
    const auto kern = nt ? gemm_resident_kernel<D, S, NT, MT, EPI, true> : gemm_resident_kernel<D, S, NT, MT, EPI, false>;
    const dim3 g((unsigned)ka.raster.grid), b((unsigned)(tile.waves * 64));
    hipLaunchKernelGGL(kern, g, b, (size_t)lds, st, ka);
    return hipGetLastError();
}

}  // namespace

namespace pcmm_resident {

hipError_t launch(const Args &a, const ResidentTile &tile, int D, int S, int epi, hipStream_t st)
{
    KArgs ka;
    ka.a = a;
    ka.ksteps = (int)pcmm_host::resident_ksteps(a.K);
    ka.groups = (int)((a.M + 16 * tile.MT - 1) / (16 * tile.MT));
    ka.groups_per_part = tile.groups_per_part;
    ka.raster = pcmm_host::strip_raster(a.L, (a.Ncols + 16 * tile.NT - 1) / (16 * tile.NT),
                                        (ka.groups + ka.groups_per_part - 1) / ka.groups_per_part, pcmm_host::whole_strips(a.M, a.K, a.Ncols, a.L, S),
                                        tile.waves == 4 ? 64 : 32);
    if (ka.ksteps > a.nkb || ka.raster.grid > 0x7fffffffLL) return hipErrorInvalidValue;
#define PCMM_RESIDENT_CASE(DD, SS, NN, EE) \
    if (D == DD && S == SS && tile.NT == NN && (epi == EE || (EE == EPI_F64_G4 && epi == EPI_F64_G4P))) \
        return launch_tile<DD, SS, NN, EE>(ka, tile, st);
    PCMM_RESIDENT_CASE(4, 1, 1, EPI_F64)
    PCMM_RESIDENT_CASE(5, 1, 1, EPI_F64)
    PCMM_RESIDENT_CASE(6, 1, 1, EPI_F64)
    PCMM_RESIDENT_CASE(7, 1, 1, EPI_F64_G4)
    PCMM_RESIDENT_CASE(7, 1, 1, EPI_INT)
    PCMM_RESIDENT_CASE(8, 1, 1, EPI_INT)
    PCMM_RESIDENT_CASE(4, 2, 1, EPI_F64)
    PCMM_RESIDENT_CASE(5, 2, 1, EPI_F64)
    PCMM_RESIDENT_CASE(6, 2, 1, EPI_F64_G4)
    PCMM_RESIDENT_CASE(7, 2, 1, EPI_F64_G4)
    PCMM_RESIDENT_CASE(7, 2, 1, EPI_INT)
    PCMM_RESIDENT_CASE(8, 2, 1, EPI_INT)
    PCMM_RESIDENT_CASE(4, 1, 2, EPI_F64)
    PCMM_RESIDENT_CASE(5, 1, 2, EPI_F64)
    PCMM_RESIDENT_CASE(6, 1, 2, EPI_F64)
    PCMM_RESIDENT_CASE(4, 2, 2, EPI_F64)
    PCMM_RESIDENT_CASE(5, 2, 2, EPI_F64)
#undef PCMM_RESIDENT_CASE
    return hipErrorInvalidValue;
}

}  // namespace pcmm_resident
