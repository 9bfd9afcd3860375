// Host-side planning of the PCMM library: argument validation, the digit count, the tile geometry, the
// sizes of the plan's buffers and the per-limb constants of the epilogue.  Plain C++ with no HIP in it,
// so that it can be compiled and run on its own under the host sanitizers; pcmm.hip includes it and
// owns everything that touches the device.
//
// The operation planned is C_j = W . A_j mod q_j for every RNS limb j (the clear matrix product that
// the paper's linear-layer PCMM reduces to, Sections 2.2 and 5.1); the weights are converted once per
// matrix (the paper's "model conversion", Section 5.3).
#ifndef PCMM_HOST_HPP
#define PCMM_HOST_HPP

#include <stddef.h>
#include <stdint.h>

#include "../../include/pcmm.h"

namespace pcmm_host {

typedef unsigned __int128 u128;

constexpr int kFragBytes = 1024;   // one 16 x 64 int8 MFMA operand fragment
constexpr int kMaxLimbs = 64;

// Per-limb constants of the epilogue.
struct LimbConst {
    uint64_t q;      // the prime
    uint64_t mu;     // floor(2^64 / q)
    uint64_t off;    // q * floor(2^62 / q) >= 2^61: added to a signed part of magnitude < 2^56 to make it positive
    uint64_t c32;    // 2^32 mod q
    uint64_t c32s;   // floor(c32 * 2^64 / q)  (Shoup companion of c32)
    uint64_t c64;    // 2^64 mod q
    uint64_t c64s;   // floor(c64 * 2^64 / q)
    double qd;       // q as a double (exact for q < 2^53)
    double invq;     // 1.0 / q, rounded to nearest
};

namespace epi {
// How the epilogue reduces sum_e acc_e 256^e modulo q.
enum Epi : int {
    EPI_F64 = 0,     // q < 2^50: exact double-precision arithmetic (fma remainders), no 64-bit multiplies
    EPI_INT = 2,     // any q < 2^62: one 64-bit Barrett per four accumulators, joined by Shoup
                     // multiplications by 2^32 and 2^64
    EPI_F64_G4 = 3,  // as EPI_F64 with the accumulators grouped in fours: |acc| < 2^28, 7 or 8 accumulators
    EPI_F64_PAIR = 5,  // EPI_F64 for two limbs at once (the digits are those of a limb pair)
    EPI_F64_G4P = 4  // as EPI_F64_G4 with pairs of accumulators first joined in int32: 257 |acc| < 2^31
};
}  // namespace epi

inline LimbConst limb_const(uint64_t q)
{
    LimbConst c;
    c.q = q;
    c.mu = (uint64_t)((((u128)1) << 64) / q);
    c.off = q * (uint64_t)((((u128)1) << 62) / q);
    c.c32 = (uint64_t)((((u128)1) << 32) % q);
    c.c32s = (uint64_t)(((u128)c.c32 << 64) / q);
    c.c64 = (uint64_t)((((u128)1) << 64) % q);
    c.c64s = (uint64_t)(((u128)c.c64 << 64) / q);
    c.qd = (double)q;
    c.invq = 1.0 / (double)q;
    return c;
}

// Two limbs whose digits are split jointly: x1 mod q1 and x2 mod q2 become
//   Y = q1 t + x1 + (Bias mod q1),  t = ((x2 - x1) q1^-1 + s) mod q2,  s = floor(Bias / q1) mod q2,
// the balanced digits of the integer X = Y - Bias with X = x1 mod q1, X = x2 mod q2 (Bias = sum_{i<9} 128 * 256^i).
constexpr int kPairDigits = 9;
struct PairConst {
    uint64_t q1;
    uint64_t bias_mod_q1;
    double q2, invq2, half_invq2;   // q2, 1/q2 and 1/(2 q2)
    double inv;                     // q1^-1 mod q2, balanced (magnitude <= q2/2)
    double s;
};

inline u128 pair_bias()
{
    u128 bias = 0;
    for (int i = 0; i < kPairDigits; ++i) bias |= (u128)0x80 << (8 * i);
    return bias;
}

// Whether two limbs of five digits each can share nine: coprime, of one size (q1 < 2 q2, which the split kernel's arithmetic
// needs, and q2 < 2 q1; the limbs of a plan always are), Y < q1 q2 + q1 <= 256^9, below 2^36 (the kernel takes th = t >> 32
// as four bits).  The limbs of a plan take five digits from 31-bit primes above 0x7F7F7F80 on.
inline bool pair_ok(uint64_t q1, uint64_t q2)
{
    const uint64_t hi = (uint64_t)1 << 36;
    if (q1 >= hi || q2 >= hi || q1 >= 2 * q2 || q2 >= 2 * q1) return false;
    uint64_t a = q1, b = q2;
    while (b) { const uint64_t r = a % b; a = b; b = r; }
    return a == 1 && (u128)q1 * q2 + q1 <= ((u128)1 << (8 * kPairDigits));
}

inline PairConst pair_const(uint64_t q1, uint64_t q2)
{
    PairConst c;
    c.q1 = q1;
    c.bias_mod_q1 = (uint64_t)(pair_bias() % q1);
    c.q2 = (double)q2;
    c.invq2 = 1.0 / (double)q2;
    c.half_invq2 = 0.5 * c.invq2;
    // extended Euclid: r0 = u0 q1 (mod q2)
    int64_t r0 = (int64_t)(q1 % q2), r1 = (int64_t)q2, u0 = 1, u1 = 0;
    while (r1) {
        const int64_t k = r0 / r1, r = r0 - k * r1, u = u0 - k * u1;
        r0 = r1; r1 = r; u0 = u1; u1 = u;
    }
    u0 %= (int64_t)q2;
    if (u0 > (int64_t)(q2 / 2)) u0 -= (int64_t)q2;
    if (u0 < -(int64_t)(q2 / 2)) u0 += (int64_t)q2;
    c.inv = (double)u0;
    c.s = (double)(uint64_t)((pair_bias() / q1) % q2);
    return c;
}

// Smallest D with (qmax - 1) + Bias_D < 256^D, Bias_D = sum_{i<D} 128 * 256^i: the number of signed
// base-256 digits that represent every residue below qmax.  0 if more than 8 would be needed.
inline int balanced_digits(uint64_t qmax)
{
    for (int d = 1; d <= 8; ++d) {
        u128 bias = 0;
        for (int i = 0; i < d; ++i) bias |= (u128)0x80 << (8 * i);
        if ((u128)(qmax - 1) + bias < ((u128)1 << (8 * d))) return d;
    }
    return 0;
}

// Accumulator footprint limits the tile: MT*NT*E*4 accumulator registers per lane (NT = 2), at most 160.
constexpr int tile_mt(int E) { return E <= 5 ? 4 : (E == 6 ? 3 : 2); }

// Whether the GEMM kernel contracts odd numbers of k-steps.  Not with eight W fragments per k-step (four digits, two
// slices): the second entry into the loop costs its two-wave kernel more than the k-step of zeros it saves (128 x 4096 by
// 4096 x 16384, two 30-bit limbs 423 -> 433 us, an even count; 2000 x 160 by 160 x 16384, four limbs 400 us either way).
constexpr bool odd_ksteps(int S, int MT) { return S * MT < 8; }

// Whether the short-contraction kernel stores C non-temporally: row pitch and address of C, its size, the strips of 64 columns
// over all limbs and the parts each strip is cut into.
// Rows that start on 128-byte lines: always; every store writes whole lines.  Rows that start inside a line at any other place
// than its middle: never; lines are joined in L2, which non-temporal stores prevent (9483 x 128 by 128 x 14636, five 44-bit
// limbs: cached 1.91 ms, non-temporal 2.62).  Rows that start on half lines: cached stores are better while the memory-side
// cache still joins the halves, non-temporal ones beyond (cached -> non-temporal: 300 x 64 by 64 x 42936, two limbs, 197 MiB
// 61 -> 69 us; 768 x 128 by 128 x 14632, five limbs, 429 MiB 187 -> 115; 3000 x 80 by 80 x 42936, two limbs, 1.9 GiB 670 ->
// 534).  Where that is depends on the parts: strips of two cross over at about 224 MiB (194 MiB 95 -> 79, 203 MiB
// 113 -> 122, 283 MiB 114 -> 71), others above 768 strips at about 400 (294 MiB 79 -> 79, 382 MiB 101 -> 114, 438 MiB
// 211 -> 152), fewer strips at about 640 (327 MiB 82 -> 89, 569 MiB 153 -> 161, 695 MiB 205 -> 183).  Over 230 shapes of 192 MiB to
// 2 GiB: 9 % faster than cached stores throughout, 3 % than non-temporal ones, 1 % behind the better of the two each time.  (Measured
// before strip_raster; with it, over 96 shapes of 150 MiB to 1.2 GiB, 2 % behind, at most 13 % but for one shape, 768 x 128 by 128 x
// 13656, five limbs, 400 MiB, 166 us cached and 108 non-temporal, and nowhere more than 6 % slower than before it.)
inline bool shortk_nt_stores(int64_t Ncols, uint64_t c_address, int64_t c_bytes, int64_t strips, int64_t parts)
{
    if (Ncols % 16 == 0) return true;
    if (Ncols % 8 != 0 || c_address % 64 != 0) return false;
    const int64_t from_mib = parts == 2 ? 224 : strips > 768 ? 416 : 640;
    return c_bytes > from_mib << 20;
}

// What of the digit split goes past the caches: nothing, the digits, or the residues too.  Both where they exceed the 256 MiB
// last-level cache by enough that nothing of them is found there again (split alone, cached -> non-temporal: 4096 x 4096 by
// 4096 x 32768, four 36-bit limbs 1.25 -> 1.16 ms; 14336 values of k, three limbs 3.28 -> 3.06).  Whole pcmm_run over 96 shapes of 199 to
// 640 MiB of residues, against cached: from 429 MiB on 0.90 to 1.01 with aligned rows (both) and 0.91 to 1.00 with others (digits only,
// since neighbouring work-groups share lines of residues; both 0.96 to 1.00); at 299 to 384 MiB 0.93 to 0.99 and 0.93 to 1.00; at
// 199 MiB 0.98 to 1.06 and 0.99 to 1.07; 78 MiB 46 -> 64 us.  The line is on the safe side of where the two are equal.
enum SplitNt : int { kNtNone = 0, kNtStores = 1, kNtBoth = 2 };
inline SplitNt split_nt(int64_t L, int64_t K, int64_t Ncols, uint64_t a_address)
{
    if (8 * L * K * Ncols <= (int64_t)384 << 20) return kNtNone;
    return ((uint64_t)Ncols * 8 | a_address) % 128 == 0 ? kNtBoth : kNtStores;
}

// Whether the GEMM kernel stores C non-temporally: rows on half lines, and a W of more than 48 MiB (both slices of int16 W), which every group
// of n-tiles reads again and cached stores push out of the last-level cache (GEMM alone, cached -> non-temporal, 36-bit limbs: 14336 x 4096 by
// 4096 x 16384, two limbs 6.60 -> 6.37 ms; 12296 columns 5.13 -> 4.82; 28672 x 2500 by 2500 x 8192 4.65 -> 4.21; W of 39 MiB,
// 10000 x 4096 4.47 -> 4.51, of 16 MiB, 4096 x 4096 7.63 -> 7.73; odd rows 1000 x 3000 by 3000 x 12301 320 -> 345 us; at 56 MiB
// 10874 x 2700 by 2700 x 4104, int16 W, seven digits 1176 -> 1175 us, 7168 x 4096 by 4096 x 4096, int16 W, integer epilogue
// 1342 -> 1324, 14336 x 4096 by 4096 x 4096, int8 W, integer epilogue 1645 -> 1648, a limb pair 7168 x 8192 by 8192 x 2048 836 -> 820).
// With 8192 columns or fewer they are 1 to 4 % faster from 16 MiB of W on too; the line is where they also are with 32768.
inline bool gemm_nt_stores(int64_t M, int64_t K, int S, int64_t Ncols, uint64_t c_address)
{
    return ((uint64_t)Ncols * 8 | c_address) % 64 == 0 && M * K * S > (int64_t)48 << 20;
}

// Raster of the kernels that give strips of columns to work-groups and may cut the rows into parts: work-group b runs on XCD b % 8.
// Whole strips: each XCD takes an eighth of the strips (counted over all limbs) and all their parts, strips fastest, so that the parts of a
// strip find its residues in their XCD's L2.  Runs: all (part, strip) pairs, strips fastest, cut into eight runs, so that the work-groups
// resident together store to the same rows side by side, but the residues of a limb are read by each of the 8 / L XCDs that its run spans.
// Whole strips where those further reads are at least a fifth of the stores, K (8 - L) / L > M / 5 (over 1500 shapes of at most 128 values of k
// and 1466 longer ones whose rows are cut, whole strips against runs: up to 0.2 the same on average and up to 1.26 times as long,
// 1792 x 121 by 121 x 2864, four limbs 36.6 and 44.3 us; from 0.3 on 2 to 9 % faster, never more than 5 % slower, 128 x 128 by 128 x 8192, two
// limbs 9.2 and 8.0 us), unless
// - the strips are few and no multiple of eight, so that more than a sixteenth of the XCDs' time would idle, or an XCD with one strip more
//   than the others would run another round of work-groups (slots: work-groups resident on an XCD.  736 x 128 by 128 x 2640, two limbs
//   12.4 and 10.5 us; 877 x 392 by 392 x 528, int16 W, three 45-bit limbs 14.6 and 10.4);
// - W counts most (heavy_w, far more rows than columns), of which runs give an XCD an eighth of the rows to read: 14336 x 512 by 512 x 128,
//   one 36-bit limb 13.3 -> 8.5 us with runs, 65536 x 512 by 512 x 256 63.0 -> 45.5, 14336 x 1250 by 1250 x 256 30.0 -> 26.3.  By rows of W's
//   slices per column: 8 to 16 equal (30 shapes), 16 to 64 whole strips 2 to 8 % slower (23), beyond 64 1.24 times as long and more (7).
inline bool heavy_w(int64_t M, int S, int64_t L, int64_t Ncols) { return M * S > 16 * L * Ncols; }
inline bool whole_strips(int64_t M, int64_t K, int64_t Ncols, int64_t L, int S) { return 5 * K * (8 - L) > M * L && !heavy_w(M, S, L, Ncols); }
struct StripRaster {
    int nstrips, mparts;      // strips per limb, parts per strip
    int whole;                // 1: all parts of a strip on one XCD
    int64_t per_xcd, total;   // strips (whole) or pairs, per XCD and in all
    int64_t grid;
};
inline StripRaster strip_raster(int64_t L, int64_t nstrips, int64_t mparts, bool whole, int64_t slots)
{
    StripRaster r;
    r.nstrips = (int)nstrips;
    r.mparts = (int)mparts;
    const int64_t strips = L * nstrips, per = (strips + 7) / 8;
    const auto rounds = [&](int64_t wgs) { return (wgs + slots - 1) / slots; };
    r.whole = whole && 16 * strips >= 15 * 8 * per && rounds(per * mparts) <= rounds((strips * mparts + 7) / 8);
    r.total = r.whole ? strips : strips * mparts;
    r.per_xcd = (r.total + 7) / 8;
    r.grid = r.per_xcd * 8 * (r.whole ? mparts : 1);
    return r;
}

// ---- the kernel that keeps the digits of a whole contraction in LDS (pcmm_resident.hip)
constexpr int64_t kLdsBytes = 160 * 1024;   // of a compute unit
struct ResidentTile {
    int NT;                // 16-column fragments per strip; 0: this kernel does not run
    int MT;                // 16-row blocks a wave takes at a time
    int waves;             // per work-group: 4 (two work-groups a compute unit, at most half of LDS each) or 8
    int groups_per_part;   // groups of MT row blocks per work-group
};
// 16-row blocks a wave takes at a time: 4 MT NT E accumulation registers, 4 MT S for each set of W fragments, 4 D for digits
constexpr int resident_mt(int D, int S, int NT)
{
    if (NT == 2) return S == 1 && D <= 5 ? 4 : 3;
    return S == 1 ? 4 : 3;
}
// k-steps by which W fragments are requested ahead of their use: what fits 256 registers without spills, at most three (two
// from seven digits on, whose contractions may have two k-steps only)
constexpr int resident_ahead(int D, int S, int NT, int MT)
{
    const int E = D + S - 1, most = E >= 7 ? 2 : 3;
    const int ahead = (226 - 4 * MT * NT * E - 4 * D - 4 * MT * S) / (4 * MT * S);
    return ahead > most ? most : ahead < 1 ? 1 : ahead;
}
// k-steps that are cut and contracted
inline int64_t resident_ksteps(int64_t K) { return K > 64 ? (K + 63) / 64 : 2; }
// rows of residues in k-step kb: 0 in one of padding
constexpr int64_t resident_rows(int64_t K, int64_t kb) { return K <= kb * 64 ? 0 : K - kb * 64 < 64 ? K - kb * 64 : 64; }
// Bytes behind the packed weights that belong to their allocation: the last row group's blocks beyond MB in the last k-step of the
// last slice (fewer than MT of them, MT <= 4) are fetched and not used.
constexpr int64_t kWpSlack = 3 * kFragBytes;

// Whether C is stored non-temporally.  Rows on half lines of 128 bytes: always (1000 x 777 by 777 x 12288, three 45-bit limbs
// 234 -> 202 us; 4096 x 500 by 500 x 8192, four 36-bit limbs 421 -> 302).  At other places lines are shared with the neighbouring
// strip and cached stores join them in L2 (over 860 shapes non-temporal ones 15 to 30 % slower), except on quarter lines from 60
// products a 16 x 16 block on, where the strips drift apart before they could be joined (1000 x 777 by 777 x 12300 242 -> 215;
// over 190 shapes 0 to 6 % faster).
inline bool resident_nt_stores(int64_t K, int64_t Ncols, uint64_t c_address, int D, int S)
{
    const uint64_t at = (uint64_t)Ncols * 8 | c_address;
    return at % 64 == 0 || (at % 32 == 0 && resident_ksteps(K) * D * S >= 60);
}

// The tile for C = W A of L limbs, or NT = 0 where none fits.  The candidates are the strip widths, work-group sizes and numbers of row
// parts that fit, up to eight parts, more where eight would leave compute units idle (eight -> more, one 36-bit limb: 65536 x 256 by
// 256 x 16 42 -> 6.3 us, digit split and GEMM kernel 11.2; 14336 x 1000 by 1000 x 16 29 -> 11.5, 15.1).  The estimate, per work-group, is a
// start, the digits that each wave cuts, and the rounds of row groups each wave runs (MFMAs of two waves sharing a SIMD, and the
// epilogue), times the rounds of work-groups, a last partial round counting 0.4 of a full one; strips of 16 columns count
// 15 % more, since each output row is stored in pieces half as long.  The constants are a fit to 2600 shapes (129 to 2048 values
// of k, all digit counts) that ranks these candidates; the tile it picks is 1 % behind the fastest of them on average.  (Limb pairs,
// nine digits for two limbs, were candidates too and gained nothing here: a tenth of the MFMAs less, but two reductions of nine
// accumulators for every output pair.)
inline ResidentTile resident_tile(int64_t M, int64_t K, int64_t Ncols, int64_t L, int D, int S)
{
    ResidentTile best = {0, 0, 0, 0};
    double best_clocks = 0.0;
    const int64_t ks = resident_ksteps(K);
    const int E = D + S - 1;
    for (int NT = 2; NT >= 1; --NT) {
        if (NT == 2 && E > 6) continue;          // no registers for two column fragments
        const int64_t lds = ks * NT * D * kFragBytes;
        if (lds > kLdsBytes) continue;
        const int MT = resident_mt(D, S, NT);
        const int64_t groups = (M + 16 * MT - 1) / (16 * MT), strips = L * ((Ncols + 16 * NT - 1) / (16 * NT));
        const double mfma = 16.0 * ks * MT * NT * D * S, epilogue = MT * NT * (32.0 * E + 360.0);
        for (int waves = 4; waves <= 8; waves += 4) {
            if (waves == 4 && lds > kLdsBytes / 2) continue;
            const int64_t slots = waves == 4 ? 512 : 256;
            const int64_t most = slots / strips > 8 ? slots / strips : 8;   // few strips: parts to fill the chip
            for (int64_t p = 1; p <= most && p <= groups; ++p) {
                const int64_t per_part = (groups + p - 1) / p, wgs = strips * ((groups + per_part - 1) / per_part);
                if ((wgs + 8 * p) * waves * 64 >= (int64_t)1 << 32) continue;   // a launch counts its threads in 32 bits (the raster rounds up)
                const double wg = 2300.0 + 1400.0 * ks * NT / waves + (double)((per_part + waves - 1) / waves) * (3.1 * mfma + epilogue);
                const double full = (double)wgs / slots, rounds = 0.4 * (double)((wgs + slots - 1) / slots) + 0.6 * (full > 1.0 ? full : 1.0);
                const double t = rounds * wg * (NT == 1 ? 1.15 : 1.0);
                if (best.NT && t >= best_clocks) continue;
                best_clocks = t;
                best.NT = NT; best.MT = MT; best.waves = waves; best.groups_per_part = (int)per_part;
            }
        }
    }
    return best;
}

// Everything about a plan that follows from its arguments alone.
struct Geometry {
    int D, S, E;               // digits per residue, int8 slices of W, accumulators per output
    int WM, MT, NT;            // waves per work-group, 16-row fragments per wave, 16-column fragments per tile
    int epi;                   // epi::Epi
    int64_t MB;                // padded M / 16
    int64_t nkb;               // padded K / 64 (even): the k-steps of the layouts
    int64_t nkb_launch;        // most k-steps one GEMM launch may contract (int32 accumulator headroom)
    int64_t ksteps;            // k-steps that are split and contracted: ceil(K / 64), and one of padding where a launch
                               // would otherwise be left with a single k-step or odd_ksteps() says so
    int64_t mtiles, ntiles;
    size_t wp_bytes, ad_bytes, lc_bytes;
    int pairs;                 // limb pairs split jointly (0 or L / 2)
    int64_t pair_ntiles;       // n-tiles of 16 columns
    int gn, pair_gn;           // n-tiles per raster group of the GEMM kernel, for single limbs and for pairs
    ResidentTile resident;     // NT > 0: the whole contraction fits LDS and runs as one kernel
    uint32_t w_kstride;        // bytes between k-steps of one packed W slice
    uint32_t a_kstride;        // bytes between k-steps of one limb's digit chunks
};

// Which of the two ways a contraction takes whose digits fit LDS is decided by an estimate of both in microseconds.  Their form: rounds of
// work-groups (a last partial one counting more than its share) times the clocks of one at 2 GHz, and the memory traffic, most of which runs
// beside them (rows of C that start inside lines cost more); the digit split in front of the GEMM kernel.  The constants are a fit to
// 3600 shapes measured both ways (16 to 30000 rows, 129 to 2560 values of k, 16 to 40000 columns, 24 to 62 bits, both widths of W), logarithmic
// deviation 0.15 and 0.12.  Taking the resident kernel where its estimate is below 0.92 of the other's is 0.66 times the GEMM kernel's time on
// average, 0.4 % behind the better of the two, longer than the GEMM kernel by more than 3 % at 37 of the shapes and by more than 10 % at 10
// (always taking it: 168 and 85, where strips are a few more than whole rounds, 1500 x 777 by 777 x 4100, two 36-bit limbs 69 -> 85 us, or
// one wave a SIMD contracts, 64 x 832 by 832 x 16384, four 58-bit limbs of int16 W 5 to 16 % slower).
constexpr double kResidentMargin = 0.92;
inline double rounds_of(double full, double whole, double part) { return part * whole + (1.0 - part) * full; }
// two kinds of work of which the shorter is hidden but for a part
inline double beside(double a, double b, double exposed) { return a > b ? a + exposed * b : b + exposed * a; }
inline double ceil_of(double x) { return (double)(int64_t)x < x ? (double)(int64_t)x + 1.0 : (double)(int64_t)x; }
inline double resident_us(const ResidentTile &t, int64_t M, int64_t K, int64_t Ncols, int64_t L, int D, int S)
{
    const int64_t ks = resident_ksteps(K), groups = (M + 16 * t.MT - 1) / (16 * t.MT), mparts = (groups + t.groups_per_part - 1) / t.groups_per_part;
    const double mfma = 16.0 * ks * t.MT * t.NT * D * S, epilogue = t.MT * t.NT * (32.0 * (D + S - 1) + 360.0);
    // a work-group: start, digits, the MFMAs of the waves that share a SIMD, and each wave's epilogues
    const int wgs_cu = t.waves == 4 ? 2 : 1;
    const double wg = 2900.0 + 1000.0 * ks * t.NT / t.waves + mfma * ((t.groups_per_part * wgs_cu + 3) / 4) +
                      (double)((t.groups_per_part + t.waves - 1) / t.waves) * (0.98 * epilogue + 0.082 * mfma);
    const double full = (double)(L * ((Ncols + 16 * t.NT - 1) / (16 * t.NT)) * mparts) / (256 * wgs_cu);
    // of two work-groups a compute unit, one alone takes half the time of both
    const double rounds = wgs_cu == 2 ? rounds_of(full, 0.5 * ceil_of(2.0 * full), 0.9) : rounds_of(full, ceil_of(full), 0.97);
    const double compute = rounds * wg / 2000.0 * (t.NT == 1 ? 1.2 : 1.0);
    const double memory = 8e-6 * L * Ncols * (M * (Ncols % 16 == 0 ? 0.13 : Ncols % 8 == 0 ? 0.17 : 0.25) + 0.16 * K);
    return 0.9 + beside(compute, memory, 0.42);
}
inline double gemm_us(const Geometry &g, int64_t M, int64_t K, int64_t Ncols, int64_t L)
{
    // work-groups a few more than whole rounds cost little: slots become free at different times
    auto products = [&](int64_t limbs, int64_t ntiles, int per_block) {       // per_block: int8 products of a row block and n-tile
        const double full = (double)(limbs * g.mtiles * ntiles) / 512;
        const double rounds = rounds_of(full, ceil_of(full), full > 1.0 && ceil_of(full) - full > 0.9 ? 0.1 : 0.48);
        return rounds * (7700.0 + g.ksteps * (780.0 + 22.4 * g.MT * per_block)) * (g.WM == 2 ? 0.86 : 1.0) / 2000.0;
    };
    const double compute = products(g.pairs, g.pair_ntiles, kPairDigits) + products(L - 2 * g.pairs, g.ntiles, g.NT * g.D * g.S);
    const double memory = 8e-6 * L * M * Ncols * (Ncols % 8 == 0 ? 0.21 : 0.29);
    return 7.6 + 0.16e-6 * (8 + g.D) * L * K * Ncols + beside(compute, memory, 0.26);
}

// Validates the arguments of pcmm_plan_create that need no device and derives the geometry.
inline pcmm_status plan_geometry(int64_t M, int64_t K, int64_t Ncols, int32_t L, const uint64_t *primes_host,
                                 int32_t prime_bits, int32_t w_bits, int32_t device, Geometry *g)
{
    if (!primes_host || !g) return PCMM_EINVAL;
    if (M <= 0 || K <= 0 || Ncols <= 0 || L <= 0 || L > kMaxLimbs) return PCMM_EINVAL;
    if (M > (int64_t)1 << 24 || Ncols > (int64_t)1 << 22) return PCMM_EINVAL;   // 32-bit row offsets in the stores
    if (w_bits != 8 && w_bits != 16) return PCMM_EINVAL;
    if (prime_bits < 24 || prime_bits > 62) return PCMM_EINVAL;
    if (device < 0) return PCMM_EINVAL;
    uint64_t qmax = 0, qmin = ~(uint64_t)0;
    for (int j = 0; j < L; ++j) {
        const uint64_t q = primes_host[j];
        if ((q & 1) == 0) return PCMM_EINVAL;
        if (q <= ((uint64_t)1 << (prime_bits - 1)) || q >= ((uint64_t)1 << prime_bits)) return PCMM_EINVAL;
        if (q > qmax) qmax = q;
        if (q < qmin) qmin = q;
    }
    const int S = w_bits / 8;
    if (K > ((int64_t)1 << 22) - 128) return PCMM_EINVAL;   // k-steps are a grid dimension of the split kernel
    // int32 headroom: one launch may contract Kl values of k with S*Kl*2^14 < 2^31, S*Kl <= 131071;
    // in k-steps of 64, rounded down to the even count the main loop needs
    const int64_t nkb_launch = 131071 / S / 128 * 2;
    const int64_t K_launch = K < nkb_launch * 64 ? K : nkb_launch * 64;

    int D = balanced_digits(qmax);
    if (D == 0) return PCMM_EUNSUPPORTED;
    if (D < 4) D = 4;   // kernels are built for 4..8 digits; spare top digits are zero
    const int E = D + S - 1;
    if (E > 9) return PCMM_EUNSUPPORTED;   // cannot happen with D <= 8 and S <= 2; kept as a guard

    g->D = D; g->S = S; g->E = E;
    g->NT = 2;
    g->MT = tile_mt(E);
    g->WM = (M > (int64_t)2 * g->MT * 16) ? 4 : 2;
    const int64_t BM = (int64_t)g->WM * g->MT * 16, BN = (int64_t)g->NT * 16;
    g->mtiles = (M + BM - 1) / BM;
    g->ntiles = (Ncols + BN - 1) / BN;
    g->MB = g->mtiles * BM / 16;
    g->nkb = (K + 127) / 128 * 2;   // the main loop takes two k-steps of 64 per round
    g->nkb_launch = nkb_launch;
    const int64_t ks = (K + 63) / 64;
    g->ksteps = !odd_ksteps(S, g->MT) ? g->nkb : (ks - 1) % nkb_launch == 0 ? ks + 1 : ks;   // at most nkb: nkb_launch is even
    if ((int64_t)L * g->mtiles * g->ntiles > 0x7fffff00LL) return PCMM_EUNSUPPORTED;   // the grid is a 32-bit count

    g->epi = qmax < ((uint64_t)1 << 50) ? epi::EPI_F64 : epi::EPI_INT;
    // short contractions leave small accumulators: |acc| <= S * K_launch * 2^14
    if (g->epi == epi::EPI_F64 && E >= 7 && qmin > ((uint64_t)1 << 37)) {
        if ((int64_t)S * K_launch <= 509) g->epi = epi::EPI_F64_G4P;   // 257 * S*K * 2^14 < 2^31
        else if ((int64_t)S * K_launch <= 16383) g->epi = epi::EPI_F64_G4;
    }

    g->wp_bytes = (size_t)S * g->MB * g->nkb * kFragBytes;
    g->ad_bytes = (size_t)L * g->ntiles * g->nkb * g->NT * D * kFragBytes;
    g->lc_bytes = (size_t)L * sizeof(LimbConst);
    // buffer loads address one W slice and one limb of digit planes with 32-bit unsigned byte offsets
    if (g->wp_bytes / S >= ((size_t)1 << 31) || g->ad_bytes / L >= ((size_t)1 << 32)) return PCMM_EUNSUPPORTED;
    // Limb pairs share nine digits where two limbs take ten.  Their digit planes, 9 * pair_ntiles fragments per k-step
    // with pair_ntiles <= 2 ntiles, are never more than the 10 * 2 ntiles of two single limbs, so ad_bytes covers them.
    // Contractions of at most 128 values of k keep single limbs: their kernel holds a limb's digits in registers.
    // An odd number of limbs leaves one that runs singly, in launches of its own behind those of the pairs: two starts and
    // two last rounds of work-groups.  That costs 10 to 30 us and pays from about 2.5 10^10 products a limb on, the digit split
    // counted as 600 rows (a line chosen over 290 shapes of 200 to 13629 rows: 0.4 % behind the better of the two on average,
    // 10 % at worst).  pcmm_run, all three limbs singly -> a pair and one single: 100 x 192 by 192 x 8192 25 -> 37 us; 1000 x
    // 400 by 400 x 8192 106 -> 114; 2048 x 672 by 672 x 4096 118 -> 134; 4096 x 1000 by 1000 x 4096 269 -> 274; 200 x 2611 by
    // 2611 x 16384 465 -> 467; 6000 x 1000 by 1000 x 4096 383 -> 386; 200 x 9000 by 9000 x 8192 828 -> 785; 4096 x 672 by 672 x
    // 8192 449 -> 433; 9344 x 2611 by 2611 x 4096 1235 -> 1202; 4096 x 4096 by 4096 x 8192 1726 -> 1674.
    // Rows of C that start inside a 128-byte line: every n-tile shares a line with its neighbour, and a pair's tiles are half as
    // wide.  With more than 16 m-tiles, where the raster below cannot make up for it, pairs then pay beyond 768 values of k
    // only (singly -> pairs, two limbs, 12301 columns: 9000 x 192 by 192 623 -> 675 us; 6000 x 512 607 -> 635; 6000 x 768
    // 739 -> 756; 6000 x 1000 863 -> 868; 6000 x 1500 1124 -> 1102; up to 16 m-tiles 2048 x 192 156 -> 161, 4096 x 400
    // 403 -> 403, 1000 x 1000 232 -> 218).
    constexpr int64_t kOddLimbsProducts = 25000000000, kSplitRows = 600;
    const bool shared_lines = Ncols % 16 != 0 && g->mtiles > 16 && K <= 768;
    g->pair_ntiles = (Ncols + 15) / 16;
    g->pairs = 0;
    if (S == 1 && D == 5 && g->nkb > 2 && (uint64_t)g->pair_ntiles * g->nkb * kPairDigits * kFragBytes < ((uint64_t)1 << 32) &&
        !shared_lines && (L % 2 == 0 || (M + kSplitRows) * K * Ncols >= kOddLimbsProducts)) {   // M * K < 2^31 (wp_bytes): the product fits
        g->pairs = L / 2;
        for (int j = 0; j < L / 2; ++j)
            if (!pair_ok(primes_host[2 * j], primes_host[2 * j + 1])) g->pairs = 0;
    }

    // The raster of the GEMM kernel: the work-groups that are resident together on one XCD (32 CUs) form a block of about
    // 8 m-tiles x gn n-tiles.  Eight n-tiles of 32 columns are 2 KiB of every output row; a pair's tiles have 16 columns and
    // take sixteen for the same 2 KiB while the contraction is short enough for the stores to count (at most 2048 values of
    // k) and the matrix has at most 16 m-tiles (pcmm_run, 8 -> 16 n-tiles: 2048 x 256 by 256 x 8192, four limbs 216 -> 198 us,
    // 198 singly; 4096 x 256 by 256 x 16384, four limbs 768 -> 650, 704 singly; 2048 x 1500 by 1500 x 8192, four limbs
    // 608 -> 569, 603 singly).  With more m-tiles sixteen are slower (14336 x 1500 by 1500 x 8192, four limbs 2930 -> 3325),
    // with longer contractions they are equal or slower (4096 x 4096 by 4096 x 32768, four limbs 8767 and 8765; 4096 x 14336 by
    // 14336 x 8192, five limbs 9147 -> 9654).
    g->gn = 8;
    g->pair_gn = g->mtiles <= 16 && K <= 2048 ? 16 : 8;

    // Contractions whose digits fit LDS run as one kernel that cuts the digits itself (those of at most 128 values of k below
    // 2^50 as pcmm_shortk's) where that is the faster way: by the estimates, or whenever a strip has no more than one row group
    // and four waves, where it always is (48 x 131 by 131 x 8208, two 56-bit limbs 24 -> 13 us).
    // A long W and few columns: limb pairs read W once for two limbs (65536 x 1000 by 1000 x 16, four 36-bit limbs, resident -> GEMM
    // kernel 46 -> 35 us; 65536 x 1250 by 1250 x 48 86 -> 74; 40000 x 1000 by 1000 x 16 30 -> 30, W of 38 MiB).
    g->resident = ResidentTile{0, 0, 0, 0};
    const bool shortk = g->nkb == 2 && D <= 7 && g->epi != epi::EPI_INT;
    const bool paired_long_w = g->pairs && M * K > (int64_t)40 << 20 && L * Ncols < 2048;
    if (!shortk && !paired_long_w) {
        const ResidentTile t = resident_tile(M, K, Ncols, L, D, S);
        if (t.NT && ((M <= 16 * t.MT && t.waves == 4) || resident_us(t, M, K, Ncols, L, D, S) < kResidentMargin * gemm_us(*g, M, K, Ncols, L)))
            g->resident = t;
    }

    g->w_kstride = (uint32_t)(g->MB * kFragBytes);
    g->a_kstride = (uint32_t)(g->ntiles * g->NT * D * kFragBytes);
    return PCMM_OK;
}

// Byte offset of k-step kk inside one W slice or one limb of digit chunks, as the kernel forms it:
// an unsigned 32-bit product.  The plan guarantees that (nkb - 1) * stride fits.
inline uint32_t kstep_offset(uint32_t kk, uint32_t kstride) { return kk * kstride; }

}  // namespace pcmm_host

#endif  // PCMM_HOST_HPP
