"""Contractions whose digits fit LDS (pcmm_resident.hip): the tile that the plan chooses, on the host, and the products against the
oracle on the GPU, bit-exact, at the edges of row groups, strips and k-steps (SHAPES, strips of 16 columns) and for every kernel variant with
several row groups a wave (TURNS)."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import pcmm_inputs as pi
import plan_forms
from seeded_products import check, run

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HOST_CHECK = r"""
#include <initializer_list>
#include <stdio.h>
#include "pcmm_host.hpp"
using namespace pcmm_host;
#define CHECK(c) do { if (!(c)) { printf("check failed: %s (M %ld K %ld N %ld L %d bits %d w %d)\n", #c, (long)M, (long)K, (long)N, L, bits, wb); return 1; } } while (0)
int main()
{
    const long Ms[] = {1, 16, 64, 100, 513, 2049, 14336, 1 << 20, 1 << 24}, Ks[] = {1, 64, 65, 128, 129, 192, 320, 512, 513, 777, 1024, 1089, 1280, 2048, 2049, 4096};
    const long Ns[] = {1, 16, 33, 4096, 12300, 32768, 1 << 22};
    const int bitss[] = {24, 31, 33, 36, 41, 45, 48, 50, 51, 55, 58, 62};
    long used = 0, parts = 0, four = 0;
    for (long M : Ms) for (long K : Ks) for (long N : Ns) for (int bits : bitss) for (int wb = 8; wb <= 16; wb += 8) for (int L : {1, 2, 3, 4, 64}) {
        uint64_t q[64];
        for (int j = 0; j < L; ++j) q[j] = ((uint64_t)1 << bits) - 1 - 2 * j;
        Geometry g;
        if (plan_geometry(M, K, N, L, q, bits, wb, 0, &g) != PCMM_OK) continue;
        const ResidentTile &t = g.resident;
        if (!t.NT) continue;
        const int D = g.D, S = g.S;
        const int64_t ks = resident_ksteps(K), lds = ks * t.NT * D * kFragBytes;
        CHECK(lds <= kLdsBytes && (t.waves == 8 || (t.waves == 4 && 2 * lds <= kLdsBytes)));
        CHECK(t.MT == resident_mt(D, S, t.NT) && ks >= resident_ahead(D, S, t.NT, t.MT) && ks <= g.nkb && ks * 64 >= K);
        CHECK(t.NT == 1 || (t.NT == 2 && D + S - 1 <= 6));
        const int64_t groups = (M + 16 * t.MT - 1) / (16 * t.MT), mparts = (groups + t.groups_per_part - 1) / t.groups_per_part;
        CHECK(t.groups_per_part >= 1 && t.groups_per_part <= groups);
        const StripRaster r = strip_raster(L, (N + 16 * t.NT - 1) / (16 * t.NT), mparts, whole_strips(M, K, N, L, S), t.waves == 4 ? 64 : 32);
        CHECK(r.grid <= 0x7fffffffL && r.grid * t.waves * 64 < (int64_t)1 << 32);
        // the epilogues the kernel is built for
        CHECK(g.epi == epi::EPI_INT ? g.D >= 7 : g.E <= 6 ? g.epi == epi::EPI_F64 : g.epi == epi::EPI_F64_G4 || g.epi == epi::EPI_F64_G4P);
        // every byte of W that a lane may ask for belongs to the allocation, by the scalar offset alone: row groups, blocks beyond the
        // last row, k-steps requested ahead (those of the next group, or of the same one again behind the last)
        const int64_t w_end = ((S - 1) * g.nkb + (ks - 1)) * g.MB + (groups - 1) * t.MT + t.MT;
        CHECK(w_end * kFragBytes <= (int64_t)g.wp_bytes + kWpSlack);
        // every residue row that is asked for by a scalar offset exists
        for (int64_t kb = 0; kb < ks; ++kb) {
            const int64_t rows = resident_rows(K, kb);
            CHECK(rows == 0 ? kb * 64 >= K : kb * 64 + rows == (rows == 64 ? kb * 64 + 64 : K) && kb * 64 + rows <= K);
        }
        // byte offsets: a k-step of residues, a block of outputs, and W up to the groups past the last row
        CHECK(64 * N * 8 <= (int64_t)1 << 31 && ((ks + 2) * g.MB + (groups + 8) * t.MT) * kFragBytes < (int64_t)1 << 32);
        // many rows and few strips: the parts fill the compute units (within what whole row groups allow), and no XCD reads all of W
        const int64_t strips = L * ((N + 16 * t.NT - 1) / (16 * t.NT)), slots = t.waves == 4 ? 512 : 256;
        if (groups >= 8192) CHECK(strips * mparts * 2 > 256 || mparts * 2 > slots / strips);
        if (groups >= 8192 && N <= 33 && L < 64) CHECK(!r.whole);
        ++used; parts += mparts > 1; four += t.waves == 4;
    }
    printf("%s\n", used > 1000 && parts > 10 && four > 100 ? "1" : "0");
    return 0;
}
"""


def test_chosen_tiles_fit(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    (tmp_path / "t.cpp").write_text(HOST_CHECK)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                    "-I", os.path.join(ROOT, "paper_2601_18511_amd", "csrc"), "-o", str(tmp_path / "t"), str(tmp_path / "t.cpp")], check=True)
    r = subprocess.run([str(tmp_path / "t")], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "1", r.stdout + r.stderr


# (M, K, Ncols, bits, L, w_bits)
SHAPES = [
    (1, 129, 1, 36, 1, 8),            # one row, one column, three k-steps
    (15, 192, 15, 30, 2, 8),          # four digits
    (64, 193, 16, 36, 1, 8),          # four k-steps; one row group
    (65, 257, 17, 36, 3, 8),          # five k-steps
    (300, 320, 32, 36, 2, 8),         # pairs or singles by the estimate
    (1000, 500, 48, 33, 4, 8),
    (1100, 448, 4096, 36, 2, 8),
    (700, 384, 31, 45, 2, 8),         # six digits
    (130, 777, 36, 45, 1, 8),         # 13 k-steps, rows on quarter lines
    (130, 780, 40, 44, 1, 8),         # rows on half lines
    (200, 1000, 33, 50, 2, 8),        # seven digits, groups of four accumulators
    (200, 700, 33, 53, 2, 8),         # seven digits, integer epilogue
    (193, 1100, 20, 62, 1, 8),        # eight digits
    (128, 128, 64, 60, 2, 8),         # two k-steps (above 2^50: not the short kernel's)
    (77, 30, 18, 52, 2, 8),           # one k-step and one of padding
    (111, 100, 18, 55, 2, 16),
    (49, 129, 16, 30, 1, 16),         # int16 W, four digits
    (300, 640, 50, 36, 2, 16),
    (1000, 900, 34, 36, 1, 16),
    (500, 400, 24, 42, 2, 16),        # six digits
    (500, 350, 24, 50, 1, 16),
    (500, 350, 24, 54, 1, 16),
    (241, 1200, 25, 62, 1, 16),       # nine accumulators
    (100, 2048, 16, 36, 1, 8),        # 32 k-steps of five digits: all of LDS
    (3000, 200, 64, 36, 1, 8),        # few strips: the rows are cut into parts
    (5000, 130, 32, 50, 1, 16),
]


# Waves that take several row groups one after the other, a line for each (digits, slices, strip width, epilogue) and in it each remainder that the
# k-steps leave in the sets of W registers; whole half lines, so that the address of C decides between the two kinds of stores
TURNS = [
    (513, 200, 2040, 30, 3, 8), (513, 300, 2040, 30, 3, 8), (600, 350, 3000, 30, 2, 8), (513, 129, 3000, 30, 2, 8),
    (2100, 193, 3000, 30, 1, 8), (257, 257, 4096, 28, 4, 8), (2049, 350, 3000, 24, 1, 8), (2100, 129, 3000, 28, 1, 8),
    (777, 193, 2000, 30, 2, 16), (777, 320, 2040, 28, 2, 16), (777, 350, 2040, 30, 2, 16), (777, 129, 2000, 30, 2, 16),
    (257, 129, 4096, 30, 4, 16), (193, 200, 4096, 28, 4, 16), (2500, 257, 2000, 28, 1, 16),
    (513, 193, 2040, 38, 3, 8), (600, 257, 2000, 36, 3, 8), (513, 350, 3000, 36, 2, 8), (513, 150, 2040, 33, 3, 8),
    (300, 193, 4096, 36, 4, 8), (300, 129, 4096, 32, 4, 8),
    (777, 193, 2000, 36, 2, 16), (777, 300, 1000, 35, 4, 16), (2049, 350, 2000, 38, 1, 16), (777, 129, 2000, 38, 2, 16),
    (2500, 193, 1000, 33, 2, 16), (193, 129, 4096, 38, 4, 16),
    (777, 193, 1000, 45, 4, 8), (777, 257, 2000, 40, 2, 8), (777, 350, 1000, 45, 4, 8), (1000, 129, 3000, 45, 1, 8),
    (513, 200, 2000, 40, 4, 8), (2500, 257, 2000, 42, 1, 8), (2500, 350, 2000, 40, 1, 8), (513, 129, 4096, 42, 2, 8),
    (193, 129, 2040, 40, 4, 16), (193, 193, 2000, 40, 4, 16), (200, 300, 2040, 45, 4, 16),
    (513, 129, 4096, 48, 1, 8), (513, 200, 2000, 50, 2, 8), (513, 257, 4096, 50, 1, 8),
    (600, 150, 1000, 52, 4, 8), (513, 193, 2000, 52, 2, 8), (600, 257, 2040, 52, 2, 8),
    (200, 129, 4096, 49, 2, 16), (193, 200, 2000, 50, 4, 16), (200, 257, 4096, 48, 2, 16),
    (200, 129, 2040, 52, 4, 16), (513, 193, 4096, 52, 1, 16), (600, 257, 2000, 52, 2, 16),
    (513, 129, 1000, 55, 4, 8), (513, 193, 2000, 55, 2, 8), (513, 257, 2040, 55, 2, 8),
    (193, 129, 4096, 55, 2, 16), (193, 193, 2000, 62, 4, 16), (193, 320, 2000, 62, 4, 16),
]
# as many digits as LDS holds, by the digit count; and one strip of 32 columns of them
FULL_LDS = [(64, 2560, 4096, 30, 1, 8), (300, 2497, 40, 28, 1, 16), (64, 2048, 100, 38, 1, 8), (100, 1664, 72, 45, 1, 8), (100, 1408, 40, 50, 1, 8),
            (70, 1280, 40, 60, 1, 8), (1000, 1280, 4096, 30, 4, 8), (1000, 1024, 4096, 36, 4, 8), (777, 832, 4096, 45, 4, 8)]


def test_the_faster_of_the_two_ways_runs(tmp_path):
    """Shapes on either side of the estimates that choose between this kernel and the digit split with the GEMM kernel, each measured both ways."""
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    gemm = [(1500, 777, 4100, 36, 2, 8), (2048, 1024, 4100, 36, 2, 8), (2500, 1024, 4100, 36, 2, 8), (600, 777, 4100, 36, 2, 16),
            (2048, 1284, 848, 36, 5, 16), (4627, 1839, 1352, 36, 2, 8), (4895, 255, 8208, 62, 2, 16), (17, 832, 16384, 58, 4, 16)]
    resident = [(1000, 777, 12300, 45, 3, 8), (128, 128, 64, 60, 2, 8), (64, 300, 4096, 58, 2, 16), (600, 300, 4096, 36, 2, 16),
                (48, 131, 8208, 56, 2, 8), (1000, 1024, 12300, 36, 2, 8), (51, 196, 14240, 48, 5, 8)]
    assert all(line.startswith("gemm") for line in plan_forms.describe(gemm, tmp_path)), plan_forms.describe(gemm, tmp_path)
    assert all(line.startswith("resident") for line in plan_forms.describe(resident, tmp_path)), plan_forms.describe(resident, tmp_path)


def test_turns_reach_every_variant(tmp_path):
    """Over a grid of shapes: every variant that a plan runs with several row groups a wave is among those of TURNS."""
    if shutil.which("g++") is None:
        pytest.skip("no g++")

    def variants(shapes):
        lines = [line.replace("g4p", "g4").split() for line in plan_forms.describe(shapes, tmp_path)]      # one kernel for both
        return {(f[1], f[2], f[3], f[4], f[6]) for f in lines if f[0] == "resident" and f[7] == "turns"}

    grid = [(M, K, N, bits, L, w_bits) for M in (193, 257, 513, 1000, 2100, 4096) for K in (129, 200, 260, 330, 400, 500, 777, 1024, 1400, 2500)
            for N in (512, 2000, 4096, 12288) for bits in (28, 36, 44, 49, 53, 60) for L in (1, 2, 4) for w_bits in (8, 16)]
    missing = variants(grid) - variants(TURNS)
    assert not missing, sorted(missing)
    assert {v[:4] for v in variants(TURNS)} == {v[:4] for v in variants(grid)} and len({v[:4] for v in variants(TURNS)}) == 17
    lines = [line.split() for line in plan_forms.describe(TURNS, tmp_path)]
    assert all(f[0] == "resident" and f[7] == "turns" for f in lines) and all(shape[2] % 8 == 0 for shape in TURNS)
    assert all(line.startswith("resident") for line in plan_forms.describe(FULL_LDS, tmp_path))


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,Ncols,bits,L,w_bits", TURNS + FULL_LDS)
def test_several_row_groups_a_wave(gpu_device, M, K, Ncols, bits, L, w_bits):
    check(*run(gpu_device, M, K, Ncols, bits, L, w_bits, M % 2 == 0, offsets=(32, 33)))


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,Ncols,bits,L,w_bits", SHAPES)
@pytest.mark.parametrize("extreme", [False, True])
def test_resident_products_bit_exact(gpu_device, M, K, Ncols, bits, L, w_bits, extreme):
    import torch

    import paper_2601_18511_amd as pkg
    from oracle import pcmm_oracle

    rng = np.random.default_rng(M + K + bits)
    primes = list(pi.ntt_primes(bits, 1 << 8, L))
    lo, hi, dt = (-128, 127, np.int8) if w_bits == 8 else (-32768, 32639, np.int16)
    if extreme:
        W = np.where(rng.random((M, K)) < 0.9, lo, hi).astype(dt)
        A = np.stack([rng.choice(np.array([0, 1, q // 2, q - 1], dtype=np.uint64), size=(K, Ncols)) for q in primes])
    else:
        W = rng.integers(lo, hi + 1, size=(M, K), dtype=np.int64).astype(dt)
        A = np.stack([rng.integers(0, q, size=(K, Ncols), dtype=np.uint64) for q in primes])
    plan = pkg.pcmm_plan_create(torch.from_numpy(W).to(gpu_device), primes, bits, Ncols)
    # rows of 64-bit words around C show stores outside it; an odd offset in words takes the cached stores
    whole = torch.full((L * M * Ncols + 64,), -1, dtype=torch.int64, device=gpu_device)
    A_dev = torch.from_numpy(A.view(np.int64)).to(gpu_device)
    want = pcmm_oracle(W, A, primes)
    for at in (32, 33):
        whole.fill_(-1)
        C = whole[at:at + L * M * Ncols].view(L, M, Ncols)
        pkg.pcmm_run(plan, A_dev, C)
        torch.cuda.synchronize()
        assert (C.cpu().numpy().view(np.uint64) == want).all()
        assert bool((whole[:at] == -1).all()) and bool((whole[at + L * M * Ncols:] == -1).all())
    pkg.pcmm_plan_destroy(plan)
