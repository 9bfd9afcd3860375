"""Limbs whose digits are split jointly (two residues below 2^36 in nine digits): the split's arithmetic on the host, the
products against the oracle on the GPU.  All bit-exact."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import pcmm_inputs as pi
import plan_forms

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_joint_digits_on_the_host(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    exe = tmp_path / "pair_digits_check"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-ffp-contract=off",
                    "-fsanitize=undefined", "-fno-sanitize-recover=all",
                    "-I", os.path.join(ROOT, "paper_2601_18511_amd", "csrc"), "-o", str(exe),
                    os.path.join(ROOT, "tests", "host", "pair_digits_check.cpp")], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "all checks held" in r.stdout


def test_the_measuring_tools_count_the_digit_planes_that_a_plan_makes(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    calls = "".join(
        'uint64_t q_%s[] = {%s}; if (plan_geometry(%d, %d, %d, %d, q_%s, %d, %d, 0, &g) != PCMM_OK) return 1;\n'
        'printf("%s %%d %%d\\n", g.pairs, 9 * g.pairs + g.D * (%d - 2 * g.pairs));\n'
        % (w.name, ", ".join("%dull" % q for q in w.primes), w.M, w.K, w.Ncols, w.L, w.name, w.prime_bits, w.w_bits, w.name, w.L)
        for w in pi.WORKLOADS.values())
    src = tmp_path / "planes.cpp"
    src.write_text('#include <stdio.h>\n#include "pcmm_host.hpp"\nint main() { using namespace pcmm_host; Geometry g;\n' + calls + "return 0; }\n")
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2601_18511_amd", "csrc"), "-o", str(tmp_path / "planes"), str(src)],
                   check=True)
    out = subprocess.run([str(tmp_path / "planes")], capture_output=True, text=True, check=True).stdout
    assert out.split("\n")[:-1] == ["%s %d %d" % (w.name, w.limb_pairs, w.digit_planes) for w in pi.WORKLOADS.values()]
    w = pi.WORKLOADS
    assert (w["attn_proj"].digit_planes, w["ffn_down"].digit_planes, w["tiny"].digit_planes) == (18, 14, 10)
    assert w["attn_proj"].run_int8_ops * 10 == w["attn_proj"].int8_ops * 9


# contractions of up to 2048 values of k whose digits fit LDS run singly, limb by limb, in the kernel that cuts the digits itself
SHORT = [
    (1, 129, 1, 36, 2, False),          # smallest contraction that pairs; one row, one column
    (128, 200, 15, 36, 2, True),        # two-wave work-groups, ragged column fragment
    (129, 192, 16, 33, 2, False),
    (200, 150, 40, 31, 2, True),        # smallest primes of five digits
    (129, 192, 33, 32, 4, False),
    (300, 129, 16, 32, 2, False),
    (129, 192, 16, 33, 3, False),       # an odd number of limbs this small: all singly
    (256, 256, 17, 34, 4, True),
    (300, 257, 63, 35, 4, False),       # ragged rows, columns and k
    (300, 257, 63, 35, 5, False),
    (257, 700, 130, 36, 6, True),
    (500, 200, 257, 36, 2, False),      # raster groups of sixteen n-tiles, the last of one tile; two m-tiles
    (4100, 150, 273, 36, 2, False),     # 17 m-tiles, rows of C inside lines: singly
    (4100, 150, 272, 36, 2, True),      # 17 m-tiles: raster groups of eight
    (64, 130944 + 64, 20, 36, 2, False),   # K in two launches: the second adds to both limbs of the pair
    (64, 130944 + 64, 20, 36, 3, False),
]
# the same edges where limbs are paired
PAIRED = [
    (1, 2049, 1, 36, 2, False),
    (128, 2100, 15, 36, 2, True),       # two-wave work-groups, ragged column fragment
    (129, 2113, 16, 33, 2, False),
    (200, 2049, 40, 31, 2, True),       # smallest primes of five digits
    (129, 2300, 33, 32, 4, False),
    (256, 2112, 17, 34, 4, True),
    (300, 2057, 63, 35, 4, False),      # ragged rows, columns and k
    (257, 2700, 130, 36, 6, True),
    (4100, 2050, 33, 36, 2, True),      # 17 m-tiles
    (1500, 777, 4100, 36, 2, False),    # raster groups of sixteen n-tiles, the last of one tile
    (64, 130944 + 64, 20, 36, 2, False),   # K in two launches: the second adds to both limbs of the pair
    (64, 130944 + 65, 40, 33, 4, True),
]


def test_the_lists_pair_limbs_where_they_say(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    for M, K, Ncols, bits, L, _ in PAIRED:
        forms = plan_forms.gemm_kernels(plan_forms.describe([(M, K, Ncols, bits, L, 8)], tmp_path)[0])
        assert [f[4] for f in forms] == ["pair"], (M, K, Ncols, bits, L)


@pytest.mark.gpu
@pytest.mark.parametrize("extreme", [False, True])
@pytest.mark.parametrize("M,K,Ncols,bits,L,ascending", SHORT + PAIRED)
def test_paired_limbs_bit_exact(gpu_device, M, K, Ncols, bits, L, ascending, extreme):
    import torch

    import paper_2601_18511_amd as pkg
    from oracle import pcmm_oracle, pcmm_oracle_select

    rng = np.random.default_rng(M + K)
    primes = pi.ntt_primes(bits, 1 << 10, L)
    primes = list(primes)[::-1] if ascending else list(primes)
    if extreme:
        W = np.where(rng.random((M, K)) < 0.9, -128, 127).astype(np.int8)
        A = np.stack([rng.choice(np.array([0, 1, q // 2, q - 1], dtype=np.uint64), size=(K, Ncols)) for q in primes])
    else:
        W = rng.integers(-128, 128, size=(M, K), dtype=np.int64).astype(np.int8)
        A = np.stack([rng.integers(0, q, size=(K, Ncols), dtype=np.uint64) for q in primes])
    plan = pkg.pcmm_plan_create(torch.from_numpy(W).to(gpu_device), primes, bits, Ncols)
    C = torch.full((L, M, Ncols), -1, dtype=torch.int64, device=gpu_device)
    pkg.pcmm_run(plan, torch.from_numpy(A.view(np.int64)).to(gpu_device), C)
    torch.cuda.synchronize()
    pkg.pcmm_plan_destroy(plan)
    got = C.cpu().numpy().view(np.uint64)
    if M * K * Ncols * L < 1 << 30:
        assert (got == pcmm_oracle(W, A, primes)).all()
    else:                                  # all rows of every 13th column and of the last tiles
        cols = sorted(set(range(0, Ncols, 13)) | set(range(Ncols - 20, Ncols)))
        assert (got[:, :, cols] == pcmm_oracle_select(W, A, primes, np.arange(M), cols)).all()


@pytest.mark.gpu
def test_pairs_and_a_single_limb(gpu_device):
    """Three limbs of 2 10^10 products each, enough for pairs: the first two as a pair, the last one singly; ragged rows, columns and k, sampled."""
    import torch

    import paper_2601_18511_amd as pkg
    from oracle import pcmm_oracle_select

    M, K, Ncols, L, bits = 2500, 2000, 4100, 3, 36
    primes = pi.ntt_primes(bits, 1 << 10, L)
    g = torch.Generator(device=gpu_device)
    g.manual_seed(7)
    W = torch.randint(-128, 128, (M, K), dtype=torch.int8, device=gpu_device, generator=g)
    A = torch.stack([torch.randint(0, q, (K, Ncols), dtype=torch.int64, device=gpu_device, generator=g) for q in primes])
    C = torch.full((L, M, Ncols), -1, dtype=torch.int64, device=gpu_device)
    plan = pkg.pcmm_plan_create(W, primes, bits, Ncols)
    pkg.pcmm_run(plan, A, C)
    torch.cuda.synchronize()
    pkg.pcmm_plan_destroy(plan)
    W_host, A_host = W.cpu().numpy(), A.cpu().numpy().view(np.uint64)
    C_host = C.cpu().numpy().view(np.uint64)
    rows = [0, 255, 256, 1023, 2304, M - 1]
    cols = list(range(0, 40)) + list(range(2040, 2060)) + list(range(Ncols - 30, Ncols))
    all_rows, all_cols = np.arange(M), np.arange(Ncols)
    assert (C_host[:, rows, :] == pcmm_oracle_select(W_host, A_host, primes, rows, all_cols)).all()
    assert (C_host[:, :, cols] == pcmm_oracle_select(W_host, A_host, primes, all_rows, cols)).all()
