"""The digit split and the GEMM kernel (contractions whose digits do not fit LDS, and those that keep these kernels for other reasons):
every form of the kernels that a plan can launch, against the oracle, bit-exact.  A host test finds the forms that plans launch over a
grid of shapes and asks that the lists below reach each of them, so that a change of the dispatch cannot empty these tests unseen."""
import shutil

import pytest

import plan_forms
from seeded_products import check, run

# (M, K, Ncols, bits, L, w_bits); k-steps are ceil(K / 64), the work-groups of two waves take 32 columns and up to 128 rows
FORMS = [
    # two waves, at most two work-groups a compute unit
    (33, 2600, 17, 24, 1, 8), (97, 2650, 40, 30, 3, 8),          # four digits, odd and even counts of k-steps
    (20, 2561, 17, 28, 1, 16), (96, 2700, 33, 30, 2, 16),
    (100, 2049, 17, 38, 1, 8), (20, 2130, 47, 38, 3, 8),         # five, too large for pairs
    (90, 2049, 17, 35, 1, 16), (96, 2120, 31, 38, 2, 16),
    (20, 1665, 17, 45, 1, 8), (95, 1730, 31, 40, 2, 8),          # six
    (33, 1700, 17, 42, 1, 16), (64, 1900, 31, 42, 2, 16),
    (20, 1409, 17, 48, 1, 8), (64, 1500, 33, 50, 2, 8),          # seven, groups of four accumulators
    (40, 16400, 17, 48, 1, 8), (40, 16480, 17, 48, 1, 8),        # groups of three
    (20, 1665, 17, 52, 1, 8), (47, 1730, 17, 53, 2, 8),          # integer epilogue
    (64, 1409, 17, 50, 1, 16), (33, 1900, 17, 50, 2, 16),
    (40, 8200, 33, 48, 1, 16), (40, 8300, 17, 50, 1, 16),
    (40, 8200, 33, 44, 1, 16), (40, 8300, 17, 44, 1, 16),        # six digits, two slices, groups of three
    (20, 1409, 17, 52, 1, 16), (64, 1500, 40, 53, 2, 16),
    (33, 1300, 17, 62, 1, 8), (64, 1400, 17, 58, 2, 8),          # eight
    (47, 1300, 17, 55, 1, 16), (63, 1400, 50, 62, 2, 16),
    (100, 2100, 17, 36, 2, 8), (128, 2130, 40, 33, 4, 8),        # limb pairs
    # two waves, more work-groups than that
    (20, 2561, 16385, 24, 1, 8), (20, 2650, 16385, 30, 1, 8),
    (20, 2600, 16390, 28, 1, 16),
    (20, 2049, 16385, 38, 1, 8), (20, 2130, 16400, 38, 1, 8),
    (20, 2049, 16385, 36, 1, 16), (20, 2130, 16385, 38, 1, 16),
    (20, 1665, 16385, 42, 1, 8), (20, 1730, 16400, 45, 1, 8),
    (20, 1665, 16385, 45, 1, 16), (20, 1730, 16385, 42, 1, 16),
    (20, 1409, 16385, 48, 1, 8), (20, 1500, 16400, 50, 1, 8),
    (20, 1409, 16385, 52, 1, 8), (20, 1500, 16385, 53, 1, 8),
    (20, 1409, 16385, 50, 1, 16), (20, 1500, 16385, 48, 1, 16),
    (20, 1409, 16385, 52, 1, 16), (20, 1500, 16400, 53, 1, 16),
    (20, 1300, 16385, 55, 1, 8), (20, 1400, 16385, 62, 1, 8),
    (20, 1300, 16385, 58, 1, 16), (20, 1400, 16385, 62, 1, 16),
    (20, 2049, 8200, 36, 2, 8), (20, 2130, 8209, 32, 2, 8),
    (20, 16400, 16385, 48, 1, 8), (20, 16480, 16385, 50, 1, 8),
    (20, 8200, 16385, 44, 1, 16), (20, 8300, 16385, 42, 1, 16),
    (20, 8200, 16385, 49, 1, 16), (20, 8300, 16385, 48, 1, 16),
    # four waves; a second tile of rows with one to three busy waves
    (300, 2600, 17, 24, 1, 8), (257, 2650, 40, 30, 3, 8),
    (300, 2561, 33, 28, 1, 16), (260, 2650, 17, 30, 2, 16),
    (150, 2049, 17, 38, 1, 8), (400, 2120, 40, 38, 1, 8),
    (250, 2049, 17, 38, 1, 16), (200, 2120, 31, 36, 2, 16),
    (150, 1665, 17, 45, 1, 8), (250, 1900, 33, 42, 2, 8),
    (150, 1700, 17, 45, 1, 16), (257, 1730, 17, 42, 2, 16),
    (193, 129, 4100, 40, 2, 16), (193, 200, 4100, 45, 2, 16),    # pairs of accumulators joined in int32
    (129, 8200, 17, 44, 1, 16), (129, 8300, 17, 44, 1, 16),      # groups of three
    (150, 1700, 17, 50, 1, 8), (257, 1730, 17, 48, 2, 8),
    (866, 400, 2056, 48, 1, 8), (1865, 340, 1030, 48, 1, 8),
    (129, 16400, 17, 48, 1, 8), (129, 16480, 17, 48, 1, 8),
    (150, 1409, 17, 52, 1, 8), (250, 1730, 17, 53, 2, 8),
    (200, 2049, 17, 48, 1, 16), (193, 1500, 33, 50, 2, 16),
    (600, 150, 4100, 49, 2, 16), (600, 193, 1030, 49, 2, 16),
    (129, 8200, 17, 48, 1, 16), (129, 8300, 17, 50, 1, 16),
    (150, 2049, 17, 52, 1, 16), (257, 1500, 17, 53, 2, 16),
    (150, 1300, 17, 58, 1, 8), (250, 1500, 33, 62, 2, 8),
    (193, 1409, 17, 55, 1, 16), (257, 1500, 17, 62, 2, 16),
    (300, 2049, 17, 32, 2, 8), (257, 2130, 40, 36, 4, 8),        # limb pairs
    # two launches: the second adds to C
    (64, 130944 + 64, 20, 28, 1, 8), (150, 65408 + 130, 17, 28, 1, 16), (150, 130944 + 130, 18, 55, 1, 8),
]

# more than 384 MiB of residues: digits, or digits and residues, past the caches
LARGE_SPLITS = [
    (20, 2650, 19010, 30, 1, 8), (20, 2650, 19008, 30, 1, 8),
    (20, 2100, 24010, 38, 1, 8), (20, 2100, 24016, 38, 1, 8),
    (20, 1700, 29650, 45, 1, 8), (20, 1700, 29648, 45, 1, 8),
    (20, 1500, 33570, 49, 1, 16), (20, 1500, 33568, 52, 1, 8),
    (20, 1400, 36010, 62, 1, 8), (20, 1400, 36016, 58, 1, 16),
    (20, 3000, 12300, 36, 2, 8), (20, 3000, 12304, 36, 2, 8),    # limb pairs
    (20, 2100, 12300, 36, 2, 8),                                 # just over: 394 MiB
]

# a W of more than 48 MiB and rows of C on half lines: stores past the caches
LARGE_W = [
    (19500, 2650, 24, 30, 1, 8), (24500, 2100, 24, 38, 1, 8), (30000, 1700, 40, 45, 1, 8), (34000, 1500, 24, 49, 1, 8), (34000, 1500, 24, 53, 1, 8),
    (36500, 1400, 24, 60, 1, 8), (9700, 2650, 24, 28, 1, 16), (12300, 2070, 24, 36, 1, 16), (15000, 1700, 24, 44, 1, 16),
    (16900, 1500, 24, 49, 1, 16), (16900, 1500, 24, 53, 1, 16), (18300, 1400, 24, 62, 1, 16), (17000, 3000, 40, 36, 2, 8),
]


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,Ncols,bits,L,w_bits", FORMS)
def test_every_form_of_the_gemm_kernel(gpu_device, M, K, Ncols, bits, L, w_bits):
    for extreme in (False, True) if Ncols <= 100 else (True,):
        check(*run(gpu_device, M, K, Ncols, bits, L, w_bits, extreme))


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,Ncols,bits,L,w_bits", LARGE_SPLITS)
def test_digits_and_residues_past_the_caches(gpu_device, M, K, Ncols, bits, L, w_bits):
    check(*run(gpu_device, M, K, Ncols, bits, L, w_bits, False))


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,Ncols,bits,L,w_bits", LARGE_W)
def test_stores_past_the_caches(gpu_device, M, K, Ncols, bits, L, w_bits):
    check(*run(gpu_device, M, K, Ncols, bits, L, w_bits, False))


def _forms(shapes, tmp_path):
    return {f for line in plan_forms.describe(shapes, tmp_path) for f in plan_forms.gemm_kernels(line)}


def test_the_lists_reach_every_form(tmp_path):
    """Over a grid of shapes, every form of the GEMM kernel that a plan launches (its template arguments and the parity of its k-steps) is
    one that FORMS launches; the lists with large operands reach every digit split and every epilogue of either width of W."""
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    grid = [(M, K, N, bits, L, w_bits)
            for M in (1, 33, 64, 65, 97, 128, 129, 200, 300, 513, 1100, 2100, 14336)
            for K in (150, 200, 257, 400, 500, 800, 1100, 1300, 1409, 1500, 1700, 2070, 2130, 2570, 2650, 4096, 17000, 17060)
            for N in (17, 64, 1000, 8200, 16385, 32768)
            for bits in (24, 30, 36, 38, 44, 48, 50, 53, 62) for L in (1, 2, 3) for w_bits in (8, 16)]
    missing = _forms(grid, tmp_path) - _forms(FORMS, tmp_path)
    assert not missing, "\n".join(" ".join(f) for f in sorted(missing))
    lines = plan_forms.describe(FORMS, tmp_path)
    assert all(plan_forms.gemm_kernels(line) for line in lines), [s for s, line in zip(FORMS, lines) if not plan_forms.gemm_kernels(line)]
    launches = [plan_forms.field(line, "launches") for line in lines]
    assert launches.count("2") == 3

    splits = set()
    for shape, line in zip(LARGE_SPLITS, plan_forms.describe(LARGE_SPLITS, tmp_path)):
        splits |= {(f[1], plan_forms.field(line, "split")) for f in plan_forms.gemm_kernels(line)}
    assert splits == {(d, kind) for d in "456789" for kind in ("stores", "both")}

    stores = set()
    for shape, line in zip(LARGE_W, plan_forms.describe(LARGE_W, tmp_path)):
        assert plan_forms.field(line, "stores") == "nt", shape
        stores |= {f[1:4] for f in plan_forms.gemm_kernels(line)}
    assert len(stores) == 13
