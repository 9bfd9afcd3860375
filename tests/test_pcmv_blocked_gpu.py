"""PCMv at ring degrees 1024 and 2048, which run on the register-blocked kernels with two or three stages in the last pass: against the
schoolbook oracle in both reduction regimes, and with more output polynomials than persistent work-groups.  Bit-exact."""
import numpy as np
import pytest

import pcmm_inputs as pi

pytestmark = pytest.mark.gpu


def _run(pt, ct, primes, bits, dev):
    import torch

    import paper_2601_18511_amd as pkg

    plan = pkg.pcmv_plan_create(torch.from_numpy(pt.astype(np.int32)).to(dev), primes, bits)
    ct_dev = torch.from_numpy(ct.view(np.int64)).to(dev)
    out = torch.full((ct.shape[0], pt.shape[0], 2, pt.shape[2]), -1, dtype=torch.int64, device=dev)
    pkg.pcmv_run(plan, ct_dev, out)
    torch.cuda.synchronize()
    pkg.pcmv_plan_destroy(plan)
    return out.cpu().numpy().view(np.uint64)


@pytest.mark.parametrize("N", [1024, 2048])
@pytest.mark.parametrize("bits", [24, 36, 37, 50])
@pytest.mark.parametrize("Kp", [1, 3])
def test_blocked_degrees_against_the_oracle(gpu_device, N, bits, Kp):
    from oracle import pcmv_oracle

    rng = np.random.default_rng(N + bits + Kp)
    primes = pi.ntt_primes(bits, 2 * N, 2)
    wmax = (1 << 31) - 1
    pt = rng.integers(-wmax, wmax, size=(5, Kp, N), dtype=np.int64)
    pt[0], pt[1] = wmax, -wmax
    ct = np.stack([rng.integers(0, q, size=(Kp, 2, N), dtype=np.uint64) for q in primes])
    for j, q in enumerate(primes):
        ct[j, 0, 0] = rng.choice(np.array([0, 1, q - 1, q // 2], dtype=np.uint64), size=N)
        ct[j, Kp - 1, 1] = q - 1
    assert (_run(pt, ct, primes, bits, gpu_device) == pcmv_oracle(pt, ct, primes)).all()


@pytest.mark.parametrize("N,Mp,Kp,L,bits", [(1024, 1400, 1, 3, 36), (1024, 2049, 2, 1, 44), (2048, 700, 1, 3, 50), (2048, 1025, 2, 1, 36)])
def test_work_queue_at_the_smaller_degrees(gpu_device, N, Mp, Kp, L, bits):
    """More output polynomials than work-groups (2048 at degree 1024, 1024 at 2048): equal to plans of at most 500 rows, which run one
    polynomial a work-group, and three rows against the oracle."""
    from oracle import pcmv_oracle_rows

    rng = np.random.default_rng(Mp)
    primes = pi.ntt_primes(bits, 2 * N, L)
    pt = rng.integers(-(1 << 15), 1 << 15, size=(Mp, Kp, N), dtype=np.int64)
    ct = np.stack([rng.integers(0, q, size=(Kp, 2, N), dtype=np.uint64) for q in primes])
    got = _run(pt, ct, primes, bits, gpu_device)
    step = 500 // L
    for r0 in range(0, Mp, step):
        assert (got[:, r0:r0 + step] == _run(pt[r0:r0 + step], ct, primes, bits, gpu_device)).all(), r0
    rows = [0, Mp // 2, Mp - 1]
    assert (got[:, rows] == pcmv_oracle_rows(pt[rows], ct, primes, list(range(len(rows))))).all()
