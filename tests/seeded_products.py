"""Products of seeded random or extreme operands on the GPU, made there, and their check against the oracle."""
import numpy as np

from plan_forms import primes


def run(gpu_device, M, K, Ncols, bits, L, w_bits, extreme, offsets=(32,)):
    """The product on the GPU and its inputs, with C at each of `offsets` 64-bit words behind a 512-byte boundary (all results alike);
    nothing beside C is written."""
    import torch

    import paper_2601_18511_amd as pkg

    qs = primes(bits, L)
    g = torch.Generator(device=gpu_device)
    g.manual_seed(M * 31 + K * 7 + Ncols)
    lo, hi, dt = (-128, 128, torch.int8) if w_bits == 8 else (-32768, 32640, torch.int16)
    W = torch.randint(lo, hi, (M, K), dtype=torch.int32, device=gpu_device, generator=g).to(dt)
    A = torch.stack([torch.randint(0, q, (K, Ncols), dtype=torch.int64, device=gpu_device, generator=g) for q in qs])
    if extreme:                                # weights of one sign, and residues at the ends of the range and of the balanced digits
        W = torch.where(W < hi // 2, lo, hi - 1).to(dt)
        for j, q in enumerate(qs):
            ends = torch.tensor([0, q - 1, q // 2, q // 2 + 1, sum(0x7F << (8 * i) for i in range(8)) % (1 << (bits - 1)),
                                 sum(0x80 << (8 * i) for i in range(8)) % (1 << (bits - 1))], dtype=torch.int64, device=gpu_device)
            A[j] = ends[A[j] % 6]
    whole = torch.empty((L * M * Ncols + 128,), dtype=torch.int64, device=gpu_device)
    plan = pkg.pcmm_plan_create(W, qs, bits, Ncols)
    first = None
    for at in offsets:
        whole.fill_(-7)
        C = whole[at:at + L * M * Ncols].view(L, M, Ncols)
        pkg.pcmm_run(plan, A, C)
        torch.cuda.synchronize()
        assert bool((whole[:at] == -7).all()) and bool((whole[at + L * M * Ncols:] == -7).all())
        assert first is None or bool((C == first).all())
        first = C.clone() if len(offsets) > 1 else C
    pkg.pcmm_plan_destroy(plan)
    return W, A, C, qs


def _sample(n, every):
    return sorted(set(range(0, n, every)) | set(range(min(4, n))) | set(range(max(0, n - 4), n)))


def check(W, A, C, qs):
    """All of C against the oracle, or a sample of its rows (every 7th) and columns (every 29th, of every tile another) where it is large."""
    from oracle import pcmm_oracle

    M, Ncols = C.shape[1:]
    rows, cols = _sample(M, 1 if M <= 3000 else 7), _sample(Ncols, 1 if Ncols <= 200 else 29)
    assert bool((C >= 0).all())
    got = C[:, rows][:, :, cols].cpu().numpy().view(np.uint64)
    want = pcmm_oracle(W[rows].cpu().numpy(), A[:, :, cols].contiguous().cpu().numpy().view(np.uint64), qs)
    assert (got == want).all(), int((got != want).sum())
