"""The performance cases: what a user of this library has it do, from the smallest call to the largest.

Every case goes through the public entry points of paper_2601_18511_amd with the plan, the inputs and the output
buffers on the GPU, as a program that serves requests holds them.  Kinds:

  pcmm             C_j = W . A_j mod q_j for all limbs (the linear layers and the plaintext-ciphertext attention products)
  ring_decompose   coefficient permutation before the product:  [npoly][N] -> [npoly][k][N/k]
  ring_compose     the inverse, after the product
  slot             rearranged plaintexts of the slot-encoded batch product, made at run time
  pcmv             ring products of the decode-time matrix-vector product

All results are whole numbers and compared exactly.
"""
import math

import torch

import paper_2601_18511_amd as lib

# Model dimensions of the layers: hidden 4096, intermediate 14336, head 128.
HIDDEN, INTER, HEAD = 4096, 14336, 128


def _pcmm(name, M, K, Ncols, L, prime_bits, w_bits):
    return {"name": name, "kind": "pcmm", "M": M, "K": K, "Ncols": Ncols, "L": L, "prime_bits": prime_bits, "w_bits": w_bits}


def listed():
    return [
        # smallest product: one 128 x 128 block of a blocked projection on one ciphertext row set of ring degree 4096;
        # launches and latency count
        _pcmm("tiny", 128, 128, 8192, 2, 36, 8),
        # a ragged product: dimensions that are no multiple of any tile (a pruned or low-rank layer), 45-bit limbs
        _pcmm("ragged", 1000, 777, 12300, 3, 45, 8),
        # attention output (and query) projection of a prefill step, ring degree 2^14
        _pcmm("attn_proj", HIDDEN, HIDDEN, 32768, 4, 36, 8),
        # feed-forward up or gate projection: the largest product of a layer
        _pcmm("ffn_up_gate", INTER, HIDDEN, 32768, 4, 36, 8),
        # feed-forward down projection: the longest contraction
        _pcmm("ffn_down", HIDDEN, INTER, 32768, 3, 36, 8),
        # plaintext keys times encrypted queries: the contraction is the head dimension, the output is huge
        _pcmm("wide_pc_attn", HIDDEN, HEAD, 131072, 6, 50, 16),
        # the projection in the 16-bit weight format under one modulus of about 64 bits
        _pcmm("attn_proj_w16_q62", HIDDEN, HIDDEN, 32768, 1, 62, 16),
        # a batch of channels of ring degree 2^16 taken to ring degree 2^12 before a projection
        {"name": "ring_decompose", "kind": "ring_decompose", "npoly": 4096, "N": 65536, "k": 16},
        # one ciphertext of four limbs put together again after a product at ring degree 2^8
        {"name": "ring_compose", "kind": "ring_compose", "npoly": 8, "N": 65536, "k": 256},
        # 64 stored 128 x 128 matrices, all 128 rearranged plaintexts of each
        {"name": "slot", "kind": "slot", "batch": 64, "d": HEAD, "ell": 1, "b": 16, "k_first": 0, "k_count": HEAD},
        # decode: one row of a 4096-column matrix per plaintext polynomial, one input ciphertext
        {"name": "pcmv_o_proj", "kind": "pcmv", "Mp": HIDDEN, "Kp": 1, "N": 4096, "L": 2, "prime_bits": 36},
        # decode: a 16384-long input spread over four ciphertexts
        {"name": "pcmv_down_proj", "kind": "pcmv", "Mp": HIDDEN, "Kp": 4, "N": 4096, "L": 2, "prime_bits": 36},
    ]


# ---------------------------------------------------------------------------------------------------------------------
# drawn cases
# ---------------------------------------------------------------------------------------------------------------------
def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi):
    """A size of [lo, hi], spread over its logarithm: a multiple of 64 in half of the draws (where there is one), any number otherwise."""
    v = _log_int(rng, lo, hi)
    return max(lo, v // 64 * 64) if rng.random() < 0.5 and v >= 64 else v


def _draw_pcmm(rng):
    largest = listed()[3]
    most = work(largest)
    while True:
        w_bits = rng.choice((8, 8, 16))
        bits = rng.choice((36, 36, 36, rng.randint(28, 49), 50, rng.randint(51, 62)))
        if rng.random() < 0.25:         # the contraction is a head dimension: short and wide
            M, K, Ncols = _size(rng, 64, 8192), rng.choice((64, 80, 96, 128, rng.randint(33, 128))), 2 << rng.randint(12, 16)
        else:
            M, K, Ncols = _size(rng, 64, INTER), _size(rng, 64, INTER), 2 << rng.randint(11, 14)
        if rng.random() < 0.25:         # part of a ciphertext row: any number of columns
            Ncols = rng.randint(Ncols // 2, Ncols)
        case = {"kind": "pcmm", "M": M, "K": K, "Ncols": Ncols, "L": rng.randint(1, 6), "prime_bits": bits, "w_bits": w_bits}
        w = work(case)
        # the digit planes of one limb stay below 4 GiB by far; time and memory stay below the largest listed case's
        if w["flops"] <= most["flops"] and w["bytes"] <= most["bytes"] and K * Ncols * 8 < 3 << 30:
            return case


def draw(rng):
    kind = rng.choice(("pcmm",) * 7 + ("ring_decompose", "ring_compose", "slot", "pcmv", "pcmv"))
    if kind == "pcmm":
        return _draw_pcmm(rng)
    if kind in ("ring_decompose", "ring_compose"):
        log_n = rng.randint(12, 16)
        log_k = rng.randint(1, log_n - 4)
        return {"kind": kind, "npoly": _log_int(rng, 2, (1 << 28) >> log_n), "N": 1 << log_n, "k": 1 << log_k}
    if kind == "slot":
        d = rng.choice((64, 128, 128, 256, 96, rng.randint(24, 200)))
        b = rng.choice([x for x in range(1, d + 1) if d % x == 0])
        k_count = rng.randint(1, d)
        most = (1 << 27) // (d * d * k_count)
        return {"kind": "slot", "batch": _log_int(rng, 1, max(2, most)), "d": d, "ell": rng.randint(-2, 2), "b": b,
                "k_first": rng.randint(0, d - k_count), "k_count": k_count}
    N = rng.choice((4096, 4096, 4096, 2048, 1024))
    Kp = rng.choice((1, 1, 1, 2, 3, 4, rng.randint(5, 16)))
    L = rng.randint(1, 4)
    bits = rng.choice((36, 36, rng.randint(28, 35), rng.randint(37, 50)))
    return {"kind": "pcmv", "Mp": _size(rng, 32, min(8192, (1 << 29) // (L * Kp * N * 2))), "Kp": Kp, "N": N, "L": L, "prime_bits": bits}


# ---------------------------------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------------------------------
def _is_prime(n):
    """Miller-Rabin with the bases that decide every n < 2^64."""
    for p in (2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37):
        if n % p == 0:
            return n == p
    d, s = n - 1, 0
    while d % 2 == 0:
        d, s = d // 2, s + 1
    for a in (2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37):
        x = pow(a, d, n)
        if x in (1, n - 1):
            continue
        for _ in range(s - 1):
            x = x * x % n
            if x == n - 1:
                break
        else:
            return False
    return True


def _primes(bits, two_n, count):
    """The largest primes of `bits` bits that are 1 modulo two_n, descending."""
    out, q = [], ((1 << bits) - 1) // two_n * two_n + 1
    while len(out) < count:
        if q < 1 << bits and _is_prime(q):
            out.append(q)
        q -= two_n
        if q <= 1 << (bits - 1):
            raise ValueError("not enough primes of %d bits" % bits)
    return out


def _residues(shape, primes, gen):
    """[L][...] int64, uniform below each prime (ciphertext residues are indistinguishable from uniform ones)."""
    out = torch.empty((len(primes),) + shape, dtype=torch.int64, device="cuda")
    for j, q in enumerate(primes):
        out[j].random_(0, q, generator=gen)
    return out


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    kind = case["kind"]
    if kind == "pcmm":
        M, K, Ncols, L, bits = (case[x] for x in ("M", "K", "Ncols", "L", "prime_bits"))
        primes = _primes(bits, 1 << min(15, bits - 18), L)
        if case["w_bits"] == 8:
            W = torch.randint(-128, 128, (M, K), dtype=torch.int8, device="cuda", generator=gen)
        else:                           # weights and keys: Gaussian, scaled by 2^10
            W = torch.randn((M, K), device="cuda", generator=gen).mul_(1024.0).round_().clamp_(-32768, 32639).to(torch.int16)
        A = _residues((K, Ncols), primes, gen)
        C = torch.empty((L, M, Ncols), dtype=torch.int64, device="cuda")
        return {"kind": kind, "plan": lib.pcmm_plan_create(W, primes, bits, Ncols), "A": A, "C": C}
    if kind == "pcmv":
        Mp, Kp, N, L, bits = (case[x] for x in ("Mp", "Kp", "N", "L", "prime_bits"))
        primes = _primes(bits, 2 * N, L)
        pt = torch.randint(-32768, 32768, (Mp, Kp, N), dtype=torch.int32, device="cuda", generator=gen)
        ct = _residues((Kp, 2, N), primes, gen)
        out = torch.empty((L, Mp, 2, N), dtype=torch.int64, device="cuda")
        return {"kind": kind, "plan": lib.pcmv_plan_create(pt, primes, bits), "ct": ct, "out": out}
    if kind == "slot":
        batch, d, k_count = case["batch"], case["d"], case["k_count"]
        S = torch.empty((batch, d, d), dtype=torch.int64, device="cuda").random_(generator=gen)
        out = torch.empty((batch, k_count, d, d), dtype=torch.int64, device="cuda")
        return {"kind": kind, "S": S, "out": out, "args": (d, case["ell"], case["b"], case["k_first"], k_count)}
    npoly, N, k = case["npoly"], case["N"], case["k"]
    whole, parts = (npoly, N), (npoly, k, N // k)
    src = torch.empty(whole if kind == "ring_decompose" else parts, dtype=torch.int64, device="cuda").random_(generator=gen)
    dst = torch.empty(parts if kind == "ring_decompose" else whole, dtype=torch.int64, device="cuda")
    return {"kind": kind, "src": src, "dst": dst, "N": N, "k": k}


def run(state):
    kind = state["kind"]
    if kind == "pcmm":
        lib.pcmm_run(state["plan"], state["A"], state["C"])
        return state["C"]
    if kind == "pcmv":
        lib.pcmv_run(state["plan"], state["ct"], state["out"])
        return state["out"]
    if kind == "slot":
        lib.pcmm_slot_rearrange(state["S"], state["out"], *state["args"])
        return state["out"]
    call = lib.pcmm_ring_decompose if kind == "ring_decompose" else lib.pcmm_ring_compose
    call(state["src"], state["dst"], state["N"], state["k"])
    return state["dst"]


def work(case):
    """Bytes: every input read once, every output written once.  Operations: for the products, int8 multiply-adds on the
    bytes of weight and residue (the precision of the operands); for the ring products, the butterflies and the pointwise
    products as modular multiplications of six and additions of one double-precision operation."""
    kind = case["kind"]
    if kind == "pcmm":
        M, K, n, L = case["M"], case["K"], case["Ncols"], case["L"]
        S, D = case["w_bits"] // 8, -(-case["prime_bits"] // 8)
        return {"bytes": 8 * L * n * (K + M) + S * M * K, "flops": 2 * M * K * n * L * D * S}
    if kind == "pcmv":
        Mp, Kp, N, L = case["Mp"], case["Kp"], case["N"], case["L"]
        logn = N.bit_length() - 1
        # a stored plaintext value needs the bits of its residue
        return {"bytes": L * N * (Mp * Kp * case["prime_bits"] // 8 + 16 * Mp + 16 * Kp),
                "flops": 2 * L * N * (Mp * (7 * Kp + 4 * logn) + Kp * 4 * logn)}
    if kind == "slot":
        d2 = case["d"] ** 2
        return {"bytes": 8 * case["batch"] * d2 * (1 + case["k_count"]), "flops": 0}
    return {"bytes": 16 * case["npoly"] * case["N"], "flops": 0}


def tolerance(case):
    return "exact"
