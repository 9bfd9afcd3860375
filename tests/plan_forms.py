"""Which kernels the plans of a list of shapes run, by the library's own planning code compiled for the host (plan_forms.cpp)."""
import os
import subprocess

import pcmm_inputs as pi

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
_primes = {}


def primes(bits, L):
    """The first L primes of a size, as the tests of these shapes use them."""
    if bits not in _primes:
        _primes[bits] = pi.ntt_primes(bits, 1 << 8, 8)
    return list(_primes[bits][:L])


def describe(shapes, tmp_path):
    """One line (the format is in plan_forms.cpp) for each (M, K, Ncols, bits, L, w_bits)."""
    exe = str(tmp_path / "plan_forms")
    if not os.path.exists(exe):
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2601_18511_amd", "csrc"), "-o", exe,
                        os.path.join(ROOT, "tests", "host", "plan_forms.cpp")], check=True)
    text = "".join("%d %d %d %d %d %d %s\n" % (M, K, N, bits, w_bits, L, " ".join(str(q) for q in primes(bits, L)))
                   for M, K, N, bits, L, w_bits in shapes)
    lines = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
    assert len(lines) == len(shapes)
    return lines


def gemm_kernels(line):
    """The forms of the GEMM kernel that a plan launches: tuples (waves, digits, slices, epilogue, pair or single, odd or even count of
    k-steps, and for two waves whether they have their SIMD alone)."""
    if not line.startswith("gemm"):
        return []
    forms = [tuple(part.split()) for part in line.split(" | ")[1:] if part[0] in "24"]
    return [f if f[0] == "2" else f[:-1] for f in forms]


def field(line, name):
    """The value of a named field of a GEMM plan."""
    return next(part.split()[1] for part in line.split(" | ") if part.startswith(name + " "))
