"""Rounding of the per-vertex routines on the CPU, against long double: host-only
builds of the library's own headers (tests/helpers/host_accuracy.cpp) over
random stencils, wide ones among them, where the probabilities' parity bounds
(1e-6 and 1e-12) would not show a loss."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "helpers", "host_accuracy.cpp")
F32, F64 = 0, 1


@pytest.fixture(scope="module")
def evaluate(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    clang = "/opt/rocm/llvm/bin/clang++"
    if not (os.path.exists(hipcc) and os.path.exists(clang)):
        pytest.skip("no HIP compiler")
    d = tmp_path_factory.mktemp("host_accuracy")
    obj, exe = str(d / "host_accuracy.o"), str(d / "host_accuracy")
    inc = ["-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2407_18015_amd", "csrc")]
    # fused multiply-adds as on the device
    subprocess.run([hipcc, "-xhip", "--offload-host-only", "-O2", "-std=c++17", "-mfma", *inc, "-c", SRC, "-o", obj],
                   check=True)
    subprocess.run([clang, obj, "-o", exe], check=True)

    def call(mode, records, *args):
        fin, fout = str(d / "in.bin"), str(d / "out.bin")
        np.ascontiguousarray(records, dtype=np.float64).tofile(fin)
        subprocess.run([exe, mode, *map(str, args), fin, fout], check=True, timeout=300)
        return np.fromfile(fout, dtype=np.float64).reshape(len(records), -1)

    return call


def stencils(seed, n, spread, offset, dtype):
    """(centre, width) of v, e, n, w, s: widths over e^+-spread, centres offset widths apart"""
    rng = np.random.default_rng(seed)
    w = 0.05 * np.exp(rng.uniform(-spread, spread, (n, 5)))
    c = 0.3 + 0.05 * offset * rng.normal(size=(n, 5))
    p = np.stack([c, w], 2).reshape(n, 10)
    return p.astype(np.float32).astype(np.float64) if dtype == F32 else p


def weighted(p, seed):
    g = np.random.default_rng(seed).normal(size=(len(p), 2)).astype(np.float32)
    return np.concatenate([p, g], 1)


def rms(e):
    return np.sqrt(np.mean(e * e))


# FP64.  What the trapezoidal rule leaves out is 2 exp(-Lam) of the density alone,
# and up to 2 Lam times that of a derivative's integrand; Lam = 37.5 makes it
# 1e-16 and 8e-15.  Rounding: a probability is a sum of positive terms of ten
# roundings each, 2e-15 at most; a derivative's terms change sign, 2e-15 of the
# largest entry with them.  Widths over e^+-2.8 hold narrow vertices beside wide
# and distant neighbours, whose step is the longest.
@pytest.mark.parametrize("spread,offset", [(0.7, 0.5), (2.0, 1.5), (2.8, 4.0)])
def test_gaussian_probabilities_fp64(evaluate, spread, offset):
    o = evaluate("gauss", weighted(stencils(3, 600, spread, offset, F64), 4), F64)
    assert np.abs(o[:, :4] - o[:, 14:18]).max() <= 2e-15


@pytest.mark.parametrize("spread", [0.7, 2.0])
def test_gaussian_derivatives_fp64(evaluate, spread):
    o = evaluate("gauss", weighted(stencils(5, 600, spread, 0.0, F64), 6), F64)
    exact = o[:, 18:]
    assert (np.abs(o[:, 4:14] - exact) / np.abs(exact).max(1, keepdims=True)).max() <= 1e-14


# FP32, narrow neighbours one to four deviations above the vertex: P_min is near 1,
# a sum of 100 to 200 nodes.  Half the parity bound of 1e-6 is left to the sum and
# the tails; the other half belongs to the hardware's reciprocal and exponential.
def test_gaussian_sums_fp32(evaluate):
    rng = np.random.default_rng(7)
    n = 2500
    w = 0.05 * np.exp(rng.uniform(-3, -1, (n, 5)))
    c = 0.3 + 0.05 * rng.uniform(1, 4, (n, 5))
    w[:, 0], c[:, 0] = 0.05, 0.3
    p = np.stack([c, w], 2).reshape(n, 10).astype(np.float32).astype(np.float64)
    o = evaluate("gauss", weighted(p, 8), F32)
    assert np.abs(o[:, :4] - o[:, 14:18]).max() <= 5e-7


# FP64 tails at every argument: zs = kTailScale z and zs^2 round to 2^-53 each, which
# the exponential turns into z^2 (1 + 1/2) 2^-53 of q, the constant's own rounding
# adds another z^2 2^-53, and 16 units cover the ratio of the polynomials.
def test_tails_fp64(evaluate):
    z = np.linspace(-30.0, 30.0, 6001)[:, None]
    err = np.abs(evaluate("tail", z)[:, 0])
    assert np.all(err <= (2.5 * z[:, 0] ** 2 + 16) * 2.0**-53)


# The saddle terms' pieces hold two or three factors by the shortest rules; the plain
# form evaluates all four on each of the five pieces.  They may round no worse:
# 20000 stencils leave about 1% of sampling error in the ratio of the rms errors,
# ten times that is allowed.
@pytest.mark.parametrize("dtype", [F32, F64])
@pytest.mark.parametrize("spread,offset", [(0.2, 0.3), (0.7, 0.5), (1.5, 1.0), (2.5, 2.0)])
def test_epanechnikov_saddle_terms(evaluate, dtype, spread, offset):
    o = evaluate("epa", stencils(9, 20000, spread, offset, dtype), dtype)
    assert rms(o[:, :2] - o[:, 4:]) <= 1.1 * rms(o[:, 2:4] - o[:, 4:])


# The sweep integrates from the midpoint of every interval; the plain form is the end
# values' in Bernstein form.  It may round no worse, both probabilities together:
# 4000 stencils leave about 1% of sampling error in the ratio of the rms errors,
# four times that is allowed.
@pytest.mark.parametrize("dtype,nbins", [(F32, 2), (F32, 4), (F32, 10), (F32, 32), (F64, 2), (F64, 4), (F64, 10),
                                         (F64, 32)])
@pytest.mark.parametrize("spread,offset", [(0.2, 0.3), (0.7, 0.5), (1.5, 1.0)])
def test_histogram_probabilities(evaluate, dtype, nbins, spread, offset):
    rng = np.random.default_rng(11)
    n = 4000
    p = stencils(12, n, spread, offset, F64).reshape(n, 5, 2)
    m = rng.integers(0, 7, (n, 5, nbins)).astype(float)
    m[..., 0] += m.sum(-1) == 0
    r = np.concatenate([(p[..., 0] - p[..., 1])[..., None], p.sum(-1)[..., None], m / m.sum(-1, keepdims=True)], 2)
    if dtype == F32:
        r = r.astype(np.float32).astype(np.float64)
    o = evaluate("hist", r.reshape(n, -1), dtype, nbins)
    assert rms(o[:, :2] - o[:, 4:]) <= 1.04 * rms(o[:, 2:4] - o[:, 4:])
