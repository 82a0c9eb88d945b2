"""Dispatch rules of the library, and forms that a rule chooses between, on the CPU
(tests/helpers/host_rules.cpp, a host-only build of its headers under
AddressSanitizer and UndefinedBehaviorSanitizer)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "helpers", "host_rules.cpp")


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    clang = "/opt/rocm/llvm/bin/clang++"
    if not (os.path.exists(hipcc) and os.path.exists(clang)):
        pytest.skip("no HIP compiler")
    d = tmp_path_factory.mktemp("host_rules")
    obj, exe = str(d / "host_rules.o"), str(d / "host_rules")
    inc = ["-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2407_18015_amd", "csrc")]
    # host pass only (no device code is built); the sanitizers apply to it
    subprocess.run([hipcc, "-xhip", "--offload-host-only", "-O1", "-g", "-std=c++17", "-fno-omit-frame-pointer",
                    "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
                    "-Xarch_host", "-fno-sanitize-recover=undefined", *inc, "-c", SRC, "-o", obj], check=True)
    subprocess.run([clang, "-fsanitize=address,undefined", obj, "-o", exe], check=True)

    def call(*args):
        r = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0 and "Sanitizer" not in r.stderr and "runtime error" not in r.stderr, r.stderr[-4000:]
        return r.stdout.split()

    return call


# every sample count that the entry point takes, to the last of 31 bits
@pytest.mark.parametrize("ns", [1, 3, 4, 5, 1000, 2**31 - 5, 2**31 - 4, 2**31 - 3, 2**31 - 1])
def test_semianalytical_blocks(rules, ns):
    assert int(rules("blocks", ns)[0]) == (ns + 3) // 4


# The form that was the faster one by more than a tenth where both were timed
# (vertex per thread 1, per wave 0).
@pytest.mark.parametrize("ns,nbins,el,side,thread", [
    (128, 10, 4, 1024, 1), (192, 10, 4, 1024, 0), (128, 2, 4, 2048, 1), (144, 2, 4, 2048, 1), (192, 2, 4, 2048, 0),
    (128, 3, 4, 1024, 1), (192, 3, 4, 1024, 0), (96, 16, 4, 2048, 1), (160, 16, 4, 2048, 0), (80, 20, 4, 2048, 1),
    (80, 24, 4, 2048, 1), (112, 24, 4, 2048, 0), (80, 32, 4, 1024, 0), (48, 32, 4, 1024, 1), (96, 4, 4, 512, 1),
    (144, 4, 4, 512, 0), (32, 10, 4, 256, 1), (64, 10, 4, 256, 0), (16, 10, 4, 128, 0), (1000, 10, 4, 40, 0),
    (128, 4, 8, 2048, 1), (64, 16, 8, 1024, 1), (96, 16, 8, 1024, 0), (64, 24, 8, 1024, 0), (32, 24, 8, 1024, 1),
    (2**31 - 1, 32, 8, 2048, 0)])
def test_semianalytical_form(rules, ns, nbins, el, side, thread):
    assert int(rules("thread", ns, nbins, el, side * side)[0]) == thread


# Ranges on both sides of the limits below and above which BinOf divides, just
# inside them and in the middle.
@pytest.mark.parametrize("dtype,scale", [(0, s) for s in (-126, -100, -99, -98, -90, -80, -67, -66, -65, -30, 0, 60,
                                                          98, 99, 100)] +
                         [(1, s) for s in (-700, -665, -664, 0, 663, 664, 665)])
def test_histogram_bin_quotients(rules, dtype, scale):
    assert rules("quotients", dtype, scale, scale + 1000) == ["0", "0"]


# The histogram adjoint's gather, one vertex or 16 bytes of a row per thread: the same
# bits, and no address outside the workspace or the gradient.  Direct entries: rows
# of one vector, whole vectors, a last vector that overlaps the one before, padded
# rows.  Rows summed on chip (workspaces past 128 MB): the last vector beside, across
# and inside the edge of a 64-vertex tile, a last tile of one vertex.
@pytest.mark.parametrize("dtype,H,W,nbins,stride,rows", [
    (0, 1, 4, 1, 4, 0), (0, 3, 5, 5, 8, 0), (0, 2, 6, 9, 6, 0), (0, 5, 7, 4, 7, 0), (0, 2, 64, 3, 64, 0),
    (0, 4, 65, 10, 67, 0), (0, 3, 131, 2, 131, 0), (0, 2, 130, 32, 132, 0),
    (1, 1, 2, 1, 2, 0), (1, 4, 3, 5, 5, 0), (1, 3, 4, 9, 4, 0), (1, 2, 65, 4, 65, 0), (1, 3, 128, 13, 129, 0),
    (0, 5500, 65, 18, 65, 1), (0, 5420, 66, 18, 66, 1), (0, 5340, 67, 18, 68, 1), (0, 6000, 128, 10, 128, 1),
    (0, 1400, 257, 18, 257, 1), (0, 900, 431, 18, 431, 1), (1, 3750, 65, 13, 65, 1), (1, 1900, 128, 13, 130, 1),
    (1, 3000, 130, 8, 130, 1)])
def test_histogram_gather_forms(rules, dtype, H, W, nbins, stride, rows):
    assert rules("gather", dtype, H, W, nbins, stride, 7) == [str(rows), "0"]
