"""The FP64 triangularisation (lq_rows of device_math.hpp), built for the host by
tests/tria_check.cpp with 24-bit stand-ins for the hardware's reciprocal
estimates."""
import os
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def check():
    """check(*arguments): the program's lines."""
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    with tempfile.TemporaryDirectory() as tmp:
        exe = os.path.join(tmp, "tria_check")
        subprocess.run([HIPCC, "-O2", "-std=c++17", "-x", "hip", "--offload-arch=gfx950",
                        "-Xarch_host", "-mfma", "-I" + os.path.join(ROOT, "include"),
                        os.path.join(ROOT, "tests", "tria_check.cpp"), "-o", exe],
                       check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
        yield lambda *a: subprocess.run([exe, *a], check=True, stdout=subprocess.PIPE,
                                        text=True).stdout.splitlines()


def test_gram_is_as_exact_as_the_textbook_sweep(check):
    """Also where one part is far smaller than the other, as process noise beside
    a factor.  0.05 units of 2^-53 are left to the draws (20 000 of them)."""
    for line in check():
        e, lib, ref = (float(v) for v in line.split())
        print("e %g: library %.3f, textbook %.3f" % (e, lib, ref))
        assert lib < ref + 0.05, e


def test_small_rows_are_kept(check):
    """Rows of norm 1e-150 are reduced as any others: to 64 units, since squares
    of their small entries are subnormal (of 1e-307, 1e-17 of the row's sum).  A
    pivot without a tail is kept at any size."""
    scaled, diag = check("small")
    assert float(scaled) < 64
    assert [float(v) for v in diag.split()] == [1e-200, 1e-200, 1e-3, 1e-200, 1e-200]
