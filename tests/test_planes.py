"""The cut of fp32 factors into three bf16 planes (csrc/psd_planes.h), compiled for the CPU: no bit of any number is lost."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_1512_06216_amd import build
from tests.conftest import ROOT


@pytest.fixture(scope="module")
def planes(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("planes") / "planes.so")
    rocm = os.path.dirname(os.path.dirname(build.HIPCC))
    subprocess.run([os.path.join(rocm, "lib", "llvm", "bin", "clang++"), "-x", "c++", "-std=c++17", "-O1", "-ffp-contract=off", "-shared", "-fPIC",
                    "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"), "-I", build.CSRC,
                    os.path.join(ROOT, "tests", "host", "planes_check.cpp"), "-o", so], check=True)
    L = ctypes.CDLL(so)
    L.scale_of_factors.restype = L.scale_of_sums.restype = ctypes.c_float

    def cut(x):
        x = np.ascontiguousarray(x, np.float32)
        out = [np.empty(x.size // 2, np.uint32) for _ in range(3)]
        L.planes_of(x.size, *(ctypes.c_void_p(a.ctypes.data) for a in (x, *out)))
        halves = [a.view(np.uint16).astype(np.uint32) for a in out]            # little endian: the first number in the low half
        return [(a << 16).view(np.float32).astype(np.float64) for a in halves]
    cut.lib = L
    return cut


def test_three_planes_are_the_number_at_every_exponent_of_a_finite_result(planes):
    """Smallest and largest number of every binade, numbers around a tie of the first and of the second plane, and random ones.
    Planes too small for a normal bf16 are taken as zero here: none may be needed."""
    assert planes.lib.scale_of_factors() ** 2 * planes.lib.scale_of_sums() == 1.0
    rng = np.random.default_rng(24)
    mantissas = np.concatenate([[0, 1, 2, 3, 0x7fff, 0x8000, 0x8001, 0x17fff, 0x18000, 0x18001, 0x807f, 0x8080, 0x8081, 0x80ff, 0x7fffff, 0x7ffffe,
                                 0x7f8000, 0x7f7fff], rng.integers(0, 1 << 23, size=2000)]).astype(np.uint32)
    for e in range(0, 127 + 104):                              # biased exponent; 0: subnormal numbers
        x = (mantissas | np.uint32(e << 23)).view(np.float32)
        x = np.concatenate([x, -x])
        h, m, l = planes(x)
        want = x.astype(np.float64) * planes.lib.scale_of_factors()
        if e == 127 + 103:                                     # rounds up to 2^128 there
            keep = np.isfinite(h)
            assert keep.mean() > 0.98
            h, m, l, want = h[keep], m[keep], l[keep], want[keep]
        assert np.array_equal(h + m + l, want), e
        assert np.all(np.abs(m) <= 2.0 ** -8 * np.abs(want)) and np.all(np.abs(l) <= 2.0 ** -17 * np.abs(want)), e
        for p in (h, m, l):
            assert np.all((p == 0) | (np.abs(p) >= 2.0 ** -126)), e


def test_numbers_that_cannot_be_cut_show(planes):
    """A plane that is not finite: the sum it goes into is then not finite either."""
    x = np.array([np.inf, -np.inf, np.nan, 3e38, -3e38, 2.0 ** 104, -2.0 ** 120, 1e32], np.float32)
    with np.errstate(invalid="ignore"):
        h, m, l = planes(x)
        assert not np.isfinite(h + m + l).any()
