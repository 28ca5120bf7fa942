"""Batched workspaces in the FP32 modes are no larger than their unit tables, partial sums,
unpadded prepared coefficients (4 or, for the jerk, 8 numbers of each), coefficients and state
one after the other, although the layout for the matrix cores pads the prepared ones."""
import ctypes
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIBPATH = os.path.join(ROOT, "paper_1406_4254_amd", "libetics.so")


@pytest.fixture(scope="module")
def L():
    if not os.path.exists(LIBPATH):
        from paper_1406_4254_amd import build
        build.build()
    lib = ctypes.CDLL(LIBPATH)
    for f in (lib.etics_batched_workspace_size, lib.etics_hermite_workspace_size):
        f.argtypes = [ctypes.c_int64] + [ctypes.c_int] * 4
        f.restype = ctypes.c_size_t
    lib.etics_plan_info.argtypes = [ctypes.c_int, ctypes.c_int64] + [ctypes.c_int] * 4 + \
        [ctypes.POINTER(ctypes.c_int), ctypes.c_int]
    return lib


def unit_of(L, n, nmax, lmax, prec):
    out = (ctypes.c_int * 9)()
    assert L.etics_plan_info(1, n, nmax, lmax, prec, 0, out, 9) == 0
    return out[4]


def total(*parts):
    return sum((max(p, 1) + 255) // 256 * 256 for p in parts)


@pytest.mark.parametrize("prec", [1, 2])
@pytest.mark.parametrize("nsys,n", [(1, 1), (1, 1000), (3, 10), (16, 16_000), (256, 256), (256, 2_560_000),
                                    (100_000, 300_000)])
def test_sizes_without_padding(L, nsys, n, prec):
    for nmax in range(21):
        # the monopole alone, one slot padded to four, and the jerk's two smallest such cutoffs are
        # left out: their padding is larger than the partial sums that it may lie on
        for lmax in range(1, 15):
            K = (nmax + 1) * (lmax + 1) * (lmax + 2) // 2
            units = nsys + -(-n // unit_of(L, n, nmax, lmax, prec))
            tables = (4 * (nsys + 1), 4 * units, 16 * K * units)
            assert L.etics_batched_workspace_size(n, nsys, nmax, lmax, prec) <= \
                total(*tables, 16 * K * nsys, 8 * K * nsys, 8 * K * nsys, 24 * n), (nmax, lmax)
            if (nmax, lmax) not in ((1, 1), (1, 2)):
                assert L.etics_hermite_workspace_size(n, nsys, nmax, lmax, prec) <= \
                    total(*tables, 32 * K * nsys, *[8 * K * nsys] * 4, 96 * n), (nmax, lmax)
