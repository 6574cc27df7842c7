"""Host build of the choice of K1's kernels (scale_rules.h): what a short row
costs the direct kernel, that many such rows are left to the scans, and which
scans share a launch."""
import ctypes
import os
import subprocess

import pytest

from scale_shapes import RESUMMED_K, RESUMMED_K_RANK2, SCANS as SCANNED_SIZES

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = tmp_path_factory.mktemp("rules") / "libscale_rules_host.so"
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-fPIC", "-shared",
                    os.path.join(HERE, "scale_rules_host.cpp"), "-o", str(out)], check=True)
    L = ctypes.CDLL(str(out))
    I, Lg = ctypes.c_int, ctypes.c_long
    L.t_direct_hold.argtypes = [Lg, I]
    L.t_direct_rule.argtypes = [Lg, I, Lg, I, Lg, Lg, Lg]
    L.t_row_cpt.argtypes = [I, I]
    L.t_scans_together.argtypes = [ctypes.POINTER(Lg)] * 2
    return L


def test_held_entries_follow_the_row(lib):
    """A held form covers the row (64 threads to a row), and beyond the shortest
    it is less than four times as long; longer rows and two sources are read
    again."""
    for k in range(1025):
        h = lib.t_direct_hold(k, 0)
        assert h in (1, 4, 8, 16) and 64 * h >= k
        assert h == 1 or 64 * h < 4 * k
        assert lib.t_direct_hold(k, 1) == 0
    assert lib.t_direct_hold(1025, 0) == 0


# entry bytes, Cauchy-Schwarz rule, k, two sources, rows of A and of B that are
# rows of a column-major matrix, columns
DIRECT = [(16, 1, 200, 0, 96, 0, 80), (16, 0, 777, 0, 500, 0, 333), (16, 1, 1024, 0, 1024, 0, 1024),
          (8, 0, 2051, 0, 1537, 1283, 0), (16, 1, 16, 0, 16384, 0, 1), (16, 0, 16, 0, 24576, 0, 0),
          (8, 1, 64, 0, 65536, 0, 8192), (16, 1, 64, 0, 32, 0, 65536), (8, 0, 16384, 0, 4, 0, 0),
          (16, 1, 64, 1, 4096, 0, 0), (16, 0, 64, 1, 16384, 0, 0), (8, 0, 0, 0, 5, 0, 7),
          (16, 1, 16, 0, 131072, 0, 8192), (8, 1, 1024, 0, 8000, 0, 0), (8, 1, 4000, 0, 1000, 0, 1000),
          (8, 1, 4000, 0, 1000, 1000, 0), (8, 0, 8000, 0, 600, 0, 0), (16, 1, 16384, 0, 64, 0, 64),
          (8, 1, 3584, 0, 0, 0, 1600), (8, 0, 16384, 0, 0, 0, 64), (8, 1, 5500, 1, 500, 0, 0)]
SCANS = [(16, 1, 16, 0, 262144, 0, 32), (16, 0, 16, 0, 262144, 0, 32), (8, 1, 16, 0, 262144, 0, 32),
         (8, 1, 64, 0, 65536, 0, 32), (16, 1, 8, 0, 65536, 0, 2048), (8, 0, 32, 0, 65536, 0, 64),
         (16, 1, 64, 1, 8192, 0, 0), (8, 1, 64, 1, 16384, 0, 0), (8, 0, 0, 0, 1 << 27, 0, 1), (16, 1, 16385, 0, 4, 0, 4),
         (16, 0, 8193, 1, 4, 0, 0), (16, 0, 2048, 0, 2048, 0, 2048), (8, 1, 8000, 0, 600, 0, 0),
         (8, 1, 3000, 0, 0, 1500, 8), (16, 1, 4100, 0, 1100, 0, 8), (8, 1, 5500, 1, 800, 0, 0), (8, 1, 1100, 0, 8000, 0, 0),
         (16, 1, 3585, 0, 0, 0, 2), (8, 1, 16384, 0, 0, 0, 128)]


def direct(lib, e, cs, k, two, ra, rb, cols):
    return lib.t_direct_rule(e, cs, k, two, ra + rb, max(ra, rb), cols)


@pytest.mark.parametrize("case", DIRECT)
def test_direct_calls(lib, case):
    assert direct(lib, *case) == 1


@pytest.mark.parametrize("case", SCANS)
def test_scanned_calls(lib, case):
    """Many short rows (a wave each in the direct kernel, a lane in the row
    scans), long rows, operands beyond the caches; under the Cauchy-Schwarz
    rule large operands read in rows, and long columns."""
    assert direct(lib, *case) == 0


MB = 1 << 20
ROWS32, ROWS16 = (0, 32, 0, 1, 256 * MB, 2048), (0, 16, 0, 0, 64 * MB, 2048)
# rows beside columns, row scans, column scans; the smaller of two loads follows
TOGETHER = [(ROWS32, (1, 4, 0, 0, 6 * MB, 192)), (ROWS32, (1, 4, 0, 0, 2 * MB, 2048)), (ROWS16, (1, 4, 0, 0, 64 * MB, 8192)),
            ((1, 4, 1, 0, 6 * MB, 192), ROWS32), (ROWS32, (0, 32, 0, 1, 200 * MB, 4096)), (ROWS16, ROWS16),
            ((1, 4, 1, 0, 20 * MB, 99), (1, 4, 1, 0, 40 * MB, 99)), ((1, 4, 0, 1, 200 * MB, 99), (1, 4, 0, 0, 15 * MB, 99))]
APART = [(ROWS32, (1, 4, 0, 0, 2 * MB, 2049)), ((1, 4, 0, 0, 8 * MB, 8192), ROWS32),      # many short columns
         (ROWS32, (1, 4, 0, 0, 16 * MB, 512)), (ROWS32, ROWS16), ((1, 4, 1, 0, 20 * MB, 99), (1, 4, 0, 0, 20 * MB, 99)),
         (ROWS16, (1, 4, 0, 1, 200 * MB, 99))]


@pytest.mark.parametrize("a,b,want", [(*c, 1) for c in TOGETHER] + [(*c, 0) for c in APART])
def test_scans_of_two_operands(lib, a, b, want):
    v = ctypes.c_long * 6
    assert lib.t_scans_together(v(*a), v(*b)) == want


@pytest.mark.parametrize("call,m,n,k,ta,tb,cpt,nt", SCANNED_SIZES)
def test_sizes_of_the_scan_tests(lib, call, m, n, k, ta, tb, cpt, nt):
    """The GPU tests of the scans reach them, in the form they name."""
    e = 16 if call == "z" else 8
    ra, rb = (m if ta == "N" else 0), (n if tb != "N" else 0)
    assert direct(lib, e, 1, k, 0, ra, rb, m + n - ra - rb) == 0
    assert (lib.t_row_cpt(m, k) if ta == "N" else 0) == cpt
    assert (e * m * k >= 128 << 20) == nt


def test_sizes_of_the_resummed_tests(lib):
    assert direct(lib, 8, 1, RESUMMED_K, 0, 1, 0, 0) == 0
    assert direct(lib, 8, 1, RESUMMED_K_RANK2, 1, 1, 0, 0) == 0
