"""Host build of the int8 GEMM's launch plan (tile_schedule.h, gemm_plan):
whichever tile shape and layout it takes, every tile of every product has
exactly one slot, the tiles cover the outputs, and an XCD's spread slots are
consecutive places of the sequence of tiles."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from gemm_shapes import CHAINED, SHAPES

HERE = os.path.dirname(os.path.abspath(__file__))
STAGE_BYTES = 256 * 64
PER_CU = {0: 1, 1: 2, 2: 3, 3: 4}


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = tmp_path_factory.mktemp("plan") / "libgemm_plan_host.so"
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", os.path.join(HERE, "gemm_plan_host.cpp"),
                    "-o", str(out)], check=True)
    L = ctypes.CDLL(str(out))
    I, Lg, P = ctypes.c_int, ctypes.c_long, ctypes.c_void_p
    L.t_plan.argtypes = [I, I, I, I, Lg, P]
    L.t_estimate.argtypes = [I, I, I, I, I, ctypes.c_double]
    L.t_estimate.restype = ctypes.c_double
    L.t_plan_tiles.argtypes = [I, I, I, I, I, Lg, P]
    return L


def plan(lib, rows, cols, kb, batch):
    out = np.zeros(11, dtype=np.int64)
    lib.t_plan(rows, cols, kb, batch, STAGE_BYTES, out.ctypes.data)
    return dict(zip(("shape", "tm", "tn", "mt", "nt", "deal", "chunk", "slots", "fixed", "grid", "chain"), (int(v) for v in out)))


CASES = [(1, 1, 1, 1), (96, 80, 4, 32), (500, 333, 13, 32), (1024, 1024, 16, 32), (1537, 1283, 33, 16),
         (2048, 2048, 32, 32), (3001, 3001, 40, 16), (4096, 96, 64, 32), (96, 4096, 64, 32), (4096, 4096, 64, 16),
         (2047, 2049, 129, 32),               # spread and pooled
         (8192, 8192, 128, 32), (5632, 5888, 375, 32), (16384, 33, 1, 74), (20000, 20000, 1, 64),
         (33, 20000, 2000, 2)]


@pytest.mark.parametrize("rows,cols,kb,batch", CASES)
def test_plan_covers_every_tile_once(lib, rows, cols, kb, batch):
    p = plan(lib, rows, cols, kb, batch)
    mt, nt, slots = p["mt"], p["nt"], p["slots"]
    assert (mt - 1) * p["tm"] < rows <= mt * p["tm"] and (nt - 1) * p["tn"] < cols <= nt * p["tn"]
    est = [lib.t_estimate(0, rows, cols, kb, batch, 0.0)]
    est += [lib.t_estimate(i, rows, cols, kb, batch, est[0] / 600) for i in (1, 2, 3)]
    assert est[p["shape"]] == min(est)
    t = np.zeros((8, slots, 4), dtype=np.int32)
    lib.t_plan_tiles(mt, nt, p["chunk"], p["deal"], batch, slots, t.ctypes.data)
    keys = t[t[..., 0].astype(bool)][:, 1:].astype(np.int64)
    assert (keys >= 0).all() and (keys < [batch, mt, nt]).all()
    flat = (keys[:, 0] * mt + keys[:, 1]) * nt + keys[:, 2]
    assert len(flat) == len(np.unique(flat)) == mt * nt * batch
    pool = slots // 8 if p["shape"] == 0 and kb >= 128 and slots >= 256 else 0
    assert slots - p["fixed"] == pool
    assert p["chain"] == int(p["shape"] == 0 and 5 <= kb <= 48 and slots > 32)
    assert p["grid"] == (256 if p["chain"] else 8 * (slots + (-(-slots // 12) if pool else 0)))
    narrow = p["shape"] == 0 and min(mt, nt) == 1
    assert (p["deal"] == 2) == (mt * nt < (8 if narrow else 256 * PER_CU[p["shape"]]))
    if p["deal"] == 2:
        # product-major over the XCDs in turn: the sequence of products never falls
        assert slots == -(-mt * nt * batch // 8) and (np.diff(keys[:, 0]) >= 0).all()


# rows, columns, k-stages, products of short launches; whether they are laid out spread
SHORT = [(1000, 1000, 1, 16, False), (1000, 1000, 4, 16, False), (1000, 1000, 5, 16, True), (1000, 1000, 4, 32, True),
         (1000, 1000, 2, 32, False), (700, 700, 4, 16, False), (1600, 1600, 2, 8, False), (2000, 2000, 2, 8, False),
         (2000, 2000, 1, 16, True), (1025, 300, 1, 32, True), (300, 1025, 1, 32, True), (400, 400, 4, 16, False),
         (200, 200, 4, 32, True), (700, 700, 2, 40, True), (700, 700, 2, 32, False),
         (841, 835, 4, 8, False), (690, 655, 4, 16, False), (850, 780, 4, 16, False)]


@pytest.mark.parametrize("rows,cols,kb,batch,spread", SHORT)
def test_short_launches_are_kept_flat(lib, rows, cols, kb, batch, spread):
    """Whichever layout, every tile has one slot."""
    p = plan(lib, rows, cols, kb, batch)
    assert (p["deal"] == 2) == spread
    mt, nt, slots = p["mt"], p["nt"], p["slots"]
    t = np.zeros((8, slots, 4), dtype=np.int32)
    lib.t_plan_tiles(mt, nt, p["chunk"], p["deal"], batch, slots, t.ctypes.data)
    keys = t[t[..., 0].astype(bool)][:, 1:].astype(np.int64)
    flat = (keys[:, 0] * mt + keys[:, 1]) * nt + keys[:, 2]
    assert (keys < [batch, mt, nt]).all() and len(flat) == len(np.unique(flat)) == mt * nt * batch
    assert p["grid"] == 8 * slots and p["fixed"] == slots


# rows, columns, k-stages, products of long outputs; their tile shape
LONG = [(2000, 20000, 1, 32, 1), (30000, 1000, 1, 16, 1), (2049, 20000, 1, 32, 2), (5000, 5000, 1, 32, 2),
        (2000, 20000, 2, 32, 2), (2048, 6145, 1, 32, 1), (2048, 6016, 1, 32, 2),
        (300, 60000, 1, 32, 2), (60000, 300, 1, 32, 1)]


@pytest.mark.parametrize("rows,cols,kb,batch,shape", LONG)
def test_long_outputs_of_one_stage(lib, rows, cols, kb, batch, shape):
    p = plan(lib, rows, cols, kb, batch)
    assert p["shape"] == shape and p["fixed"] == p["slots"] and p["grid"] == 8 * p["slots"]
    assert (p["mt"] - 1) * p["tm"] < rows <= p["mt"] * p["tm"] and (p["nt"] - 1) * p["tn"] < cols <= p["nt"] * p["tn"]
    assert p["slots"] * 8 >= p["mt"] * p["nt"] * batch


def test_empty_problem(lib):
    for c in [(0, 4, 4, 4), (4, 0, 4, 4), (4, 4, 0, 4), (4, 4, 4, 0)]:
        assert plan(lib, *c)["grid"] == 0


def test_sizes_take_their_shapes(lib):
    """The sizes that the GPU test runs reach every kernel."""
    for shape, sizes in SHAPES.items():
        for rows, cols, k, batch in sizes:
            assert plan(lib, rows, cols, -(-k // 64), batch)["shape"] == shape, (rows, cols, k, batch)
    for rows, cols, k, batch in CHAINED:
        assert plan(lib, rows, cols, -(-k // 64), batch)["chain"] == 1, (rows, cols, k, batch)
