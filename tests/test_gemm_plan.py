"""Host build of the int8 GEMM's launch plan (tile_schedule.h, gemm_plan): on
both sides of the line between the spread layout and the product-major one,
every tile of every product has exactly one slot, and spread slots keep an
XCD's tiles in consecutive places of the sequence."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
STAGE_BYTES = 256 * 64


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = tmp_path_factory.mktemp("plan") / "libgemm_plan_host.so"
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", os.path.join(HERE, "gemm_plan_host.cpp"),
                    "-o", str(out)], check=True)
    L = ctypes.CDLL(str(out))
    I, Lg, P = ctypes.c_int, ctypes.c_long, ctypes.c_void_p
    L.t_plan.argtypes = [I, I, I, I, Lg, P]
    L.t_plan_tiles.argtypes = [I, I, I, I, I, Lg, P]
    return L


@pytest.mark.parametrize("mt,nt,kb,batch", [
    (1, 1, 1, 1), (1, 1, 4, 32), (2, 2, 13, 32), (4, 4, 16, 32), (7, 6, 33, 16), (8, 8, 32, 32), (12, 12, 40, 16),
    (7, 1, 5, 32), (1, 8, 5, 32), (16, 1, 64, 32), (2, 127, 3, 74), (15, 17, 64, 5), (16, 16, 64, 16), (17, 16, 64, 16),
    (8, 8, 129, 32),                      # spread and pooled
    (0, 4, 4, 4), (4, 4, 0, 4)])
def test_plan_covers_every_tile_once(lib, mt, nt, kb, batch):
    out = np.zeros(5, dtype=np.int64)
    lib.t_plan(mt, nt, kb, batch, STAGE_BYTES, out.ctypes.data)
    deal, chunk, slots, fixed, grid = (int(v) for v in out)
    if mt * nt * kb * batch == 0:
        assert grid == 0
        return
    assert (deal == 2) == (mt * nt < (256 if min(mt, nt) > 1 else 8))
    t = np.zeros((8, slots, 4), dtype=np.int32)
    lib.t_plan_tiles(mt, nt, chunk, deal, batch, slots, t.ctypes.data)
    keys = [tuple(k[1:]) for k in t.reshape(-1, 4) if k[0]]
    assert len(keys) == len(set(keys)) == mt * nt * batch
    assert all(0 <= p < batch and 0 <= i < mt and 0 <= j < nt for p, i, j in keys)
    pool = slots // 8 if kb >= 128 and slots >= 256 else 0
    assert slots - fixed == pool and grid == 8 * (slots + (-(-slots // 12) if pool else 0))
    if deal == 2:
        assert slots == -(-mt * nt * batch // 8)
        # product-major over the XCDs in turn: the sequence of products never falls
        p = t[..., 1][t[..., 0].astype(bool)]
        assert (np.diff(p) >= 0).all()
