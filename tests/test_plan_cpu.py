"""The persistent GEMM kernels' launch plans and tile numbering
(csrc/sharq_plan.hpp, compiled for the host) over sizes whose tile counts are
and are not multiples of 8: every tile is computed once, and no workgroup gets
more tiles than the rounds that the plan counts."""

import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#include "sharq_plan.hpp"
using namespace sharq;
extern "C" {
// {nf, gx, gy, full, grid} of the plan
void plan_mx8(int64_t M, int N, int cus, int* out) {
  const Plan8 p = plan8(M, N, cus);
  out[0] = p.nf, out[1] = p.gx, out[2] = p.gy, out[3] = p.full, out[4] = p.grid;
}
void plan_16(int64_t M, int N, int cus, int* out) {
  const Plan16 p = plan16(M, N, cus);
  out[0] = p.nf, out[1] = p.gx, out[2] = p.gy, out[3] = p.full, out[4] = p.grid;
}
// row and column tile of every id in [0, units)
void walk(int units, int gx, int gy, int* mt, int* nt) {
  for (int id = 0; id < units; ++id) tile_in_groups(xcd_unit(id, units), gx, gy, mt[id], nt[id]);
}
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "shim.cpp").write_text(SHIM)
    so = str(d / "shim.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2606_26587_amd", "csrc"), str(d / "shim.cpp"), "-o", so], check=True)
    L = ctypes.CDLL(so)
    for f in (L.plan_mx8, L.plan_16):
        f.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.POINTER(ctypes.c_int)]
    return L


SIZES = [(M, N) for N in (1024, 3584, 4096, 4608, 5120, 6104, 7168, 8008, 18944, 28672)
         for M in list(range(256, 4097, 256)) + [300, 1111, 2041, 2300, 4090]]


def rounds_of(L, units, gx, gy, grid):
    """The largest number of tiles of one workgroup; every tile exactly once."""
    mt, nt = (np.full(units, -1, np.int32) for _ in range(2))
    as_p = [v.ctypes.data_as(ctypes.POINTER(ctypes.c_int)) for v in (mt, nt)]
    L.walk(units, gx, gy, *as_p)
    assert mt.min() >= 0 and mt.max() < gy and nt.min() >= 0 and nt.max() < gx
    assert np.unique(nt.astype(np.int64) * gy + mt).size == units
    return int(np.bincount(np.arange(units) % grid, minlength=grid).max())


@pytest.mark.parametrize("name", ["plan_mx8", "plan_16"])
@pytest.mark.parametrize("cus", [256, 64, 38])
def test_rounds(plan, name, cus):
    out = (ctypes.c_int * 5)()
    odd = 0
    for M, N in SIZES:
        getattr(plan, name)(M, N, cus, out)
        nf, gx, gy, full, grid = out
        assert gx == -(-N // (64 * nf)) and gy == -(-M // 256)
        odd += full % 8 != 0
        assert rounds_of(plan, full, gx, gy, grid) == -(-full // grid), (M, N, nf, full, grid)
        rest = gx * gy - full   # a last round of half tiles
        assert rest == 0 or (nf == 4 and full % cus == 0 and 2 * rest <= grid)
    assert odd > 20   # tile counts that are no multiple of 8 are among them
