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
// {nf, gx, gy, full, grid, rows of a tile} of the plan
void plan_mx8(int64_t M, int N, int cus, int* out, int) {
  const Plan8 p = plan8(M, N, cus);
  out[0] = p.nf, out[1] = p.gx, out[2] = p.gy, out[3] = p.full, out[4] = p.grid, out[5] = kRows8;
}
void plan_16(int64_t M, int N, int cus, int* out, int form) {
  const Plan16 p = plan16(M, N, form, cus);
  out[0] = p.nf, out[1] = p.gx, out[2] = p.gy, out[3] = p.full, out[4] = p.grid, out[5] = p.rows;
}
// {small-M kernel or not, mf, nb, ks of its configuration above 32 rows}
void plan_skinny(int64_t M, int N, int K, int form, int cus, int* out) {
  const SkinnyWide w = skinny_wide(M, N, K, form, cus);
  out[0] = use_skinny(M, N, K, form, form, cus), out[1] = w.mf, out[2] = w.nb, out[3] = w.ks;
}
void plan_skinny16(int64_t M, int N, int K, int form, int cus, int* out) {
  const Wide16 w = wide16(M, N, K, form, cus);
  out[0] = use_skinny16(M, N, K, form, cus), out[1] = w.mf, out[2] = w.nb, out[3] = w.ks;
}
// {few-row kernel or not, column fragments, K splits} of a grouped call
void plan_grouped(int64_t total, int E, int N, int K, int cus, int* out) {
  const GroupedCfg c = grouped_cfg(total, E, N, K, cus);
  out[0] = use_grouped_skinny(total, E, N, cus), out[1] = c.nb, out[2] = c.ks;
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
        f.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.POINTER(ctypes.c_int), ctypes.c_int]
    for f in (L.plan_skinny, L.plan_skinny16, L.plan_grouped):
        f.argtypes = [ctypes.c_int64] + [ctypes.c_int] * 4 + [ctypes.POINTER(ctypes.c_int)]
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


@pytest.mark.parametrize("name,form", [("plan_mx8", 0)] + [("plan_16", f) for f in range(4)])
@pytest.mark.parametrize("cus", [256, 64, 38])
def test_rounds(plan, name, form, cus):
    out = (ctypes.c_int * 6)()
    odd = 0
    for M, N in SIZES:
        getattr(plan, name)(M, N, cus, out, form)
        nf, gx, gy, full, grid, rows = out
        assert gx == -(-N // (64 * nf)) and gy == -(-M // rows)
        odd += full % 8 != 0
        assert rounds_of(plan, full, gx, gy, grid) == -(-full // grid), (M, N, nf, full, grid)
        rest = gx * gy - full   # a last round of half tiles
        assert rest == 0 or (nf == 4 and full % cus == 0 and 2 * rest <= grid)
    assert odd > 20   # tile counts that are no multiple of 8 are among them


@pytest.mark.parametrize("form,M,N,tile", [
    # the tiles that tests/test_gpu_linear16.py runs (forms: NVFP4 dense, 2:4, 4:8, HiF4): rows, columns, halves
    *[(f, 2100, 1992, (256, 128, False)) for f in range(3)], (3, 2100, 1992, (128, 256, False)),
    *[(f, 2040, 6104, (256, 192, False)) for f in range(4)], *[(f, 2290, 7101, (256, 256, False)) for f in range(4)],
    (0, 2300, 8008, (256, 256, True)), (3, 2300, 8008, (256, 192, False)), *[(f, 2300, 22400, (256, 256, True)) for f in (1, 2, 3)],
    *[(f, 300, 17000, (128, 256, False)) for f in range(4)],
    *[(f, 384, 37888, (128, 256, False)) for f in range(4)],
])
def test_tiles(plan, form, M, N, tile):
    out = (ctypes.c_int * 6)()
    plan.plan_16(M, N, 256, out, form)
    assert (out[5], 64 * out[0], out[3] < out[1] * out[2]) == tile


DENSE, C24, C48 = 0, 1, 2


@pytest.mark.parametrize("form,M,N,K,small", [
    # (us on one card, the weight streamed: small-M kernel / main kernel)
    (DENSE, 64, 18944, 1024, False),     # 11.7 / 10.0
    (DENSE, 768, 2048, 768, False),      # 9.7 / 8.8
    (C48, 192, 7168, 2048, False),       # 22.5 / 18.1
    (C48, 768, 2048, 768, False),        # 13.0 / 10.8
    (C48, 48, 18944, 3584, False),       # 35.8 / 26.6
    (C24, 320, 4096, 14336, True),       # 79.5 / 84.6
    (C48, 96, 4096, 4096, True),         # 13.0 / 28.8
    (DENSE, 256, 4096, 14336, True),     # 36.8 / 70.6
    (DENSE, 512, 1024, 4096, True),      # 9.3 / 23.2
    (DENSE, 32, 28672, 4096, True), (C48, 1, 64, 128, True),    # up to 32 rows always
    (DENSE, 2048, 4096, 4096, False), (C24, 33, 64, 96, False), (DENSE, 5000, 64, 128, False),
])
def test_small_m_choice(plan, form, M, N, K, small):
    out = (ctypes.c_int * 4)()
    plan.plan_skinny(M, N, K, form, 256, out)
    assert bool(out[0]) == small, (M, N, K)


@pytest.mark.parametrize("form,M,N,K,cfg", [
    # 37 us; 42 and more with the other configurations
    (DENSE, 192, 4096, 14336, (4, 4, 4)), (DENSE, 256, 4096, 14336, (4, 4, 4)),
    # what tests/test_gpu_ragged_mx.py::test_row_tiles runs
    (DENSE, 97, 4100, 2176, (4, 4, 4)), (DENSE, 128, 4100, 2048, (4, 4, 4)), (DENSE, 100, 4100, 1280, (2, 4, 4)),
    (C24, 97, 4100, 2080, (4, 4, 4)), (C24, 130, 2000, 416, (2, 4, 8)), (C24, 130, 4100, 512, (2, 4, 4)),
    (C48, 97, 4100, 2176, (4, 4, 4)), (C48, 300, 1000, 416, (2, 4, 8)),
])
def test_small_m_configuration(plan, form, M, N, K, cfg):
    out = (ctypes.c_int * 4)()
    plan.plan_skinny(M, N, K, form, 256, out)
    assert tuple(out) == (1, *cfg)


NV_DENSE, NV24, NV48, HIF4 = 0, 1, 2, 3


@pytest.mark.parametrize("form,M,N,K,small", [
    # (us on one card, the weight streamed: small-M kernel / prefill kernel)
    (NV48, 1024, 6144, 4096, False),
    (NV24, 4096, 2048, 768, False),
    (NV48, 1792, 2048, 768, False),      # 54 / 29
    (NV48, 2560, 2048, 768, False),
    (NV48, 768, 5000, 2080, True),       # 71 with 32 x 64 columns / 104, K not a multiple of 128
    (NV_DENSE, 256, 6144, 4096, True),   # 32 / 75
    (NV48, 128, 4096, 4096, True), (HIF4, 96, 4096, 4096, True), (NV24, 64, 28672, 4096, True),
    (NV_DENSE, 32, 37888, 3584, True), (HIF4, 1, 64, 64, True), (NV24, 4097, 64, 128, False),
])
def test_small_m_choice_16_bit(plan, form, M, N, K, small):
    out = (ctypes.c_int * 4)()
    plan.plan_skinny16(M, N, K, form, 256, out)
    assert bool(out[0]) == small, (M, N, K)


@pytest.mark.parametrize("form,M,N,K,cfg", [
    # what tests/test_gpu_skinny16.py::test_row_tiles runs
    (NV_DENSE, 97, 6200, 256, (2, 4, 4)), (NV24, 300, 3000, 256, (2, 4, 4)), (NV48, 100, 4100, 576, (2, 4, 4)),
    (NV48, 300, 3000, 256, (4, 4, 4)), (HIF4, 97, 6200, 256, (4, 4, 4)), (HIF4, 100, 4100, 448, (4, 4, 4)),
    (NV_DENSE, 257, 500, 128, (2, 2, 8)), (NV24, 128, 300, 448, (2, 1, 8)),
])
def test_small_m_configuration_16_bit(plan, form, M, N, K, cfg):
    out = (ctypes.c_int * 4)()
    plan.plan_skinny16(M, N, K, form, 256, out)
    assert tuple(out) == (1, *cfg)


def test_small_m_configurations_are_built(plan):
    """Over 32 rows no form is given a configuration that it is not built for (64 x 64: NVFP4 4:8 and HiF4)."""
    out = (ctypes.c_int * 4)()
    for form in range(4):
        for M in (33, 64, 128, 257, 1000, 4096):
            for N in (1, 100, 1000, 4100, 12000, 50000, 1 << 20):
                for K in (128, 4096, 16384) if form == NV_DENSE else (64, 128, 576, 4096, 16384):
                    plan.plan_skinny16(M, N, K, form, 256, out)
                    assert tuple(out)[1:] in {(2, 1, 8), (2, 2, 8), (2, 4, 4), (4, 4, 4)}
                    assert form >= 2 or out[1] == 2


@pytest.mark.parametrize("total,E,N,K,want", [
    # a single expert with all rows has to be no slower than on the persistent kernel: 64 rows 42 / 21 us
    (64, 8, 28672, 4096, None), (8, 8, 28672, 4096, (4, 4)),
    (512, 32, 1536, 4096, None), (512, 16, 4096, 1024, None),
    # many experts
    (512, 128, 2048, 768, (4, 2)), (512, 128, 1536, 2048, (4, 4)), (1024, 256, 512, 1024, (4, 2)),
    (768, 128, 2048, 768, None),
    # few column groups
    (64, 8, 2048, 4096, (2, 4)), (128, 8, 2048, 4096, (4, 4)), (8, 8, 4096, 14336, (2, 4)),
    # what tests/test_gpu_grouped_small.py runs
    (81, 6, 200, 1664, (4, 4)), (81, 6, 200, 1632, (4, 4)), (3, 3, 70, 1600, (2, 4)), (74, 8, 200, 256, (4, 2)),
    (11, 4, 330, 1184, (2, 4)), (512, 130, 384, 256, (4, 2)),
    # more threads than a launch may have
    (8, 1024, 1 << 21, 32, None), (8, 8, 1 << 28, 32, None),
])
def test_grouped_choice(plan, total, E, N, K, want):
    out = (ctypes.c_int * 3)()
    plan.plan_grouped(total, E, N, K, 256, out)
    assert (tuple(out)[1:] if out[0] else None) == want


@pytest.mark.parametrize("name,forms", [("plan_skinny", 3), ("plan_skinny16", 4)])
def test_launches_stay_below_2_32_threads(plan, name, forms):
    """Wide layers with few rows, which the tiled kernels take (N 2^30, K 32, one row: 18 GB of weight)."""
    out = (ctypes.c_int * 4)()
    for form in range(forms):
        for M in (1, 16, 17, 32, 33, 100, 1000, 4096):
            for logn in range(10, 31):
                for N in (1 << logn, (1 << logn) - 1):
                    for K in (128, 256, 4096):
                        getattr(plan, name)(M, N, K, form, 256, out)
                        small, mf, nb, ks = out
                        if M > 32 and small:
                            assert -(-N // (16 * nb)) * -(-M // (16 * mf)) * 64 * ks < 1 << 32
                        if M <= 32:
                            assert small == (8 * N < 1 << 32 and N <= 1 << 28)
