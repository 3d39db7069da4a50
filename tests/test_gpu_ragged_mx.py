"""MXFP4 GEMMs with K not a multiple of 128 against the fp64 oracle: the
small-M kernel (each configuration, K splits whose last panel is 1, 2 or 3
blocks), the persistent kernel's last panel (whole and half tiles), and the
grouped form, with expert scales at any byte."""

import numpy as np
import pytest
import torch

from oracle import sharq_oracle as O
from paper_2606_26587_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_26587_amd import sharq
    return sharq


@pytest.fixture(scope="module")
def G(S):
    import gpu_util
    return gpu_util


def within(got, ref, mag, K):
    # fp32 sums of 2K exact products
    err = np.abs(got.astype(np.float64) - ref)
    assert (err <= 2 * K * 2.0 ** -24 * mag).all(), float(err.max())


@pytest.mark.parametrize("n,m", [(2, 4), (4, 8)])
@pytest.mark.parametrize("T,N,K", [
    (1, 17, 160), (16, 6200, 192), (3, 12300, 224), (2, 40, 8352),    # up to 16 rows, K split 4 to 16
    (20, 100, 1184), (32, 12300, 160),                                # two row fragments
    (40, 100, 416), (100, 1000, 1120), (257, 1000, 288), (500, 1000, 480), (1000, 1000, 672),   # several row tiles
    (300, 5000, 416), (700, 4000, 224), (1500, 5900, 288),            # the persistent kernel, with half tiles
    (40, 300, 96), (5, 40, 32),                                       # below one panel
    (400, 1000, 512), (1030, 1100, 1024),                             # whole panels on the wider small-M range
])
def test_ragged_linear(S, G, n, m, T, N, K):
    x = synth.activations(T, K, seed=T + N)
    o = O.prepare(x, synth.gamma(K, seed=3), 1e-6, n, m, "mx")
    wo = O.quantize_weight(synth.weight(N, K, seed=7), "mx")
    a, w = G.oracle_to_act(o), G.oracle_to_weight(wo)
    y = torch.full((T + 1, N + 3), float("nan"), dtype=torch.float32, device="cuda")
    S.sharq_linear(a, w, out=y[:T, :N])
    y16 = S.sharq_linear(a, w, dtype=torch.bfloat16)
    torch.cuda.synchronize()
    got = G.host(y)
    assert np.isnan(got[T]).all() and np.isnan(got[:, N:]).all(), "written outside the output"
    within(got[:T, :N], O.linear(o, wo), O.linear_abs(o, wo), K)
    assert torch.equal(y16, y[:T, :N].to(torch.bfloat16))


@pytest.mark.parametrize("T,N,K,n,m,dense", [
    (97, 4100, 2176, 2, 4, True), (128, 4100, 2048, 4, 8, True),            # 64-row tiles, dense copy: 5 + 2 and 4 panels
    (97, 4100, 2080, 2, 4, False), (97, 4100, 2176, 4, 8, False),           # compressed, ragged and whole panels
    (130, 2000, 416, 2, 4, False), (300, 1000, 416, 4, 8, False),           # 32 rows, K over 8: one panel each or none
    (100, 4100, 1280, 2, 4, True), (130, 4100, 512, 2, 4, False),           # 32 rows, K over 4
])
def test_row_tiles(S, G, T, N, K, n, m, dense):
    """Above 32 rows: each order of loads and MFMAs of the small-M kernel, with panel counts per
    wavefront that are odd, even, one and none."""
    o = O.prepare(synth.activations(T, K, seed=T + N), synth.gamma(K, seed=3), 1e-6, n, m, "mx")
    wo = O.quantize_weight(synth.weight(N, K, seed=7), "mx")
    a, w = G.oracle_to_act(o, dense_backbone=dense), G.oracle_to_weight(wo)
    if dense:
        a.sp_codes = a.sp_meta = None
    y = torch.full((T + 1, N + 3), float("nan"), dtype=torch.float32, device="cuda")
    S.sharq_linear(a, w, out=y[:T, :N])
    torch.cuda.synchronize()
    got = G.host(y)
    assert np.isnan(got[T]).all() and np.isnan(got[:, N:]).all(), "written outside the output"
    rows = np.unique(np.concatenate([np.arange(0, T, 7), np.arange(T - 5, T)]))
    within(got[rows, :N], O.linear(o, wo, rows=rows), O.linear_abs(o, wo, rows=rows), K)


@pytest.mark.parametrize("gather", [True, False])
@pytest.mark.parametrize("N,K", [(328, 416), (201, 416), (201, 544), (130, 96)])
def test_ragged_grouped(S, G, gather, N, K):
    E, topk, T = 5, 2, 300
    ri, off = synth.router_topk(T, E, topk, seed=3)
    total = int(off[-1])
    rows = T if gather else total
    o = O.prepare(synth.activations(rows, K, seed=5), None, 1e-6, 2, 4, "mx")
    ws = [O.quantize_weight(synth.weight(N, K, seed=20 + e), "mx") for e in range(E)]
    w = S.stack_weights([G.oracle_to_weight(x) for x in ws])
    y = S.sharq_linear_grouped(G.oracle_to_act(o), torch.from_numpy(ri).cuda() if gather else None,
                               torch.from_numpy(off).cuda(), total, w, dtype=torch.float32)
    torch.cuda.synchronize()
    got = G.host(y)
    for e in range(E):
        s = slice(int(off[e]), int(off[e + 1]))
        r = ri[s] if gather else np.arange(s.start, s.stop)
        within(got[s], O.linear(o, ws[e], rows=r), O.linear_abs(o, ws[e], rows=r), K)
