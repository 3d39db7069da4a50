"""The small-M kernel of the formats on 16-bit MFMA (NVFP4, HiF4) against the
fp64 oracle, where it can go wrong: row and column counts around its fragment
and row-tile edges, K below a panel, ragged and across its K splits, strided
output rows, each backbone form.  The prefill kernels' ragged-K forms, which
small shapes no longer reach, are run at a shape they still serve."""

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


def check(S, G, fmt, T, N, K, n, m, dense):
    x = synth.activations(T, K, seed=T + N)
    o = O.prepare(x, synth.gamma(K, seed=3), 1e-6, n, m, fmt)
    wo = O.quantize_weight(synth.weight(N, K, seed=N + 7), fmt)
    a, w = G.oracle_to_act(o, dense_backbone=dense), G.oracle_to_weight(wo)
    y = torch.full((T + 1, N + 3), float("nan"), dtype=torch.float32, device="cuda")
    S.sharq_linear(a, w, out=y[:T, :N])
    y16 = S.sharq_linear(a, w, dtype=torch.bfloat16)
    torch.cuda.synchronize()
    got = G.host(y)
    assert np.isnan(got[T]).all() and np.isnan(got[:, N:]).all(), "written outside the output"
    got = got[:T, :N]
    err = np.abs(got.astype(np.float64) - O.linear(o, wo))
    # fp32 sums of 2K exact products, and two roundings of the tensor scales' product and its use
    bound = (2 * K + 2) * 2.0 ** -24 * O.linear_abs(o, wo)
    assert (err <= bound).all(), (fmt, T, N, K, float((err - bound).max()))
    assert torch.equal(y16, y[:T, :N].to(torch.bfloat16))


@pytest.mark.parametrize("T,N,K", [
    (1, 1, 64), (3, 17, 128), (16, 31, 192), (5, 3100, 320),      # one row fragment; 1, 2 and 4 column fragments
    (2, 12300, 128), (1, 48, 8192), (1, 6150, 4096),               # K splits of 4, 8 and 16
    (17, 33, 64), (33, 65, 1216), (128, 300, 448), (40, 6200, 256),   # two row fragments, several row tiles
    (129, 70, 192), (200, 1000, 576), (257, 500, 128),             # one row past a tile
])
@pytest.mark.parametrize("fmt,n,m,dense", [("nv", 2, 4, False), ("nv", 4, 8, False), ("nv", 4, 8, True),
                                           ("hif4", 2, 4, False)])
def test_skinny16(S, G, fmt, n, m, dense, T, N, K):
    if dense and K % 128:
        pytest.skip("the dense backbone copy needs K a multiple of 128")
    check(S, G, fmt, T, N, K, n, m, dense)


@pytest.mark.parametrize("fmt,T,N,K,n,m,dense", [
    ("nv", 97, 6200, 256, 4, 8, True), ("nv", 300, 3000, 256, 2, 4, False), ("nv", 100, 4100, 576, 4, 8, False),   # 32 x 64
    ("nv", 300, 3000, 256, 4, 8, False), ("hif4", 97, 6200, 256, 2, 4, False), ("hif4", 100, 4100, 448, 2, 4, False),   # 64 x 64
])
def test_row_tiles(S, G, fmt, T, N, K, n, m, dense):
    """The wider configurations above 32 rows, with a last row tile of one row or more and ragged columns."""
    check(S, G, fmt, T, N, K, n, m, dense)


@pytest.mark.parametrize("T,N,K", [(4, 40, 32), (20, 40, 96), (130, 40, 160)])
def test_skinny16_odd_blocks_nv(S, G, T, N, K):
    check(S, G, "nv", T, N, K, 2, 4, False)


@pytest.mark.parametrize("fmt", ["nv", "hif4"])
@pytest.mark.parametrize("K", [416, 512])
def test_prefill_kernels_mid_shape(S, G, fmt, K):
    if fmt == "hif4" and K == 416:
        K = 448
    check(S, G, fmt, 2100, 3000, K, 2, 4, False)
