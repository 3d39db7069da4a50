"""The 8-wavefront MXFP4 kernel (dense backbone copy, several rounds of
tiles): bit-identical to the 4-wavefront kernel, which the compressed backbone
runs on, at each tile width, with ragged rows and columns, half tiles, K of one
panel and up, each output type and strided output rows."""

import numpy as np
import pytest
import torch

from oracle import sharq_oracle as O
from paper_2606_26587_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,N,K", [
    (2041, 6104, 128),     # 192 columns
    (2048, 6144, 384),
    (4090, 4099, 256),     # 256 columns, odd rows
    (2300, 8008, 512),     # 256 columns and half tiles
    (2048, 28672, 640),
])
def test_mx8_equals_the_compressed_form(T, N, K):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util as G
    from paper_2606_26587_amd import sharq as S
    x, g = G.dev_bf16(synth.activations(T, K, seed=T + N)), G.dev_bf16(synth.gamma(K, seed=3))
    wo = O.quantize_weight(synth.weight(N, K, seed=7), "mx")
    w = G.oracle_to_weight(wo)
    d = S.sharq_prepare(x, g, 1e-6, out=S.alloc_act(T, K, dense_only=True))
    c = S.sharq_prepare(x, g, 1e-6)
    for dt in (torch.float32, torch.bfloat16):
        yd = torch.full((T + 1, N + 8), float("nan"), dtype=dt, device="cuda")
        S.sharq_linear(d, w, out=yd[:T, :N])
        yc = S.sharq_linear(c, w, dtype=dt)
        torch.cuda.synchronize()
        assert bool(torch.isnan(yd[T]).all()) and bool(torch.isnan(yd[:, N:]).all()), "written outside the output"
        assert torch.equal(yd[:T, :N], yc)
    rows = np.array([0, 1, 31, 32, 255, 256, T // 2, T - 1])
    o = G.act_to_oracle(c)
    err = np.abs(G.host(yc.float())[rows].astype(np.float64) - O.linear(o, wo, rows=rows))
    # fp32 sums of 2K exact products, then one rounding to bf16
    ref = np.abs(O.linear(o, wo, rows=rows))
    assert (err <= 2 * K * 2.0 ** -24 * O.linear_abs(o, wo, rows=rows) + 2.0 ** -8 * ref).all()
