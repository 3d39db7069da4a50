"""The grouped MXFP4 GEMM with few rows per expert against the fp64 oracle:
experts with no rows, one, a full tile and several tiles (found by a scan, here
over more than 64 experts too), row maps, ragged K (expert scales at any byte),
each configuration (columns, K splits) and each backbone form."""

import numpy as np
import pytest
import torch

from oracle import sharq_oracle as O
from paper_2606_26587_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,N,K,counts", [
    (8, 200, 256, [0, 1, 16, 17, 5, 0, 33, 2]),            # few column groups, up to 24 rows a mean
    (4, 330, 1184, [3, 0, 7, 1]),
    (4, 64, 512, [90, 0, 1, 0]),
    (64, 776, 384, [0, 1, 17, 3] * 16),                    # many column groups
    (96, 520, 160, [40, 2] + [0, 2] * 46 + [70, 33]),
    (130, 384, 256, [0] * 70 + [300] + [0] * 57 + [212, 0]),   # 512 rows, the most
    (4, 64, 64, [0, 0, 0, 33]),                            # less than a panel
    (4, 64, 256, [0, 0, 0, 33]),
    (6, 200, 1664, [20, 0, 3, 40, 1, 17]),                 # K in four parts, 13 panels
    (6, 200, 1632, [20, 0, 3, 40, 1, 17]),
    (3, 70, 1600, [1, 0, 2]),                              # 32 columns
])
@pytest.mark.parametrize("gather", [True, False])
@pytest.mark.parametrize("n,m,dense", [(2, 4, False), (4, 8, False), (4, 8, True)])
def test_grouped_small(E, N, K, counts, gather, n, m, dense):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if dense and K % 128:
        pytest.skip("the dense backbone copy needs K a multiple of 128")
    import gpu_util as G
    from paper_2606_26587_amd import sharq as S
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    total = int(off[-1])
    rng = np.random.default_rng(E + K)
    rows = 40 if gather else total
    ri = rng.integers(0, rows, size=total).astype(np.int32) if gather else np.arange(total)
    o = O.prepare(synth.activations(rows, K, seed=5), None, 1e-6, n, m, "mx")
    ws = [O.quantize_weight(synth.weight(N, K, seed=20 + e), "mx") for e in range(4)]
    w = S.stack_weights([G.oracle_to_weight(ws[e % 4]) for e in range(E)])
    act, idx = G.oracle_to_act(o, dense_backbone=dense), torch.from_numpy(ri).cuda() if gather else None
    offs = torch.from_numpy(off).cuda()
    y = torch.full((total + 1, N + 4), float("nan"), dtype=torch.float32, device="cuda")
    S.sharq_linear_grouped(act, idx, offs, total, w, out=y[:total, :N])
    y16 = S.sharq_linear_grouped(act, idx, offs, total, w, dtype=torch.bfloat16)
    torch.cuda.synchronize()
    got = G.host(y)
    assert np.isnan(got[total]).all() and np.isnan(got[:, N:]).all(), "written outside the output"
    assert torch.equal(y16, y[:total, :N].to(torch.bfloat16))
    for e in range(E):
        s = slice(int(off[e]), int(off[e + 1]))
        r = ri[s]
        err = np.abs(got[s, :N].astype(np.float64) - O.linear(o, ws[e % 4], rows=r))
        # fp32 sums of 2K exact products
        assert (err <= 2 * K * 2.0 ** -24 * O.linear_abs(o, ws[e % 4], rows=r)).all(), e
