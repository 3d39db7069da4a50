"""The NVFP4 per-tensor scale of the preparation (its amax pre-pass) bit for
bit: row lengths around the pre-pass's wavefront splits, row counts that loop
over its workgroups, and the sources it reads."""

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


def bits(v):
    return np.asarray(v, np.float32).view(np.uint32)


@pytest.mark.parametrize("T,K", [(1, 32), (3, 2048), (5, 2080), (2, 4096), (3, 4128), (1, 8192), (2, 8224), (3, 16384),
                                 (4300, 64), (2100, 2112), (1030, 4160)])
@pytest.mark.parametrize("src", ["plain", "norm", "residual", "silu"])
def test_tensor_scale(S, G, T, K, src):
    x = synth.activations(T, K, seed=T + K, massive=False)
    # the largest magnitude in the last row's last block, so that a lost part would show
    x[-1, -1] = synth.f32_to_bf16_bits(np.float32([300.0]))[0]
    x2 = synth.activations(T, K, seed=T + K + 1, massive=False)
    g = synth.gamma(K, seed=K)
    if src == "plain":
        a = S.sharq_prepare(G.dev_bf16(x), None, 1e-6, 2, 4, "nv")
        y = O.bf16_bits_to_f32(x)
    elif src == "norm":
        a = S.sharq_prepare(G.dev_bf16(x), G.dev_bf16(g), 1e-6, 2, 4, "nv")
        y = O.rmsnorm(O.bf16_bits_to_f32(x), O.bf16_bits_to_f32(g), 1e-6)
    elif src == "residual":
        a, _ = S.sharq_prepare_residual(G.dev_bf16(x), G.dev_bf16(x2), G.dev_bf16(g), 1e-6, 2, 4, "nv")
        y = O.rmsnorm(O.bf16_bits_to_f32(O.residual_add_bf16(x, x2)), O.bf16_bits_to_f32(g), 1e-6)
    else:
        a = S.sharq_prepare_silu_mul(G.dev_bf16(x), G.dev_bf16(x2), 2, 4, "nv")
        y = O.bf16_bits_to_f32(O.silu_mul_bf16(x, x2))
    torch.cuda.synchronize()
    y = y[0] if isinstance(y, tuple) else y
    want = np.float32(np.abs(y).max()) / np.float32(2688.0)
    assert bits(G.host(a.tensor_scale)[0]) == bits(want)


@pytest.mark.parametrize("T,K", [(4096, 8192), (8195, 8224)])
@pytest.mark.parametrize("src", ["plain", "silu"])
def test_tensor_scale_many_long_rows(S, T, K, src):
    """A row per wavefront, and rows left over for a second round of them; h of SiLU.mul as the call writes it."""
    g = torch.Generator(device="cuda").manual_seed(T)
    x = torch.randn((T, K), device="cuda", generator=g, dtype=torch.bfloat16)
    x[-1, -1] = 300.0
    if src == "plain":
        y, a = x, S.sharq_prepare(x, None, 1e-6, 2, 4, "nv")
    else:
        y = torch.empty_like(x)
        a = S.sharq_prepare_silu_mul(x, torch.randn((T, K), device="cuda", generator=g).to(torch.bfloat16), 2, 4, "nv",
                                     h_out=y)
    torch.cuda.synchronize()
    want = np.float32(y.float().abs().amax().item()) / np.float32(2688.0)
    assert bits(a.tensor_scale.cpu().numpy()[0]) == bits(want)
