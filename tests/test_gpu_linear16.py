"""The persistent kernel of the formats on 16-bit MFMA (NVFP4, HiF4 at
prefill sizes) against the fp64 oracle: each tile width with ragged rows and
columns, half tiles, every backbone form, and NVFP4 scales on both sides of
the rule that adds the two paths' operands."""

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


def check(S, G, o, wo, dense, T, N, K, dtypes=(torch.float32, torch.bfloat16)):
    a, w = G.oracle_to_act(o, dense_backbone=dense), G.oracle_to_weight(wo)
    ref, mag = O.linear(o, wo), O.linear_abs(o, wo)
    y32 = None
    for dt in dtypes:
        y = torch.full((T + 1, N + 8), float("nan"), dtype=dt, device="cuda")
        S.sharq_linear(a, w, out=y[:T, :N])
        torch.cuda.synchronize()
        assert bool(torch.isnan(y[T]).all()) and bool(torch.isnan(y[:, N:]).all()), "written outside the output"
        if dt == torch.float32:
            y32 = y[:T, :N]
            err = np.abs(G.host(y32).astype(np.float64) - ref)
            # fp32 sums of 2K exact products and the tensor scales' two roundings
            bound = (2 * K + 2) * 2.0 ** -24 * mag
            assert (err <= bound).all(), float((err - bound).max())
        else:
            assert torch.equal(y[:T, :N], y32.to(dt))


@pytest.mark.parametrize("T,N", [
    (2100, 1992),    # 256 x 128 tiles (HiF4: 128 x 256), ragged in both
    (2040, 6104),    # 256 x 192 tiles
    (2290, 7101),    # 256 x 256 tiles, rows of odd length
    (300, 17000),    # 128 x 256 tiles, the last with 44 rows
    (2300, 8008),    # 256 x 256 tiles and a last round of half tiles (NVFP4 compressed, HiF4: 256 x 192)
])
@pytest.mark.parametrize("fmt,n,m,dense,K", [("nv", 2, 4, True, 256), ("nv", 2, 4, False, 128),
                                             ("nv", 4, 8, False, 384), ("hif4", 2, 4, False, 256)])
def test_linear16(S, G, fmt, n, m, dense, K, T, N):
    x = synth.activations(T, K, seed=T + N)
    o = O.prepare(x, synth.gamma(K, seed=3), 1e-6, n, m, fmt)
    check(S, G, o, O.quantize_weight(synth.weight(N, K, seed=7), fmt), dense, T, N, K)


@pytest.mark.parametrize("fmt,n,m", [("nv", 2, 4), ("nv", 4, 8), ("hif4", 2, 4)])
def test_linear16_half_tiles_compressed(S, G, fmt, n, m):
    """792 tiles of 256 x 256 on 256 CUs: three rounds and one of half tiles."""
    T, N, K = 2300, 22400, 128
    o = O.prepare(synth.activations(T, K, seed=1), synth.gamma(K, seed=3), 1e-6, n, m, fmt)
    check(S, G, o, O.quantize_weight(synth.weight(N, K, seed=7), fmt), False, T, N, K, (torch.float32,))


def crafted(T, K, sp, dn, seed=9, n=2, m=4):
    """A prepared NVFP4 activation with the given scale codes ([T, K / 32] and [T, K / 16]) and random codes."""
    rng = np.random.default_rng(seed)
    keep = np.zeros((T, K // m, m), bool)
    np.put_along_axis(keep, rng.random((T, K // m, m)).argsort(axis=2)[..., :n], True, axis=2)
    keep = keep.reshape(T, K)
    codes = np.where(keep, rng.integers(0, 16, size=(T, K)), 0).astype(np.uint8)
    sp_codes, sp_meta = O.pack_backbone(codes, keep, n, m)
    return {"rows": T, "K": K, "n": n, "m": m, "pairs": False, "fmt": "nv", "tensor_scale": np.float32(0.5),
            "mode": "sharq", "sp_codes": sp_codes, "sp_meta": sp_meta, "sp_scale": sp.astype(np.uint8),
            "dn_codes": O.pack_nibbles(rng.integers(0, 16, size=(T, K)).astype(np.uint8)),
            "dn_scale": dn.astype(np.uint8), "dn_meta": np.zeros((T, 0), np.uint8)}


def test_nv_row_beside_other_rows(S, G):
    """Whether the paths are added is decided for 32 rows together: a row's sums may round otherwise beside
    an outlier row, within the same bound; the rows of other groups keep their bits."""
    T, N, K = 2100, 1992, 512
    sp, dn = np.full((T, K // 32), 56), np.full((T, K // 16), 40)    # scales 1 and 1/4: added
    a = crafted(T, K, sp, dn)
    sp[37] = 112                                                     # 2^7 beside 1/4: apart
    b = crafted(T, K, sp, dn)
    wo = O.quantize_weight(synth.weight(N, K, seed=7), "nv")
    w, ys = G.oracle_to_weight(wo), []
    for o in (a, b):
        ys.append(S.sharq_linear(G.oracle_to_act(o), w, dtype=torch.float32))
        torch.cuda.synchronize()
        rows = np.arange(96)
        err = np.abs(G.host(ys[-1][:96]).astype(np.float64) - O.linear(o, wo, rows=rows))
        # fp32 sums of 2K exact products and the tensor scales' two roundings
        assert (err <= (2 * K + 2) * 2.0 ** -24 * O.linear_abs(o, wo, rows=rows)).all()
    assert torch.equal(ys[0][:32], ys[1][:32]) and torch.equal(ys[0][64:], ys[1][64:])


def test_nv_scales_around_the_merge_rule(S, G):
    """Block scales whose ratio runs from equal to far apart, constant over
    32 rows (the kernel decides for 32 rows together) or mixed, zero scales
    and both ends of the E4M3 range among them."""
    T, N, K, n, m = 2100, 1992, 512, 2, 4
    rng = np.random.default_rng(5)
    groups = (T + 31) // 32
    base = rng.integers(0, 127, size=(groups, K // 32))
    gap = rng.integers(-45, 46, size=(groups, K // 32))
    sp = np.repeat(base, 32, axis=0)[:T]
    dn = np.repeat(np.repeat(np.clip(base + gap, 0, 126), 32, axis=0)[:T], 2, axis=1)
    mixed = rng.random((T, K // 16)) < 0.01      # single rows that differ from their group
    dn = np.where(mixed, rng.integers(0, 127, size=dn.shape), dn)
    keep = np.zeros((T, K // m, m), bool)
    np.put_along_axis(keep, rng.random((T, K // m, m)).argsort(axis=2)[..., :n], True, axis=2)
    keep = keep.reshape(T, K)
    codes = np.where(keep, rng.integers(0, 16, size=(T, K)), 0).astype(np.uint8)
    sp_codes, sp_meta = O.pack_backbone(codes, keep, n, m)
    o = {"rows": T, "K": K, "n": n, "m": m, "pairs": False, "fmt": "nv", "tensor_scale": np.float32(0.5),
         "mode": "sharq", "sp_codes": sp_codes, "sp_meta": sp_meta, "sp_scale": sp.astype(np.uint8),
         "dn_codes": O.pack_nibbles(rng.integers(0, 16, size=(T, K)).astype(np.uint8)),
         "dn_scale": dn.astype(np.uint8), "dn_meta": np.zeros((T, 0), np.uint8)}
    check(S, G, o, O.quantize_weight(synth.weight(N, K, seed=7), "nv"), False, T, N, K)
