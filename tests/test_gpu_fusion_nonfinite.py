"""The encoder fused into the FFN output projection where n is not a multiple of its
256-column tiles: the columns behind the last reach neither a nor b, whatever the
weights are.  An infinite W_down entry leaves a and b with the infinities and NaNs of
resbm_encode_fwd on the written z, and products that would overflow in columns that
do not exist leave them finite.
"""
import numpy as np
import pytest
import torch

from gpu_helpers import check, lib, say
from oracle import resbm_oracle as R
from test_gpu_fusion import data, f64

INF = float("inf")
SHAPES = [(333, 200, 520, 40), (70, 512, 8, 8), (300, 1000, 1000, 72)]


def run(L, d, T, n, r, act):
    z, b = (torch.zeros(T, k, dtype=torch.bfloat16, device="cuda") for k in (n, r))
    a = torch.zeros(T, r, device="cuda")
    x, W_e = d["x_attn"].cuda(), d["W_e"].cuda()
    L.ffn_encode_fwd(d["h"].cuda(), d["W_down"].cuda(), x, W_e, z, b, a_save=a, act=act)
    return x, W_e, z, b, a


@pytest.mark.gpu
@pytest.mark.parametrize("act", [R.ACT_IDENTITY, R.ACT_SILU])
@pytest.mark.parametrize("T,d_ff,n,r", SHAPES[:1] + SHAPES[2:], ids=["n520", "n1000"])
def test_infinite_weight(T, d_ff, n, r, act):
    say(f"ffn infinite weight T={T} d_ff={d_ff} n={n} r={r} act={act}")
    L = lib()
    d = data(T, d_ff, n, r, seed=11)
    d["W_down"][7, 2] = INF
    d["W_down"][9, 2] = INF  # z[:, 2]: an infinity of either sign, or their NaN
    x, W_e, z, b, a = run(L, d, T, n, r, act)
    assert bool(torch.isinf(z[:, 2]).any()) and bool(torch.isfinite(z[:, 3:]).all())
    # the same encoder on the written z (n a multiple of 64 there: zero columns added)
    m = (n + 63) // 64 * 64
    pad = lambda t, rows, cols: torch.nn.functional.pad(t, (0, cols - t.shape[1], 0, rows - t.shape[0]))
    rb, ra = torch.zeros_like(b), torch.zeros_like(a)
    L.encode_fwd(pad(x, T, m), pad(z, T, m), pad(W_e, m, r), rb, ra, act=act)
    assert bool(torch.isinf(ra).any())
    for got, ref in ((a, ra), (b, rb)):
        assert torch.equal(torch.isnan(got), torch.isnan(ref))
        assert torch.equal(torch.isposinf(got), torch.isposinf(ref))
        assert torch.equal(torch.isneginf(got), torch.isneginf(ref))


@pytest.mark.gpu
@pytest.mark.parametrize("T,d_ff,n,r", SHAPES, ids=["n520", "n8", "n1000"])
def test_no_overflow_from_missing_columns(T, d_ff, n, r):
    say(f"ffn large weight T={T} d_ff={d_ff} n={n} r={r}")
    L = lib()
    d = data(T, d_ff, n, r, seed=12)
    d["W_down"][7, 2] = 2.0 ** 127
    d["h"][:, 7], d["h"][:, 6] = 2.0 ** -3, 8.0  # z[:, 2] about 2^124; row 7 meets h[:, 6] one row on
    x, W_e, z, b, a = run(L, d, T, n, r, R.ACT_IDENTITY)
    assert bool(torch.isfinite(z).all())
    rb, ra = R.encode_fwd(f64(x), f64(z), f64(W_e), R.ACT_IDENTITY)
    check("a", a, ra, False)
    check("b", b, rb, True)
