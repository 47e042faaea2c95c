"""The two-linear ops' matrix products at the edges of their tile shapes: one
row or column past a 128 or 256 tile, K tails of every stage parity, more work
items than compute units (a block then walks several), and token sums with and
without splits.  With the identity activation every output is a product, or a
product of a product rounded to bf16 once, so the bounds are derived: bf16
outputs may differ from 64 bits by half an ulp (2^-9 relative, doubled for ties
and double rounding) and by the float32 accumulation of K terms, K 2^-24 of the
sum of absolute terms; a bf16 intermediate adds 2^-8 of the absolute terms.
"""
import pytest
import torch

from gpu_helpers import lib, say
from paper_2604_11947_amd import resbm as R

pytestmark = pytest.mark.gpu

CASES = [
    # T, n, m, r
    (255, 264, 256, 8),       # one 128-tile row short of two
    (257, 512, 264, 32),      # a row past, K of 8 stages and of 5
    (1030, 264, 520, 40),     # 64 x 64 tiles, ragged both ways; dW4 and dW1 in 256 x 256
    (4360, 4104, 72, 8),      # 306 tiles of 256 x 256 on 256 blocks, K = 72 (one stage pair)
    (8200, 2312, 200, 24),    # 330 tiles, K = 200 (four stages)
    (40000, 72, 128, 16),     # 313 tiles of 128 x 128 by four waves
    (33000, 64, 8, 8),        # 64 x 32 and 64 x 64 tiles, one stage
]


def _close(name, got, ref, absref, K, bf16, inter=0.0):
    tol = ref.abs() * (2.0 ** -8 if bf16 else 2.0 ** -23) + absref * (K * 2.0 ** -24 + inter)
    bad = (got.double() - ref).abs() > tol
    assert not bool(bad.any()), f"{name}: {int(bad.sum())} of {bad.numel()} outside the bound"


@pytest.mark.parametrize("T,n,m,r", CASES)
def test_products_at_tile_edges(T, n, m, r):
    say(f"gemm tiles T={T} n={n} m={m} r={r}")
    L = lib("bf16")
    g = torch.Generator(device="cuda").manual_seed(T + n)
    rn = lambda *s, std=1.0: (torch.randn(*s, generator=g, device="cuda") * std).to(torch.bfloat16)
    bf = lambda *s: torch.full(s, float("nan"), dtype=torch.bfloat16, device="cuda")
    f32 = lambda *s: torch.full(s, float("nan"), device="cuda")
    W1, W2, W3, W4 = rn(n, m, std=n ** -0.5), rn(m, r, std=m ** -0.5), rn(r, m, std=r ** -0.5), rn(m, n, std=m ** -0.5)
    x, z, b, g_b, g_zt = rn(T, n), rn(T, n), rn(T, r), rn(T, r), rn(T, n)
    d = lambda t: t.double()
    a = lambda t: t.double().abs()
    ident = R.ACT_IDENTITY

    bo, u = bf(T, r), bf(T, m)
    L.encode2_fwd(x, z, W1, W2, bo, u, act=ident)
    _close("u", u, d(z) @ d(W1), a(z) @ a(W1), n, True)
    _close("b", bo, d(x)[:, :r] + d(u) @ d(W2), a(x)[:, :r] + a(u) @ a(W2), m + 1, True)

    zt, v = bf(T, n), bf(T, m)
    L.decode2_fwd(b, W3, W4, zt, v, act=ident)
    _close("v", v, d(b) @ d(W3), a(b) @ a(W3), r, True)
    _close("z~", zt, d(v) @ d(W4), a(v) @ a(W4), m, True)

    g_z, dW1, dW2 = bf(T, n), f32(n, m), f32(m, r)
    L.encode2_bwd(z, u, g_b, W1, W2, g_z, dW1, dW2, act=ident)
    gu, agu = d(g_b) @ d(W2).t(), a(g_b) @ a(W2).t()
    _close("dW2", dW2, d(u).t() @ d(g_b), a(u).t() @ a(g_b), T, False)
    _close("dW1", dW1, d(z).t() @ gu, a(z).t() @ agu, T, False, 2.0 ** -8)
    _close("g_z", g_z, gu @ d(W1).t(), agu @ a(W1).t(), m, True, 2.0 ** -8)

    go, dW3, dW4 = bf(T, r), f32(r, m), f32(m, n)
    L.decode2_bwd(b, v, g_zt, None, W3, W4, go, dW3, dW4, act=ident)
    gv, agv = d(g_zt) @ d(W4).t(), a(g_zt) @ a(W4).t()
    _close("dW4", dW4, d(v).t() @ d(g_zt), a(v).t() @ a(g_zt), T, False)
    _close("dW3", dW3, d(b).t() @ gv, a(b).t() @ agv, T, False, 2.0 ** -8)
    _close("g_b", go, gv @ d(W3).t(), agv @ a(W3).t(), m, True, 2.0 ** -8)
