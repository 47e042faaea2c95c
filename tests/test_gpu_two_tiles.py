"""The two-linear ops with SiLU and a fused skip gradient on every tile shape of their
T-row products: narrow tiles, the pipelined 128 x 128 and 256 x 256 kernels with one
item per block and with several (the counted waits behind the epilogues that store
twice or read a second operand), the four-wave 128 x 128 one.  References in 64 bits;
bounds as in test_gpu_gemm_tiles.py with a relative 2^-8 of the absolute terms for each
bf16 intermediate (phi(u), phi(v), g_u, g_v), and |phi'| <= 1.1.
"""
import pytest
import torch

from gpu_helpers import lib, say
from paper_2604_11947_amd import resbm as R
from test_gpu_gemm_tiles import _close

CASES = [
    # T, n, m, r
    (24000, 264, 520, 8),     # u, g_v: 282 tiles of 256 x 256, K = 264 (5 stages); v, g_u: one stage, 940 of 128 x 128
    (100, 72, 33000, 16),     # u: 258 tiles of 128 x 128, two stages
    (20000, 200, 120, 40),    # u: 157 tiles of 128 x 128; z~, g_z: four-wave, 314
    (40000, 72, 128, 16),     # four-wave, 313 tiles
    (70000, 64, 168, 8),      # 256 x 256 with a padded column tile, 274 tiles
    (32769, 40, 256, 8),      # one stage, 514 tiles of 128 x 128
    (16384, 64, 136, 24),     # 256 tiles of 128 x 128, and one more:
    (16385, 72, 136, 24),
    (8192, 136, 248, 64),     # 128 tiles of 128 x 128 (narrow ones run), and two more:
    (8193, 136, 248, 72),
    (65, 32, 40, 16),         # narrow tiles of 32 and 64 columns
    (130, 64, 24, 8),
    (4000, 520, 64, 136),     # g_z on 128 x 128 tiles, one column tile with the skip gradient, one with part of it
    (20000, 520, 136, 264),   # the same on 256 x 256 tiles
]


@pytest.mark.gpu
@pytest.mark.parametrize("T,n,m,r", CASES, ids=["T%d_n%d_m%d_r%d" % c for c in CASES])
def test_silu_and_fused_skip(T, n, m, r):
    say(f"two-linear tiles T={T} n={n} m={m} r={r}")
    L = lib()
    g = torch.Generator(device="cuda").manual_seed(T + m)
    rn = lambda *s, std=1.0: (torch.randn(*s, generator=g, device="cuda") * std).bfloat16()
    bf = lambda *s: torch.full(s, float("nan"), dtype=torch.bfloat16, device="cuda")
    f32 = lambda *s: torch.full(s, float("nan"), device="cuda")
    W1, W2, W3, W4 = rn(n, m, std=n ** -0.5), rn(m, r, std=m ** -0.5), rn(r, m, std=r ** -0.5), rn(m, n, std=m ** -0.5)
    x, z, b, g_b, g_zt, g_id = rn(T, n), rn(T, n), rn(T, r), rn(T, r), rn(T, n), rn(T, n)
    d = lambda t: t.double()
    a = lambda t: t.double().abs()
    phi = lambda t: t * torch.sigmoid(t)
    dphi = lambda t: torch.sigmoid(t) * (1 + t * (1 - torch.sigmoid(t)))
    E = 2.0 ** -8

    bo, u = bf(T, r), bf(T, m)
    L.encode2_fwd(x, z, W1, W2, bo, u, act=R.ACT_SILU)
    u64 = d(z) @ d(W1)
    _close("u", u, u64, a(z) @ a(W1), n, True)
    # (phi(u) from the float32 u: its accumulation error, at most 1.1 n 2^-24 of |z| |W1|, is far below E)
    _close("b", bo, d(x)[:, :r] + phi(u64) @ d(W2), a(x)[:, :r] + (phi(u64).abs() + E) @ a(W2), m + 1, True, E)

    zt, v = bf(T, n), bf(T, m)
    L.decode2_fwd(b, W3, W4, zt, v, act=R.ACT_SILU)
    v64 = d(b) @ d(W3)
    _close("v", v, v64, a(b) @ a(W3), r, True)
    _close("z~", zt, phi(v64) @ d(W4), (phi(v64).abs() + E) @ a(W4), m, True, E)

    g_z, dW1, dW2 = bf(T, n), f32(n, m), f32(m, r)
    L.encode2_bwd(z, u, g_b, W1, W2, g_z, dW1, dW2, g_x=g_z, act=R.ACT_SILU)
    gu, agu = (d(g_b) @ d(W2).t()) * dphi(d(u)), 1.1 * (a(g_b) @ a(W2).t())
    _close("dW2", dW2, phi(d(u)).t() @ d(g_b), phi(d(u)).abs().t() @ a(g_b), T, False, E)
    _close("dW1", dW1, d(z).t() @ gu, a(z).t() @ agu, T, False, E)
    ref = gu @ d(W1).t()
    ref[:, :r] += d(g_b)
    _close("g_z", g_z, ref, agu @ a(W1).t() + 1.0, m + 1, True, E)

    go, dW3, dW4 = bf(T, r), f32(r, m), f32(m, n)
    L.decode2_bwd(b, v, g_zt, g_id, W3, W4, go, dW3, dW4, act=R.ACT_SILU)
    gv, agv = (d(g_zt) @ d(W4).t()) * dphi(d(v)), 1.1 * (a(g_zt) @ a(W4).t())
    _close("dW4", dW4, phi(d(v)).t() @ d(g_zt), phi(d(v)).abs().t() @ a(g_zt), T, False, E)
    _close("dW3", dW3, d(b).t() @ gv, a(b).t() @ agv, T, False, E)
    _close("g_b", go, d(g_id)[:, :r] + gv @ d(W3).t(), agv @ a(W3).t() + 1.0, m + 1, True, E)
