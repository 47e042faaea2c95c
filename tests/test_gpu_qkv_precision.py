"""The fused decoder + RMSNorm + QKV projection keeps the precision of the form
that builds z~ first: contracting the weights before the payload must not lose
bits where the sum over r cancels.  Rows of W_d share a component `shared` times
their differences and every payload row is orthogonal to it, so that z~ is made
of the differences alone while the r x N matrix of the weights is made of the
shared component.  The yardstick is the other order on the same operands (W_d as
hi + lo bf16 parts, z~ gamma in float32 rounded to bf16 once, the product in 64
bits, the result rounded to bf16), measured against 64 bits; both errors are
means over 1.6e5 outputs of independent roundings, which agree to a few per cent,
so a tenth more is the bound.
"""
import pytest
import torch

from gpu_helpers import lib, say

EPS = 1e-5


def _parts(x):
    hi = x.bfloat16().float()
    return hi.double() + (x - hi).bfloat16().double()


@pytest.mark.gpu
@pytest.mark.parametrize("shared", [0.0, 300.0, 3000.0])
@pytest.mark.parametrize("T,n,r,N", [(96, 4096, 32, 1696), (300, 2048, 64, 520), (8704, 512, 64, 64)],
                         ids=["r32", "r64", "r64_long"])
def test_cancelling_payload(T, n, r, N, shared):
    say(f"qkv precision T={T} n={n} r={r} N={N} shared={shared}")
    L = lib()
    g = torch.Generator(device="cuda").manual_seed(r)
    rn = lambda *s: torch.randn(*s, generator=g, device="cuda")
    h = rn(T, r // 2).bfloat16()
    b = torch.cat([h, -h], 1).contiguous()
    W_d = rn(r, n) / r ** 0.5 + shared * rn(1, n)
    gamma = 1.0 + 0.1 * rn(n)
    W = (rn(n, N) * n ** -0.5).bfloat16()
    out = torch.empty(T, N, dtype=torch.bfloat16, device="cuda")
    L.decode_qkv_fwd(b, W_d, gamma, W, out, eps=EPS)
    zt = b.double() @ W_d.double()
    s = torch.rsqrt(zt.square().mean(1, keepdim=True) + EPS)
    exact = (zt * gamma.double()) @ W.double() * s
    z32 = (b.double() @ _parts(W_d)).float()
    other = (((z32 * gamma).bfloat16().double() @ W.double()) * s).bfloat16()
    err = lambda y: float((y.double() - exact).norm() / exact.norm())
    say(f"    error {err(out):.3e}, z~ first {err(other):.3e}")
    assert err(out) <= 1.1 * err(other)
