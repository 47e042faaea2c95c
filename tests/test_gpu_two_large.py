"""A float32 weight gradient of the two-linear ops beyond 4 GiB (n m > 2^30): every
element lands in its place.  The rows checked lie in front of, at and behind the 4 GiB
line and at both ends; bounds as in test_gpu_gemm_tiles.py.
"""
import pytest
import torch

from gpu_helpers import lib, say
from paper_2604_11947_amd import resbm as R
from test_gpu_gemm_tiles import _close


@pytest.mark.gpu
def test_weight_gradients_beyond_4_gib():
    T, n, m, r = 24, 32784, 32776, 8
    say(f"two-linear large T={T} n={n} m={m} r={r}")
    L = lib()
    g = torch.Generator(device="cuda").manual_seed(5)
    bf = lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()
    big = lambda *s: torch.empty(*s, dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    z, u, g_b, W2 = bf(T, n), bf(T, m), bf(T, r), bf(m, r)
    W1, g_z = big(n, m), torch.empty_like(z)
    dW1, dW2 = torch.full((n, m), float("nan"), device="cuda"), torch.empty(m, r, device="cuda")
    L.encode2_bwd(z, u, g_b, W1, W2, g_z, dW1, dW2, act=R.ACT_IDENTITY)
    gu, agu = g_b.double() @ W2.double().t(), g_b.double().abs() @ W2.double().abs().t()
    line = 2 ** 30 // m
    rows = [0, 1, 255, 256, line - 1, line, line + 1, n - 257, n - 256, n - 1]
    _close("dW1", dW1[rows], z[:, rows].double().t() @ gu, z[:, rows].double().abs().t() @ agu, T, False, 2.0 ** -8)
    assert not bool(torch.isnan(dW1).any())
