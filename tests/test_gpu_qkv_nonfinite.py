"""The fused decoder + RMSNorm + QKV projection with infinite and NaN weights:
NaNs and infinities, with their signs, sit exactly where the 64-bit oracle's are
(out is a sum over the n columns of z~, so one infinite gamma or W_qkv entry gives
a signed infinity), every other output keeps the parity bound.  Shapes cover the
32- and 64-column strips at both depths of r, with column and token tails.
"""
import numpy as np
import pytest
import torch

from gpu_helpers import lib, say
from test_gpu_fusion import EPS, dq_data, dq_ref
from test_gpu_nonfinite import same_nonfinite

INF, NAN = float("inf"), float("nan")
SHAPES = [(70, 256, 16, 72), (300, 512, 48, 200), (2100, 512, 32, 136), (8200, 1024, 40, 72)]
# tensor -> {index: value}
POISON = {
    "W_qkv_inf": {"W_qkv": {(5, 3): INF, (5, 40): -INF, (9, 71): INF}},
    "W_qkv_two": {"W_qkv": {(5, 3): INF, (6, 3): INF, (7, 17): NAN}},
    "gamma_inf": {"gamma": {(11,): INF}},
    "gamma_-inf": {"gamma": {(250,): -INF}},
    "W_d_inf": {"W_d": {(2, 33): -INF}},
    "gamma_W_qkv": {"gamma": {(11,): INF}, "W_qkv": {(11, 8): 0.0, (12, 9): NAN}},
}


@pytest.mark.gpu
@pytest.mark.parametrize("kind", POISON)
@pytest.mark.parametrize("T,n,r,N", SHAPES, ids=["T%d_n%d_r%d_N%d" % c for c in SHAPES])
def test_qkv_nonfinite(T, n, r, N, kind):
    say(f"qkv non-finite T={T} n={n} r={r} N={N} {kind}")
    L = lib()
    d = dq_data(T, n, r, N, seed=8)
    for k, at in POISON[kind].items():
        for i, v in at.items():
            d[k][i] = v
    d["b"][T // 2] = 0  # z~ = 0 there: 0 x inf
    out = torch.zeros(T, N, dtype=torch.bfloat16, device="cuda")
    L.decode_qkv_fwd(d["b"].cuda(), d["W_d"].cuda(), d["gamma"].cuda(), d["W_qkv"].cuda(), out, eps=EPS)
    with np.errstate(invalid="ignore", over="ignore"):
        ref = dq_ref(d)
    if np.isfinite(ref).any():
        same_nonfinite("out", out, ref, True)
    else:
        assert not bool(torch.isfinite(out.float()).any())
        assert np.array_equal(torch.isnan(out).cpu().numpy(), np.isnan(ref))
