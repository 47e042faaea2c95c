"""The decoder fused into RMSNorm + QKV at the edges of its strips: column tails
of 32- and 64-column strips, token tails, several token ranges, more rows than
row scales held at a time, units behind the prepared fragments, both depths of r
(three shapes take the other order, in tiles: see test_gpu_qkv_tiles.py, which has
the chunks of tokens too); every workspace byte behind the required ones kept.
"""
import pytest
import torch

from gpu_helpers import check, guarded, lib, say
from test_gpu_fusion import EPS, dq_data, dq_ref

CASES = [(1, 64, 8, 8), (1300, 64, 8, 72), (1300, 64, 64, 64), (257, 4032, 24, 40), (2049, 1024, 32, 72),
         (2100, 256, 16, 9000), (8200, 1024, 48, 200), (300, 2112, 64, 4000)]


@pytest.mark.gpu
@pytest.mark.parametrize("T,n,r,N", CASES, ids=["T%d_n%d_r%d_N%d" % c for c in CASES])
def test_qkv_strip(T, n, r, N):
    L = lib()
    say(f"qkv strip T={T} n={n} r={r} N={N}")
    d = dq_data(T, n, r, N, seed=3)
    nb = int(L.cdll.resbm_decode_qkv_workspace_bytes(n, r))
    buf = torch.full((nb + 4096,), 0xFF, dtype=torch.uint8, device="cuda")
    out, _, intact = guarded((T, N), torch.bfloat16, "cuda", pad=8)
    L.decode_qkv_fwd(d["b"].cuda(), d["W_d"].cuda(), d["gamma"].cuda(), d["W_qkv"].cuda(), out, eps=EPS, ws=buf[:nb])
    torch.cuda.synchronize()
    intact()
    assert bool((buf[nb:] == 0xFF).all()), "written behind the workspace"
    check("out", out, dq_ref(d), True)
