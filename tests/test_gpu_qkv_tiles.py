"""The fused decoder + RMSNorm + QKV projection at the rule between its two orders.
With more tokens than the workspace holds row sums for, or many strips, a narrow n
forms z~ gamma first, in 256 x 256 tiles (two launches whatever T is); a wide one goes
in chunks of tokens.  Both against the 64-bit oracle, with guard bands and every byte
behind the workspace kept.
"""
import ctypes

import pytest
import torch

from gpu_helpers import check, guarded, lib, say
from test_gpu_fusion import EPS, dq_data, dq_ref

TILES = [(600, 64, 8, 8), (2000, 64, 16, 192), (1100, 64, 64, 264), (9000, 128, 32, 384), (20001, 256, 40, 136),
         (33000, 192, 8, 16),
         (5, 64, 8, 9528)]
CHUNKS = [(4200, 512, 16, 6000), (4200, 256, 40, 6144)]


def launches(L, call):
    """Kernel launches of one call, counted in a captured graph."""
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    count = ctypes.c_size_t(0)
    assert L.cdll.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(count)) == 0
    return count.value


@pytest.mark.gpu
@pytest.mark.parametrize("T,n,r,N", TILES + CHUNKS, ids=["T%d_n%d_r%d_N%d" % c for c in TILES + CHUNKS])
def test_qkv_many_tokens(T, n, r, N):
    say(f"qkv many tokens T={T} n={n} r={r} N={N}")
    L = lib()
    d = dq_data(T, n, r, N, seed=9)
    g = {k: v.cuda() for k, v in d.items()}
    nb = int(L.cdll.resbm_decode_qkv_workspace_bytes(n, r))
    buf = torch.full((nb + 4096,), 0xFF, dtype=torch.uint8, device="cuda")
    out, _, intact = guarded((T, N), torch.bfloat16, "cuda", pad=8)
    call = lambda: L.decode_qkv_fwd(g["b"], g["W_d"], g["gamma"], g["W_qkv"], out, eps=EPS, ws=buf[:nb])
    call()
    torch.cuda.synchronize()
    intact()
    assert bool((buf[nb:] == 0xFF).all()), "written behind the workspace"
    check("out", out, dq_ref(d), True)
    count = launches(L, call)
    assert count == (2 if (T, n, r, N) in TILES else 4)
