"""The one-pass kernels of short streams at the edges of their tiles and of the
rules that choose them (16 / 32 / 64-token blocks and slices of n in encode_fwd,
64 x 256 tiles in the backward ops), and the streaming kernels right behind
those edges: the whole chain of ops against the oracle, with guard bands around
every output and behind the workspace.
"""
import pytest
import torch

from gpu_helpers import lib, say
from test_gpu_random_shapes import test_random_shape_chain as chain

# (T, n, r, act, add_identity, fused)
CASES = [
    (1, 64, 4, 1, False, False),        # one token, one unit
    (17, 8192, 48, 1, False, True),     # sixteen slices, three j-tiles in a group of four
    (15, 1088, 68, 0, True, True),      # wide r: two j-groups, the second ragged
    (65, 576, 36, 1, False, False),     # token tail of one, third column group of 64 columns
    (255, 2048, 256, 1, True, False),   # four j-groups
    (4080, 512, 16, 1, False, True),    # last 16-token blocks of encode_fwd
    (4081, 512, 20, 0, False, False),   # first 32-token blocks
    (8192, 576, 12, 1, True, True),     # last 32-token blocks
    (8193, 576, 16, 1, False, False),   # first 64-token blocks; several steps per backward block
    (16400, 768, 40, 1, False, True),   # more 64-token blocks than units; encode_bwd streams
    (3572, 6592, 4, 1, True, False),    # decode_bwd: steps rounded up to one round of blocks
    (32768, 192, 28, 0, False, True),   # encode_bwd: the longest token range
    (8193, 2112, 32, 1, False, True),   # encode_fwd back on the streaming kernel
    (16385, 2112, 20, 1, False, False),  # all ops on the streaming kernels (more than 2^25 elements)
    (2049, 1024, 132, 1, False, True),  # wide r: 32-token blocks, decode_bwd in three j-groups
]


@pytest.mark.gpu
@pytest.mark.parametrize("c", CASES, ids=["T%d_n%d_r%d" % c[:3] for c in CASES])
def test_short_streams(c, monkeypatch):
    L = lib()
    say("short streams", c)
    guards = []

    def workspace(T, n, r, device):
        nb = L.workspace_bytes(T, n, r)
        buf = torch.full((nb + 4096,), 0xFF, dtype=torch.uint8, device=device)  # NaN bits in stale partials
        guards.append(buf[nb:])
        return buf[:nb]

    monkeypatch.setattr(L, "workspace", workspace)
    chain.hypothesis.inner_test((*c, 7))
    for g in guards:
        assert bool((g == 0xFF).all()), "written behind the workspace"


@pytest.mark.gpu
def test_short_streams_deterministic():
    """Cross-wave, cross-slice and cross-block sums run in a fixed order."""
    L = lib()
    T, n, r = 1024, 4096, 32
    say("short streams deterministic", T, n, r)
    g = torch.Generator(device="cuda").manual_seed(3)
    x, z = (torch.randn(T, n, generator=g, device="cuda").bfloat16() for _ in range(2))
    W_e, W_d = torch.randn(n, r, generator=g, device="cuda"), torch.randn(r, n, generator=g, device="cuda")
    outs = []
    for _ in range(3):
        b, a = torch.empty(T, r, dtype=torch.bfloat16, device="cuda"), torch.empty(T, r, device="cuda")
        gz, gb, dWe, dWd = torch.empty_like(z), torch.empty_like(b), torch.empty_like(W_e), torch.empty_like(W_d)
        ws = L.workspace(T, n, r, "cuda")
        L.encode_fwd(x, z, W_e, b, a, ws=ws)
        L.encode_bwd(z, W_e, a, b, gz, dWe, ws=ws)
        L.decode_bwd(b, W_d, z, x, gb, dWd, ws=ws)
        outs.append((b, a, gz, dWe, gb, dWd))
    torch.cuda.synchronize()
    for o in outs[1:]:
        for p, q in zip(o, outs[0]):
            assert torch.equal(p, q)
