"""The native argument marshalling: it hands anything but plain CUDA tensors back
to the Python path (None), whose errors are unchanged, and on a GPU it makes the
same calls as that path, on the current stream."""
import pytest
import torch

from gpu_helpers import lib
from paper_2604_11947_amd import resbm as R


def test_built_and_refuses_host_tensors():
    assert R._marshal is not None, "the marshalling module is not built"
    b, W, zt = torch.zeros(4, 8, dtype=torch.bfloat16), torch.zeros(8, 64), torch.zeros(4, 64, dtype=torch.bfloat16)
    assert R._marshal.decode_fwd(0, 0, b, W, zt, False, None) is None
    assert R._marshal.decode_fwd(0, 0, b, W, None, False, None) is None
    assert R._marshal.encode_fwd(0, 0, b) is None


@pytest.mark.gpu
def test_same_calls_as_the_python_path(monkeypatch):
    L = lib()
    T, n, r = 70, 192, 12
    g = torch.Generator(device="cuda").manual_seed(0)
    rn = lambda *s: torch.randn(*s, generator=g, device="cuda")
    W_e, W_d, a = rn(n, r), rn(r, n), rn(T, r)
    x, z, gzt = (rn(T, n + 8).bfloat16()[:, :n] for _ in range(3))
    b, gb = rn(T, r).bfloat16(), rn(T, r).bfloat16()

    def run():
        o = {k: torch.zeros_like(v) for k, v in dict(b=b, a=a, zt=z, gb=b, dW_d=W_d, gz=z, dW_e=W_e).items()}
        W, M = W_e.clone(), W_d.t().contiguous()
        ws, mws = L.workspace(T, n, r, "cuda"), L.matrix_workspace(n, r, "cuda")
        st = torch.cuda.Stream()
        st.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(st):
            L.encode_fwd(x, z, W_e, o["b"], o["a"], ws=ws)
            L.decode_fwd(b, W_d, o["zt"], add_identity=True, ws=ws)
            L.decode_bwd(b, W_d, gzt, None, o["gb"], o["dW_d"], ws=ws)
            L.encode_bwd(z, W_e, a, gb, o["gz"], o["dW_e"], g_x=o["gz"], ws=ws)
            L.muon_update(W, W_e, M, 0.01, nesterov=True, ws=mws)
        torch.cuda.current_stream().wait_stream(st)
        torch.cuda.synchronize()
        return [*o.values(), W, M]

    fast = run()
    assert R._marshal.decode_fwd(L._at["resbm_decode_fwd"], L.io_code, b, W_d, torch.zeros_like(z), False, None) == R.OK
    bad = torch.zeros(T, n + 1, dtype=torch.bfloat16, device="cuda")
    with pytest.raises(ValueError, match="z_tilde: expected shape"):
        L.decode_fwd(b, W_d, bad)
    with pytest.raises(TypeError, match="W_d"):
        L.decode_fwd(b, W_d.half(), torch.zeros_like(z))
    with pytest.raises(R.ResbmError, match="resbm_encode_fwd"):
        L.encode_fwd(x, z, W_e, fast[0], fast[1], act=7, ws=L.workspace(T, n, r, "cuda"))
    monkeypatch.setattr(R, "_marshal", None)
    for p, q in zip(fast, run()):
        assert torch.equal(p, q)
