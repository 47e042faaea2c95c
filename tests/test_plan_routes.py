"""The rules that choose between the one-pass kernels of short streams and the
streaming ones, and the place of their partial sums, evaluated from the plan that
kernels and host share (compiled here for the host).
"""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#include "resbm_plan.hpp"
using namespace resbm;
extern "C" void routes(int64_t T, int n, int r, int* out) {
  const Plan p = make_plan(T, n, r);
  out[0] = p.ef_smt; out[1] = p.db_once; out[2] = p.eb_once; out[3] = p.wide;
}
// The partial sums of every short kernel lie inside its op's workspace.
static bool fits(int64_t T, int n, int r) {
  const Plan p = make_plan(T, n, r);
  const size_t dw = (size_t)p.RP * n * 4;
  const int64_t steps = ceil_div(T, 64);
  return (!p.ef_smt || p.ef_nsl == 1 || (size_t)p.ef_nsl * T * p.RP * 4 <= p.ef_ws) &&
         (!p.db_once || (p.db_once_dwp >= (size_t)p.once_ncg * T * p.RP * 4 &&
                         p.db_once_dwp + ceil_div(steps, p.db_once) * dw <= p.db_ws)) &&
         (!p.eb_once || ceil_div(steps, p.eb_once) * dw <= p.eb_ws);
}
extern "C" int64_t first_misfit(int64_t count) {
  uint64_t s = 12345;
  auto rnd = [&](uint64_t m) { s = s * 6364136223846793005ull + 1442695040888963407ull; return (s >> 33) % m; };
  for (int64_t i = 0; i < count; ++i) {
    const int n = 64 * (1 + (int)(rnd(4) ? rnd(64) : rnd(1024)));
    int r = 4 * (1 + (int)rnd(64));
    if (r > n) r = n;
    const int64_t T = 1 + rnd((uint64_t)1 << (1 + rnd(20)));
    if (!fits(T, n, r)) return T << 32 | n << 12 | r;
  }
  return 0;
}
"""


@pytest.fixture(scope="session")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, lib = d / "plan.cpp", d / "plan.so"
    src.write_text(SOURCE)
    subprocess.run([shutil.which("g++"), "-O2", "-std=c++17", "-shared", "-fPIC", "-DRESBM_IO_F32_BUILD=0",
                    "-I", os.path.join(ROOT, "paper_2604_11947_amd", "csrc"), str(src), "-o", str(lib)], check=True)
    c = ctypes.CDLL(str(lib))
    c.first_misfit.restype = ctypes.c_int64
    c.first_misfit.argtypes = [ctypes.c_int64]

    def routes(T, n, r):
        out = (ctypes.c_int * 4)()
        c.routes(ctypes.c_int64(T), n, r, out)
        return dict(zip(("encode_fwd", "decode_bwd", "encode_bwd", "wide"), out))

    routes.first_misfit = c.first_misfit
    return routes


def test_partial_sums_fit_the_workspace(plan):
    assert plan.first_misfit(1_000_000) == 0


# (op, T, n, r): the largest T (or n) of a rule, and the next one outside it
EDGES = [
    ("encode_fwd", (16384, 1024, 32), (16385, 1024, 32)),   # more 64-token blocks than units: n <= 768 above r = 16
    ("encode_fwd", (16385, 768, 32), (16385, 832, 32)),
    ("encode_fwd", (32768, 768, 64), (32769, 768, 64)),
    ("encode_fwd", (32768, 4096, 16), (32768, 4160, 16)),
    ("encode_fwd", (8192, 1024, 128), (8193, 1024, 128)),   # two groups of j-tiles: one round of blocks
    ("encode_fwd", (8192, 1024, 68), (8193, 64, 68)),
    ("encode_bwd", (16384, 64, 64), (16385, 64, 64)),
    ("encode_bwd", (16385, 192, 32), (16385, 128, 32)),
    ("encode_bwd", (32768, 192, 32), (32769, 192, 32)),
    ("encode_bwd", (16384, 2048, 64), (16385, 2048, 32)),   # 2^25 elements
    ("decode_bwd", (26214, 1088, 40), (26215, 1088, 40)),   # 2^25 elements in whole column tiles
    ("decode_bwd", (131072, 64, 20), (131073, 64, 20)),
]


@pytest.mark.parametrize("op,inside,outside", EDGES)
def test_edges_of_the_rules(plan, op, inside, outside):
    assert plan(*inside)[op] > 0 and plan(*outside)[op] == 0


def test_streaming_shapes_reach_the_streaming_kernels(plan):
    import test_gpu_streaming as S

    for op, shapes in (("encode_fwd", S.ENCODE_FWD), ("decode_bwd", S.DECODE_BWD), ("encode_bwd", S.ENCODE_BWD)):
        for s in shapes:
            assert plan(*s[:3])[op] == 0, (op, s)
