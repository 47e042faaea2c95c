"""The streaming kernels of the bf16 build at the edges of their tiles: the checks of
test_gpu_parity.py and test_gpu_nonfinite.py on shapes that the rules leave to them
(those files' own shapes run the one-pass kernels of short streams, but for decode_fwd,
encode_bwd above r = 64 and the float32 build).  Every tiling of r, ragged r, token
tails, row strides, accumulation, every g_id and g_x mode, NaN and infinity patterns,
run-to-run identity.  test_plan_routes.py holds each shape to its kernel.
"""
import pytest

import test_gpu_nonfinite as NF
import test_gpu_parity as P

ids = lambda shapes: ["T%d_n%d_r%d" % s[:3] for s in shapes]

ENCODE_FWD = [
    # W_e split in LDS (r <= 16)
    (32800, 64, 4), (8200, 4160, 12), (32769, 128, 16),
    # fragments prepared, two to four tiles of r
    (32769, 64, 20), (16400, 832, 28), (16401, 832, 40), (8200, 1088, 44), (16387, 832, 52), (8193, 1088, 64),
    # wide r, five to eleven tiles, and split over two blocks from twelve on
    (8200, 128, 68), (8210, 192, 92), (8195, 128, 100), (8193, 320, 124), (5500, 192, 132), (5444, 192, 160),
    (5443, 256, 172), (5500, 192, 188), (4100, 256, 196), (4099, 256, 220), (4111, 256, 236), (4097, 1088, 256),
]
DECODE_BWD = [
    # (T, n, r, mode)
    (131100, 64, 4, "none"), (26300, 1088, 12, "separate"), (131073, 64, 20, "alias"), (32801, 1024, 32, "accumulate"),
    (131100, 64, 36, "separate"), (43700, 576, 52, "accumulate"), (131077, 64, 64, "alias"),
    (1000, 1088, 68, "separate"), (3000, 320, 92, "alias"), (1500, 704, 104, "accumulate"), (700, 1600, 116, "none"),
    (9000, 320, 140, "accumulate"), (6500, 704, 152, "separate"), (9001, 320, 164, "alias"), (9000, 576, 188, "none"),
    (9003, 320, 200, "separate"), (9000, 320, 212, "accumulate"), (6500, 1088, 236, "alias"), (9000, 320, 256, "none"),
]
ENCODE_BWD = [
    # (T, n, r, act, g_x): SiLU without g_x accumulates
    (32800, 192, 4, P.SILU, "none"), (16400, 128, 12, P.ID, "fused"), (16390, 64, 20, P.SILU, "separate"),
    (32771, 320, 32, P.SILU, "fused"), (16401, 832, 40, P.ID, "separate"), (16400, 64, 44, P.SILU, "none"),
    (16387, 832, 52, P.SILU, "fused"), (16449, 64, 64, P.SILU, "separate"),
]


@pytest.mark.gpu
@pytest.mark.parametrize("i,shape", list(enumerate(ENCODE_FWD)), ids=ids(ENCODE_FWD))
def test_encode_fwd(i, shape):
    P.test_encode_fwd(shape, P.SILU if i % 2 else P.ID)


@pytest.mark.gpu
@pytest.mark.parametrize("case", DECODE_BWD, ids=ids(DECODE_BWD))
def test_decode_bwd(case):
    P.test_decode_bwd(case[:3], case[3])


@pytest.mark.gpu
@pytest.mark.parametrize("case", ENCODE_BWD, ids=ids(ENCODE_BWD))
def test_encode_bwd(case):
    P.test_encode_bwd(case[:3], case[3], case[4])


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(32769, 128, 16), (16401, 832, 40), (8195, 128, 100), (4111, 256, 236)],
                         ids=["r16", "r40", "r100", "r236"])
def test_encode_fwd_nonfinite(shape):
    NF.test_encode_fwd_inf_weight_nan_token(shape, P.SILU)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(131073, 64, 20), (43700, 576, 52), (1500, 704, 104)], ids=["r20", "r52", "r104"])
def test_decode_bwd_nonfinite(shape):
    NF.test_decode_bwd_inf_weight_nan_gradient(shape)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(16400, 128, 12), (16401, 832, 40)], ids=["r12", "r40"])
def test_encode_bwd_nonfinite(shape):
    NF.test_encode_bwd_nan_gradient_inf_weight(shape, P.SILU)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(43700, 576, 40), (9000, 320, 188)], ids=["r40", "r188"])
def test_bitwise_deterministic(shape):
    P.test_bitwise_deterministic(shape)
