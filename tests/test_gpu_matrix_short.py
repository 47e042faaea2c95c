"""The optimizer step's short-side kernels at their edges: tile counts of the
short side, row tails of the 128-row chunks and 16-row output tiles, several
chunks per block, both orientations, partial sums added by the recurrence block
and by the reduction.
"""
import pytest

from test_gpu_matrix import test_muon_update_two_steps as two_steps

CASES = [(1, 1), (16, 16), (129, 16), (15, 257), (2049, 17), (33, 1000), (49, 4100), (4000, 64), (40000, 4), (5, 33000)]


@pytest.mark.gpu
@pytest.mark.parametrize("p,q", CASES, ids=["%dx%d" % c for c in CASES])
@pytest.mark.parametrize("nesterov", [False, True])
def test_muon_short_side(p, q, nesterov):
    two_steps(p, q, nesterov)
