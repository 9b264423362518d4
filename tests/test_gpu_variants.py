"""GPU parity at the sizes where a kernel variant or a launch rule changes: each test names the
edge it stands on.  Same oracle, same bounds as test_gpu_parity."""
import numpy as np
import pytest
import torch

from paper_2512_02541_amd import binding as agg
from paper_2512_02541_amd import harness, inputs
from test_gpu_parity import _idx_case, run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H", [(1, 1), (1, 7), (1, 8), (3, 3), (1, 12), (2, 10)])
@pytest.mark.parametrize("nq", [200, 600])
def test_pairs_around_the_xcd_count(B, H, nq):
    """(batch, head) pairs below, at and above a multiple of the eight XCDs, at one and at three
    query tiles per pair: the pairs beyond the multiple share the XCDs, and their tiles do not
    divide evenly among them."""
    shape = agg.make_shape(B, 1, 1, nq, 0, H, 64, 1, 3, 0)
    q, k, v = inputs.iid_qkv(B, nq, H, 64, seed=5000 + 100 * B + H, device="cuda")
    run_case(shape, q, k, v, what="pairs %d" % (B * H))
    _idx_case(shape, q, k, v, "pairs %d" % (B * H))
