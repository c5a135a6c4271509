"""fp32 launch-per-layer path (gemm_f32.hip) at the sizes where its tiles and pieces end: rows that are no multiple of
four words, extents below one piece, batches around 32 and 64, split and unsplit contractions, several layers per
update launch, learner momentum -- against the oracle."""
import numpy as np
import pytest

from tests.test_gpu_small import TOL_FP32, _pair, _run_and_compare

pytestmark = pytest.mark.gpu

CASES = [
    # P, K, B, dims, learner momentum
    (2, 2, 31, (37, 65, 10), 0.0),               # one 32-row tile, one column over a 64-wide tile
    (3, 2, 33, (129, 127, 63, 24), 0.9),         # one row over a 32-row tile, odd rows everywhere, generic last layer
    (2, 2, 64, (130, 128, 64, 10), 0.0),         # whole tiles next to a ragged one; 64-row batch
    (2, 2, 65, (191, 66, 33), 0.9),              # one row over a 64-row tile, three 32-row tiles
    (40, 2, 128, (96, 192, 10), 0.0),            # 64-row tiles, unsplit
    (2, 2, 20, (3, 5, 2), 0.9),                  # inputs below one piece of four words
    (2, 2, 4, (40, 3, 30, 1), 0.0),              # a hidden layer of three units, a single class
    (1, 2, 96, (3071, 70, 40), 0.0),             # long odd contraction split over workgroups, remainder of the last split
    (2, 1, 7, (50, 20, 20, 20, 20, 20, 20, 20, 20, 10), 0.0),   # nine layers: two update launches
    (3, 2, 40, (700, 30), 0.9),                  # no hidden layer: gathered rows on both sides
]


@pytest.mark.parametrize("P,K,B,dims,beta", CASES, ids=["P%d-B%d-%s" % (c[0], c[2], "-".join(map(str, c[3]))) for c in CASES])
def test_learner_loop_at_tile_edges(P, K, B, dims, beta):
    g, o = _pair(P, K, 0.05, 0.9, dims, B, False, 211)
    g.set_fused(False)
    if beta:
        g.set_learner_momentum(beta)
        g.set_params(g.params())                 # velocities start at zero
        o.beta, o.u = beta, np.zeros((o.P, o.n))
    _run_and_compare(g, o, dims, 2, TOL_FP32, "tiles %s" % (dims,))


@pytest.mark.parametrize("P,K,B,dims,beta", [
    (2, 2, 1, (20, 17, 8), 0.9),                 # one sample, one unit over a workgroup's sixteen, classes as one row of eight
    (3, 2, 17, (33, 15, 9), 0.0),                # one sample over the sixteen groups, fewer units than a workgroup, nine classes
    (2, 2, 80, (40, 64, 31, 16), 0.9),           # five samples per lane, sixteen classes
    (3, 2, 65, (100, 12), 0.0),                  # the head alone, on gathered rows
], ids=lambda v: "-".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_head_in_the_update_launch(P, K, B, dims, beta):
    test_learner_loop_at_tile_edges(P, K, B, dims, beta)


@pytest.mark.parametrize("P,K,B,dims", [
    (3, 2, 9, (129, 64, 4)),                     # two splits, one unit per lane
    (2, 2, 5, (512, 130, 10)),                   # eight splits, units beyond two per lane, odd batch
    (2, 2, 6, (70, 784, 127, 16)),               # nine splits, an odd number of units
    (1, 2, 33, (1024, 65, 2)),                   # sixteen splits
    (1, 2, 33, (2112, 65, 2)),                   # more: added up by a launch of their own
])
def test_split_product_finished_by_the_head(P, K, B, dims):
    test_learner_loop_at_tile_edges(P, K, B, dims, 0.0)
