"""All updates of a local step in one launch (update_bf16.hip) at the sizes where its tiles (64 x 128), slices of 64 samples
and groups of eight layers end, against the oracle on the scale of the steps taken: replica - start."""
import numpy as np
import pytest

from tests.test_gpu_small import _pair
from tests.util import layer_slices

pytestmark = pytest.mark.gpu

CASES = [
    # P, K, B, dims, learner momentum
    (3, 1, 64, (128, 64, 10), 0.0),              # whole tiles, one whole slice, the last layer beside it
    (3, 1, 65, (136, 72, 17), 0.0),              # one piece, eight units and one sample over; 17 classes in padded columns
    (2, 1, 129, (8, 8, 1), 0.0),                 # the smallest layers, three slices
    (2, 1, 200, (264, 200, 136, 40), 0.0),       # three column tiles, four row tiles
    (1, 1, 7, (64, 24, 24, 24, 24, 24, 24, 24, 24, 10), 0.0),       # nine layers: two launches
    (2, 1, 33, (120, 24), 0.0),                  # no hidden layer: gathered rows only
    (2, 2, 70, (200, 136, 24), 0.9),             # momentum over two steps
    (3, 2, 9, (3080, 4104, 24), 0.9),            # velocities and lo planes that exceed the memory-side cache
]


@pytest.mark.parametrize("P,K,B,dims,beta", CASES, ids=["B%d-%s-%g" % (c[2], "-".join(map(str, c[3])), c[4]) for c in CASES])
def test_steps(P, K, B, dims, beta):
    """Both sides start from the same state and round at the same points, so a step differs by fp32 sums (1e-6 of it) and,
    rarely, by a value whose rounding to bf16 falls the other way: 2^-8 of one term of a gradient element."""
    g, o = _pair(P, K, 0.1, 0.9, dims, B, True, 231)
    if beta:
        g.set_learner_momentum(beta)
        g.set_params(g.params())                 # velocities start at zero
        o.beta, o.u = beta, np.zeros((o.P, o.n))
    start = g.params().astype(np.float64)
    g.local_steps()
    o.local_steps()
    for j in sorted({0, P - 1}):
        got, want = g.replica(j) - start, np.asarray(o.replica(j)) - start
        for name, sl in layer_slices(dims):
            e = np.max(np.abs(got[sl] - want[sl])) / max(np.max(np.abs(want[sl])), 1e-30)
            assert e < K * 2.0 ** -8, "%s of learner %d: %.3g" % (name, j, e)
