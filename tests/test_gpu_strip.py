"""Data gradient and update of a layer in one pass over its weights (strip_bf16.hip), at the sizes where strips, chunks and
batches end, against the oracle on the scale of one local step: replica - start = -lr * gradient.  The kernel takes a
layer when its strips of 128 inputs, over all learners, fill the chip; 200 learners do with one strip each."""
import numpy as np
import pytest

from tests.test_gpu_small import _pair
from tests.util import layer_slices

pytestmark = pytest.mark.gpu

CASES = [
    # P, B, dims
    (200, 3, (40, 136, 72, 24)),         # two strips, the second one piece wide; chunks of 32 units, the last one 8; 24 classes
    (200, 64, (40, 128, 256, 17)),       # a whole strip, 64 samples, 17 classes in padded columns
    (200, 65, (40, 264, 96, 24)),        # three strips, one sample over 64; three chunks, all of one round of the loop
    (200, 128, (40, 72, 40, 10)),        # 128 samples, the last layer on the head kernels
    (200, 129, (40, 136, 104, 24)),      # one sample over 128
    (200, 256, (40, 128, 8, 40)),        # 256 samples; a layer of eight units: one chunk
]


@pytest.mark.parametrize("P,B,dims", CASES, ids=["B%d-%s" % (c[1], "-".join(map(str, c[2]))) for c in CASES])
def test_one_step(P, B, dims):
    """Both sides start from the same state and round at the same points, so they differ by fp32 sums (1e-6 of the step)
    and, rarely, by a value whose rounding to bf16 falls the other way: 2^-8 of one term of a gradient element."""
    g, o = _pair(P, 1, 0.5, 0.9, dims, B, True, 221)
    start = g.params().astype(np.float64)
    sample = [0, 1, P // 2, P - 1]
    g.local_steps()
    o.local_steps(learners=sample)
    for j in sample:
        got, want = g.replica(j) - start, np.asarray(o.replica(j)) - start
        for name, sl in layer_slices(dims):
            e = np.max(np.abs(got[sl] - want[sl])) / max(np.max(np.abs(want[sl])), 1e-30)
            assert e < 2.0 ** -8, "%s of learner %d: %.3g" % (name, j, e)
