"""Forward products of launches that give each compute unit one workgroup or little more (gemm_bf16.hip, DEEP and the tile rule), at the
sizes where their slices of 128, tiles and bounds end, against the oracle on the scale of one local step: replica - start."""
import numpy as np
import pytest

from tests.test_gpu_small import _pair
from tests.util import chained_layers, layer_slices

pytestmark = pytest.mark.gpu

CASES = [
    # P, B, dims
    (2, 70, (264, 392, 520, 648, 24)),       # 64x64 tiles, four slices in flight: contractions of 3, 4, 5 slices, each ending in a piece of 8
    (3, 65, (384, 512, 640, 24)),            # ... of 3, 4 and 5 whole slices
    (2, 130, (264, 2728, 17)),               # 258 workgroups of 64x64: two slices in flight
    (4, 130, (1032, 1288, 24)),              # 128x64 tiles in two k groups, 168 of them: 9 slices, rows and columns beyond the last tile
    (4, 128, (1024, 4096, 10)),              # ... 256 of them, whole ones
    (13, 70, (136, 2504, 24)),               # 260 tiles of 128x128, the last column tile ragged
]


@pytest.mark.parametrize("P,B,dims", CASES, ids=["B%d-%s" % (c[1], "-".join(map(str, c[2]))) for c in CASES])
def test_one_step(P, B, dims):
    """Both sides start from the same state and round at the same points, so a step differs by fp32 sums (1e-6 of it) and,
    rarely, by a value whose rounding to bf16 falls the other way: 2^-8 of one term of a gradient element."""
    assert not chained_layers(P, B, dims)    # (a forward launch per layer)
    g, o = _pair(P, 1, 0.1, 0.9, dims, B, True, 251)
    start = g.params().astype(np.float64)
    sample = sorted({0, P - 1})
    g.local_steps()
    o.local_steps(learners=sample)
    for j in sample:
        got, want = g.replica(j) - start, np.asarray(o.replica(j)) - start
        for name, sl in layer_slices(dims):
            e = np.max(np.abs(got[sl] - want[sl])) / max(np.max(np.abs(want[sl])), 1e-30)
            assert e < 2.0 ** -8, "%s of learner %d: %.3g" % (name, j, e)
