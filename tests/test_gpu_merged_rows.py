"""Products with weights that all learners share run over the rows of all learners at once (gemm_bf16.hip, MERGED): tiles that
hold rows of several learners, rows and columns beyond the last tile, against the oracle."""
import pytest

from tests.test_gpu_deferred import TOL_BF16, _setup
from tests.util import replica_error

pytestmark = pytest.mark.gpu

CASES = [
    # P, K, B, dims, m
    (25, 3, 61, (128, 4096, 136, 17), 3),        # 1525 rows in tiles of 256 and 128, two slices; the data gradient 4096 wide
    (13, 2, 127, (192, 4104, 24), 2),            # a ragged last column tile, an odd batch
    (24, 2, 64, (64, 4096, 4096, 10), 2),        # one slice: the first layer stays per learner
]


@pytest.mark.parametrize("P,K,B,dims,m", CASES, ids=[str(c[3]) for c in CASES])
def test_local_steps(P, K, B, dims, m):
    g, o = _setup(P, K, B, dims, 57, m)
    g.local_steps()
    o.local_steps()
    for j in sorted({0, P // 2, P - 1}):
        e = replica_error(g.replica(j), o.replica(j), dims)
        assert e < TOL_BF16, "replica %d: %.3g" % (j, e)
    g.close()
