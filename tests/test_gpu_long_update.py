"""Updates that contract over more than 256 rows (gemm_bf16.hip, LATE), as a refresh of deferred updates does: a last slice
of few rows, ragged tiles on both sides, tile rows behind the last whole group of eight, both kinds of access to the bf16 plane --
against the oracle.  Cases of few tiles run in the tiles of shorter updates."""
import pytest

from tests.test_gpu_deferred import TOL_BF16, _setup
from tests.util import replica_error

pytestmark = pytest.mark.gpu

CASES = [
    # P, K, B, dims, m
    (2, 5, 53, (136, 1032, 264, 24), 5),         # 265 rows, few tiles
    (3, 4, 65, (264, 200, 136, 10), 4),          # 260 rows, a thin last layer (few tiles: 128x64, as with fewer rows)
    (13, 2, 131, (136, 2568, 264, 24), 2),       # 262 rows; 546 and 819 tiles, 21 tile rows, planes in the cache
    (2, 3, 256, (8, 16, 40), 2),                 # operands narrower than a tile; 512 rows, then 256 (few tiles)
    (520, 2, 131, (8, 16, 40), 2),               # ... many tiles of one layer each
    # planes of all learners beyond the cache; 262 rows.  (Two steps: over five steps of 57 rows at this width, with the same
    # bits as a kernel that requests the master first, roundings that fall the other way flip ReLU masks: 3.6e-2 off the
    # oracle.  Two steps: 5.4e-3.)
    (26, 2, 131, (520, 4104, 456, 24), 2),
]


@pytest.mark.parametrize("P,K,B,dims,m", CASES, ids=[str(c[3]) for c in CASES])
def test_refresh(P, K, B, dims, m):
    g, o = _setup(P, K, B, dims, 61, m)
    g.local_steps()
    o.local_steps()
    for j in sorted({0, P // 2, P - 1}):
        e = replica_error(g.replica(j), o.replica(j), dims)
        assert e < TOL_BF16, "replica %d: %.3g" % (j, e)
    g.close()
