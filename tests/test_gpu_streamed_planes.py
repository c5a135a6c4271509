"""Updates of weights whose planes, over all learners, do not stay in the memory-side cache: rows of whole 128-byte lines (streaming
accesses) and ragged ones (ordinary accesses), in each kernel that a layer's update can run in."""
import numpy as np
import pytest

from paper_2110_00625_amd import kavg
from tests.test_gpu_order_of_sums import _model, _order_shows
from tests.test_gpu_small import _pair
from tests.util import bf16_plane_bits, layer_slices

pytestmark = pytest.mark.gpu

# (HALVES: every other row begins in the middle of a line)
WHOLE, RAGGED, HALVES = (576, 1984, 320, 24), (584, 1976, 328, 24), (608, 2016, 352, 24)       # 1.78 M weights and more, 228 MB of bf16 planes over 64 learners
CASES = [
    # B, dims, learner momentum
    (33, RAGGED, 0.0),                # strips of up to 64 samples; the first layer in tiles of 64x128
    (100, RAGGED, 0.0),               # strips of up to 128 samples
    (136, RAGGED, 0.0),               # tiles of 128x128
    (264, RAGGED, 0.0),               # ... with the late master
    (264, WHOLE, 0.0),
    (33, HALVES, 0.0),                # ordinary accesses to strips and tiles of 64x128,
    (136, HALVES, 0.0),               # streaming ones in tiles of 128x128
    (264, HALVES, 0.0),
    (33, WHOLE, 0.9),                 # with velocities: all layers in one launch
    (33, RAGGED, 0.9),
    (136, RAGGED, 0.9),
    (136, WHOLE, 0.9),
    (400, RAGGED, 0.9),               # ... up to 400 rows
    (400, WHOLE, 0.9),
    (401, RAGGED, 0.9),               # a launch per layer
    (401, WHOLE, 0.9),
]


@pytest.mark.parametrize("B,dims,beta", CASES, ids=["B%d-%s-%g" % (c[0], "-".join(map(str, c[1])), c[2]) for c in CASES])
def test_streamed_and_cached_planes_end_the_same(B, dims, beta):
    """Integer data and weights, exact activations and back-propagated gradients: a learner among 64 ends a step with exactly what
    it ends with among 3, whose planes stay in the cache."""
    import torch
    X, y, w0 = _model(dims, 500, 331)
    assert _order_shows(dims, X, y, w0, B)
    replicas = []
    for P in (64, 3):
        g = kavg.MAvg(P, 1, 0.5, 0.9, dims, B, kavg.KAVG_BF16, index_seed=13)
        g.set_data(torch.from_numpy(bf16_plane_bits(X).view(np.int16)).cuda(), torch.from_numpy(y).cuda())
        if beta:
            g.set_learner_momentum(beta)
        g.set_params(w0)
        g.local_steps()
        replicas.append([g.replica(j) for j in range(3)])
        g.close()
    for j in range(3):
        assert np.any(replicas[0][j] != w0)
        assert np.array_equal(replicas[0][j], replicas[1][j]), "learner %d: %d of %d differ" % (
            j, np.sum(replicas[0][j] != replicas[1][j]), w0.size)


@pytest.mark.parametrize("B,dims", [(33, (576, 3072, 24)), (33, (584, 3048, 24)), (136, (584, 3048, 24)), (136, (576, 3072, 24))])
def test_velocities_over_two_steps(B, dims):
    """Against the oracle, on the scale of the steps taken.  Sums differ by 1e-6 and roundings that fall the other way by 2^-8 of
    a term.  A pre-activation that rounding moves across zero (about 1e-4 of them: the second step's weights) adds or drops one of
    B * units / 2 terms of an unordered sum, which is sqrt(2 / (B * units)) of the step in the 2-norm; 2^-5 allows 48 of them at
    33 samples.  Velocities left out are 0.4 of the step, a tile of 64x128 gone wrong is 0.07, the last piece of all rows 0.12."""
    P = 64
    g, o = _pair(P, 2, 0.1, 0.9, dims, B, True, 241)
    g.set_learner_momentum(0.9)
    g.set_params(g.params())                 # velocities start at zero
    o.beta, o.u = 0.9, np.zeros((o.P, o.n))
    start = g.params().astype(np.float64)
    g.local_steps()
    o.local_steps(learners=[0, P - 1])
    for j in (0, P - 1):
        got, want = g.replica(j) - start, np.asarray(o.replica(j)) - start
        for name, sl in layer_slices(dims):
            e = np.linalg.norm(got[sl] - want[sl]) / np.linalg.norm(want[sl])
            assert e < 2.0 ** -5, "%s of learner %d: %.3g" % (name, j, e)
