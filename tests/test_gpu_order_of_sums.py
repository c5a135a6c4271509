"""What a learner computes depends on neither how many others there are nor, with that, on which kernels run: many learners
of this model take the strip kernel, the one-layer update and the head's update (weights that stream), few take the separate
data gradient and all updates in one launch.  Integer data and weights make every activation and every back-propagated
gradient exact, whatever the order of its sum; the gradients of the weights span too many bits for that, so they come out
bit for bit the same only if their sums are taken in the same order."""
import numpy as np
import pytest

from oracle import mavg_oracle as O
from paper_2110_00625_amd import kavg
from tests.util import bf16_plane_bits

pytestmark = pytest.mark.gpu


def _model(dims, N, seed):
    """Hidden layers: rows of -1, 0, 1 with about 12 non-zeros.  Last layer: 2^14 times random values of eight bits, so that
    logits lie far apart (the softmax is 0 or 1) and the gradients carry as many bits as bf16 holds."""
    rng = np.random.default_rng(seed)
    X = (rng.integers(-100, 101, size=(N, dims[0])) * 2.0 ** rng.integers(0, 8, size=(N, 1))).astype(np.float32)    # samples of all sizes
    y = rng.integers(0, dims[-1], size=N).astype(np.int32)
    w0 = []
    for l in range(1, len(dims)):
        W = (rng.integers(0, 2, size=(dims[l], dims[l - 1])) * 2.0 - 1.0) * (rng.random((dims[l], dims[l - 1])) < 12.0 / dims[l - 1])
        if l == len(dims) - 1:
            W = 2.0 ** 14 * (rng.integers(0, 2, size=W.shape) * 2.0 - 1.0) * (1.0 + rng.integers(0, 128, size=W.shape) / 128.0)
        w0 += [W.ravel(), rng.integers(-2, 3, size=dims[l]).astype(float)]
    return X, y, np.concatenate(w0).astype(np.float32)


def _order_shows(dims, X, y, w0, B):
    """The gradient of the second layer in float32, samples in one ascending chain and in two halves."""
    Ws, bs = O.unpack(w0.astype(np.float64), dims)
    rows = np.arange(B)
    Zs, As = O.forward([O.rne_bf16(W) for W in Ws], bs, X[rows].astype(np.float64), O.rne_bf16)
    top = np.sort(Zs[-1], axis=1)
    assert np.min(top[:, -1] - top[:, -2]) > 200.0
    dZ = O.rne_bf16(O.softmax_cross_entropy(Zs[-1], y[rows])[1])
    for l in range(len(Ws) - 1, 1, -1):
        dZ = O.rne_bf16((dZ @ Ws[l]) * (As[l] > 0))
    terms = (dZ[:, :128, None] * As[1][:, None, :128]).astype(np.float32)
    chain = lambda t: np.add.accumulate(t, axis=0, dtype=np.float32)[-1]
    return np.any(chain(terms) != chain(terms[:B // 2]) + chain(terms[B // 2:]))


@pytest.mark.parametrize("B,beta", [(64, 0.0), (100, 0.0), (256, 0.0), (100, 0.9)])
@pytest.mark.parametrize("C", [3, 10, 16])
def test_many_learners_and_few_take_the_same_steps(B, beta, C):
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    dims = (256, 1024, 1024, C)
    many, few, N = 80, 3, 500                                 # 80 learners: 213 MB of bf16 planes, 640 strips
    X, y, w0 = _model(dims, N, 311 + C)
    assert _order_shows(dims, X, y, w0, B)
    replicas = []
    for P in (many, few):
        g = kavg.MAvg(P, 1, 0.5, 0.9, dims, B, kavg.KAVG_BF16, index_seed=13)
        g.set_data(torch.from_numpy(bf16_plane_bits(X).view(np.int16)).cuda(), torch.from_numpy(y).cuda())
        if beta:
            g.set_learner_momentum(beta)
        g.set_params(w0)
        g.local_steps()
        replicas.append([g.replica(j) for j in range(few)])
        g.close()
    for j in range(few):
        assert np.any(replicas[0][j] != w0)
        assert np.array_equal(replicas[0][j], replicas[1][j]), "learner %d: %d of %d differ" % (
            j, np.sum(replicas[0][j] != replicas[1][j]), w0.size)


@pytest.mark.parametrize("B", [40, 64, 100, 128])
@pytest.mark.parametrize("C", [10, 24])
def test_strips_of_small_launches_take_every_sum_as_the_separate_kernels(B, C):
    """240 strips, so few that the separate data gradient would split its contraction: on ordinary data, over three steps, a
    learner among thirty (strips) ends with exactly what it ends with among three (separate kernels)."""
    import torch
    from paper_2110_00625_amd import synth
    dims, K, N = (256, 1024, 1024, C), 3, 600
    data = synth.make_dataset(N, dims[0], C, bf16=True, seed_data=321, seed_teacher=322, teacher_hidden=32)
    w0 = synth.he_normal_params(dims, 323)
    replicas = []
    for P in (30, 3):
        g = kavg.MAvg(P, K, 0.05, 0.9, dims, B, kavg.KAVG_BF16, index_seed=17)
        g.set_data(torch.from_numpy(data["Xbits"].view(np.int16)).cuda(), torch.from_numpy(data["y"]).cuda())
        g.set_params(w0)
        g.local_steps()
        replicas.append([g.replica(j) for j in range(3)])
        g.close()
    for j in range(3):
        assert np.array_equal(replicas[0][j], replicas[1][j]), "learner %d" % j
