"""Forward pass, loss and data gradients of a small model in one launch (chain_bf16.hip) against the same steps as separate
launches (a profiled class takes them apart): every sum is taken in the same order, so the states agree bit for bit."""
import numpy as np
import pytest
import torch

from paper_2110_00625_amd import kavg, synth
from tests.test_gpu_small import _pair
from tests.util import chained_layers

pytestmark = pytest.mark.gpu

CASES = [
    # P, K, B, dims, learner momentum, layers in the launch
    (2, 2, 8, (64, 32, 32, 2), 0.0, 3),              # one whole workgroup, one set, one block; two classes
    (3, 2, 9, (72, 40, 16), 0.0, 2),                 # one row, eight inputs, eight units over; sixteen classes
    (2, 2, 1, (8, 8, 17), 0.0, 2),                   # the smallest layers; seventeen classes in padded columns
    (2, 2, 33, (448, 144, 10), 0.9, 2),              # seven sets (an odd number), the last workgroup with one row
    (3, 2, 20, (64, 544, 64, 20), 0.0, 3),           # seventeen blocks: a third turn of the wavefronts, forward and backward
    (2, 2, 11, (64, 544, 64, 10), 0.0, 3),           # ... below a head
    (2, 2, 8, (136, 264, 136, 100), 0.0, 2),         # nine blocks: a second turn; the first layer runs by itself
    (2, 2, 13, (200, 72, 302), 0.0, 2),              # ten blocks of logits
    (2, 2, 13, (200, 72, 552), 0.0, 2),              # eighteen
    (2, 2, 8, (128, 128, 128, 128, 128, 128, 5), 0.0, 6),    # as many layers as a launch takes
    (2, 1, 8, (64, 64, 64, 64, 64, 64, 64, 64, 3), 0.0, 6),  # more: the first two run one by one
    (2, 2, 16, (1032, 80, 64), 0.0, 2),              # gathered rows longer than one pass of a wavefront takes
    (2, 2, 16, (1032, 64, 64, 4), 0.0, 3),           # ... below a head of four classes
    (2, 2, 16, (3080, 80, 64), 0.0, 1),              # the last layer alone, its rows not gathered
]
CONVOLUTIONS = [
    # channels, hidden units, B, classes, layers in the launch
    ((8, 16), (24,), 5, 4, 2),
    ((8, 16), (24,), 5, 40, 2),
    ((8, 32, 128), (264,), 11, 10, 2),
    ((8, 32, 128), (264, 64), 11, 4, 3),
    ((8, 32, 128), (264,), 11, 40, 2),
    ((8, 32, 128), (544,), 11, 16, 2),               # a third turn of the wavefronts; the head above the gradient of the mean
]


def _state(g, profiled):
    if profiled:
        g.profile(["forward"])
    g.local_steps()
    g.meta_update()
    g.local_steps()
    return [g.params(), g.momentum(), g.losses()] + [g.replica(j) for j in range(g.P)]


@pytest.mark.parametrize("P,K,B,dims,beta,layers", CASES, ids=["B%d-%s-%g" % (c[2], "-".join(map(str, c[3])), c[4]) for c in CASES])
def test_mlp(P, K, B, dims, beta, layers):
    assert chained_layers(P, B, dims) == layers          # else both sides below are the same launches
    states = []
    for profiled in (False, True):
        g, _ = _pair(P, K, 0.05, 0.9, dims, B, True, 77)
        if beta:
            g.set_learner_momentum(beta)
            g.set_params(g.params())
        states.append(_state(g, profiled))
        g.close()
    for a, b in zip(*states):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("channels,hidden,B,C,layers", CONVOLUTIONS, ids=["-".join(map(str, c[0] + c[1])) + "-%d" % c[3] for c in CONVOLUTIONS])
def test_behind_convolutions(channels, hidden, B, C, layers):
    P, K, H, W, N = 2, 2, 7, 9, 50
    dims = (channels[-1],) + hidden + (C,)
    assert chained_layers(P, B, dims, True) == layers
    gen = torch.Generator(device="cuda").manual_seed(5)
    X = torch.randn(N, H, W, channels[0], generator=gen, device="cuda").to(torch.bfloat16)
    y = torch.randint(0, C, (N,), generator=gen, device="cuda").to(torch.int32)
    n_conv = sum(channels[t] * (9 * channels[t - 1] + 1) for t in range(1, len(channels)))
    w0 = np.concatenate([(np.random.default_rng(3).standard_normal(n_conv) * 0.1).astype(np.float32),
                         synth.he_normal_params(dims, 4).astype(np.float32)])
    states = []
    for profiled in (False, True):
        g = kavg.MAvg(P, K, 0.05, 0.9, dims, B, kavg.KAVG_BF16, index_seed=6, conv=(H, W, channels))
        g.set_data(X, y)
        g.set_params(w0)
        states.append(_state(g, profiled))
        g.close()
    for a, b in zip(*states):
        assert np.array_equal(a, b)
