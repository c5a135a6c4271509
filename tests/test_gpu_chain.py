"""Forward pass, loss and data gradients of a small model in one launch (chain_bf16.hip) against the same steps as separate
launches (a profiled class takes them apart): every sum is taken in the same order, so the states agree bit for bit."""
import numpy as np
import pytest
import torch

from paper_2110_00625_amd import kavg, synth
from tests.test_gpu_small import _pair

pytestmark = pytest.mark.gpu

CASES = [
    # P, K, B, dims, learner momentum
    (2, 2, 8, (64, 32, 2), 0.0),                     # one whole workgroup, one set, one block
    (3, 2, 9, (72, 40, 16), 0.0),                    # one row, eight inputs, eight units over; sixteen classes
    (2, 2, 1, (8, 8, 17), 0.0),                      # the smallest layers; seventeen classes in padded columns
    (2, 2, 33, (448, 144, 10), 0.9),                 # seven sets (an odd number), the last workgroup with one row
    (3, 2, 20, (136, 264, 520, 100), 0.0),           # nine and seventeen blocks: a second and a third turn of the wavefronts
    (2, 2, 13, (200, 72, 302), 0.0),                 # ten blocks of logits
    (2, 2, 8, (128, 128, 128, 128, 128, 128, 5), 0.0),       # as many layers as a launch takes
    (2, 1, 8, (64, 64, 64, 64, 64, 64, 64, 64, 3), 0.0),     # more: the first two run one by one
    (2, 2, 16, (3080, 80, 64), 0.0),                 # long rows
]


def _state(g, profiled):
    if profiled:
        g.profile(["forward"])
    g.local_steps()
    g.meta_update()
    g.local_steps()
    return [g.params(), g.momentum(), g.losses()] + [g.replica(j) for j in range(g.P)]


@pytest.mark.parametrize("P,K,B,dims,beta", CASES, ids=["B%d-%s-%g" % (c[2], "-".join(map(str, c[3])), c[4]) for c in CASES])
def test_mlp(P, K, B, dims, beta):
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


@pytest.mark.parametrize("C", [4, 40])
@pytest.mark.parametrize("channels,hidden,B", [((8, 16), 24, 5), ((8, 32, 128), 264, 11)])
def test_behind_convolutions(channels, hidden, B, C):
    P, K, H, W, N = 2, 2, 7, 9, 50
    dims = (channels[-1], hidden, C)
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
