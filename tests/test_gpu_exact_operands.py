"""Weight gradients in mixed precision, from operands that both sides hold exactly: integer data and weights, and logits so
far apart that the softmax is 0 or 1.  Every sum below is then a sum of integers under 2^24 (times a power of two and, for
a batch that is none, the bf16 value of 1/B), so activations and back-propagated gradients round the same way here and in
the oracle, whatever the order of the sums, and a gradient can differ by its own fp32 sum only.  Sums of up to 256 terms
(positions of a convolution: some thousands) of 16-bit products, and the fp32 weight they are taken from: 2^-18 of the
largest step holds for both; a gradient rounded to bf16 on its way is off by 2^-9 of itself, which the test checks on the
oracle's."""
import numpy as np
import pytest

from oracle import conv_oracle as C
from oracle import mavg_oracle as O
from paper_2110_00625_amd import kavg
from tests import test_gpu_conv_flat, test_gpu_strip, test_gpu_update_group
from tests.test_gpu_conv import conv_slices
from tests.util import bf16_plane_bits, layer_slices

pytestmark = pytest.mark.gpu

BOUND = 2.0 ** -18
LR = 1024.0          # (steps of the size of the last layer's weights, 2^14: rounding the new weight to fp32 stays below the bound)


def _ternary(rng, shape, fan_in):
    """-1, 0, 1 with about 12 non-zeros per row at most"""
    keep = min(1.0, 12.0 / fan_in)
    return rng.integers(0, 2, size=shape) * 2.0 - 1.0, rng.random(shape) < keep


def _weights(rng, rows, fan_in, scale=1.0):
    sign, keep = _ternary(rng, (rows, fan_in), fan_in)
    return np.concatenate([(sign * keep * scale).ravel(), rng.integers(-2, 3, size=rows) * scale])


def _mlp_weights(rng, dims):
    """The last layer's weights are multiples of 2^14 and its biases differ by multiples of 256, no two by a multiple of
    2^14: the logits of a sample lie at least 256 apart."""
    out = [_weights(rng, dims[l], dims[l - 1], 16384.0 if l == len(dims) - 1 else 1.0) for l in range(1, len(dims))]
    out[-1][-dims[-1]:] += 256.0 * np.arange(dims[-1])
    assert dims[-1] <= 64
    return out


def _compare(g, o, P, slices):
    start = g.params().astype(np.float64)
    sample = sorted({0, 1, P - 1}) if P > 1 else [0]
    g.local_steps()
    o.local_steps(learners=sample)
    seen = 0
    for j in sample:
        got, want = g.replica(j).astype(np.float64) - start, np.asarray(o.replica(j)) - start
        for name, sl in slices:
            scale = max(np.max(np.abs(want[sl])), 1e-30)
            e = np.max(np.abs(got[sl] - want[sl])) / scale
            assert e < BOUND, "%s of learner %d: %.3g" % (name, j, e)
            rounded = O.rne_bf16(want[sl])
            seen += np.max(np.abs(rounded - want[sl])) / scale > 8 * BOUND
    assert seen > 0, "no tensor of this case would show a rounded gradient"


def _mlp(P, B, dims, seed, beta=0.0):
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    N = 40
    rng = np.random.default_rng(seed)
    X = rng.integers(-30, 31, size=(N, dims[0])).astype(np.float32)
    y = rng.integers(0, dims[-1], size=N).astype(np.int32)
    w0 = np.concatenate(_mlp_weights(rng, dims)).astype(np.float32)
    g = kavg.MAvg(P, 1, LR, 0.9, dims, B, kavg.KAVG_BF16, index_seed=seed)
    g.set_data(torch.from_numpy(bf16_plane_bits(X).view(np.int16)).cuda(), torch.from_numpy(y).cuda())
    if beta:
        g.set_learner_momentum(beta)
    g.set_params(w0)
    o = O.MAvgOracle(P, 1, LR, 0.9, dims, B, bf16=True, index_seed=seed, learner_momentum=beta)
    o.set_data(X, y)
    o.set_params(w0)
    return g, o


@pytest.mark.parametrize("P,B,dims", test_gpu_strip.CASES, ids=["B%d-%s" % (c[1], "-".join(map(str, c[2]))) for c in test_gpu_strip.CASES])
def test_strips(P, B, dims):
    g, o = _mlp(P, B, dims, 281)
    _compare(g, o, P, layer_slices(dims))
    g.close()


GROUPS = [(P, B, dims, beta) for P, K, B, dims, beta in test_gpu_update_group.CASES if dims[-1] > 1 and len(dims) < 6]


@pytest.mark.parametrize("P,B,dims,beta", GROUPS, ids=["B%d-%s-%g" % (c[1], "-".join(map(str, c[2])), c[3]) for c in GROUPS])
def test_grouped_updates(P, B, dims, beta):
    g, o = _mlp(P, B, dims, 291, beta)
    _compare(g, o, P, layer_slices(dims))
    g.close()


@pytest.mark.parametrize("P,B,H,W,channels,dims", test_gpu_conv_flat.CASES,
                         ids=["%dx%d-%s" % (c[2], c[3], "-".join(map(str, c[4]))) for c in test_gpu_conv_flat.CASES])
def test_convolutions(P, B, H, W, channels, dims):
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    N, seed = 24, 301
    spec = C.ConvSpec(H, W, channels, dims)
    rng = np.random.default_rng(seed)
    X = rng.integers(-30, 31, size=(N, H * W * channels[0])).astype(np.float32)
    y = rng.integers(0, dims[-1], size=N).astype(np.int32)
    w0 = np.concatenate([_weights(rng, channels[t], 9 * channels[t - 1]) for t in range(1, len(channels))]
                        + _mlp_weights(rng, dims)).astype(np.float32)
    g = kavg.MAvg(P, 1, LR, 0.9, dims, B, kavg.KAVG_BF16, index_seed=seed, conv=(H, W, channels))
    g.set_data(torch.from_numpy(bf16_plane_bits(X).view(np.int16).reshape(N, H, W, channels[0])).cuda(), torch.from_numpy(y).cuda())
    g.set_params(w0)
    o = C.make_oracle(P, 1, LR, 0.9, spec, B, bf16=True, index_seed=seed)
    o.set_data(X, y)
    o.set_params(w0)
    _compare(g, o, P, conv_slices(spec))
    g.close()
