"""A gradient that overflows bf16 in one channel of a convolution leaves the weight and bias gradients of its other channels alone
(images 32 pixels wide: conv_first.hip, conv_wgrad.hip)."""
import numpy as np
import pytest

from oracle import conv_oracle as C
from tests.test_gpu_conv import _setup, conv_slices

pytestmark = pytest.mark.gpu

CHANNELS, DIMS = (8, 32, 64, 64), (64, 16, 3)
CASES = [(1, 3), (1, 20), (2, 3), (2, 36), (3, 20), (3, 35)]     # convolution, channel (of a block of 32: either half)


@pytest.mark.parametrize("t,bad", CASES)
def test_an_infinite_gradient_stays_in_its_channel(t, bad):
    """Channel `bad` of convolution t is 1e-30 everywhere, and one unit above it takes it with a weight so large that its gradient is
    infinite and the unit itself is not: the unit then decides the class, and its gradient is some hundreds.  (64 learners of four images: the
    weight gradients run on the kernels for 32 pixels.)  The other channels' steps are compared as in the step tests: fp32 sums in another
    order (1e-6) and a rounding to bf16 that falls the other way, 2^-8 of one term."""
    P, B, H, W = 64, 4, 8, 32
    g, o, spec = _setup(P, 1, B, H, W, CHANNELS, DIMS, 83, lr=0.5, mu=0.0)
    w = g.params().astype(np.float64)
    convs, Ws, bs = C.unpack(w, spec)                            # (views into w)
    convs[t - 1][0][bad], convs[t - 1][1][bad] = 0.0, 1e-30
    Ws[1][...] *= 1e3
    if t == len(convs):
        Ws[0][:, bad] = 0.0
        Ws[0][0, bad] = 3e37
    else:
        convs[t][0][..., bad] = 0.0
        convs[t][0][0, 1, 1, bad] = 2e38
        for Wc, _ in convs[t + 1:]:                              # output channel 0 of the layer above, alone, up to hidden unit 0
            Wc[..., 0] = 0.0
            Wc[0, 1, 1, 0] = 1e2
        Ws[0][:, 0] = 0.0
        Ws[0][0, 0] = 1e2
    w = w.astype(np.float32)
    g.set_params(w)
    o.set_params(w)
    g.local_steps()
    sample = (0, P - 1)
    o.local_steps(learners=list(sample))
    others = np.arange(CHANNELS[t]) != bad
    for j in sample:
        got, want = (np.asarray(r, dtype=np.float64) - w for r in (g.replica(j), o.replica(j)))
        for name, sl in conv_slices(spec):
            if name.startswith("conv%d." % t):
                a, b = (v[sl].reshape(CHANNELS[t], -1) for v in (got, want))
                if name.endswith(".b"):
                    assert not np.isfinite(a[bad, 0])            # (the gradient did overflow)
                e = np.max(np.abs(a - b)[others]) / np.max(np.abs(b[others]))
                assert np.all(np.isfinite(a[others])) and e < 2.0 ** -8, "%s of learner %d: %.3g" % (name, j, e)
    g.close()
