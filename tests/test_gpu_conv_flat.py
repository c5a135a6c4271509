"""Convolutions on images of any size (conv_flat.hip, conv_flat_wgrad.hip) where their tiles, rings and channel groups end,
against the oracle, on the scale of one local step: replica - start = -lr * gradient."""
import numpy as np
import pytest

from oracle import conv_oracle as C
from paper_2110_00625_amd import kavg
from tests.test_gpu_conv import _setup, conv_slices

pytestmark = pytest.mark.gpu

CASES = [
    # P, B, H, W, channels, dims
    (2, 3, 5, 6, (8, 16), (16, 10)),                 # one convolution on small images: every tile holds several of them
    (40, 1, 4, 4, (8, 8, 16), (16, 10)),             # many learners, a range shorter than a slice
    (2, 4, 9, 28, (8, 32, 64), (64, 10)),
    (1, 2, 7, 33, (8, 24, 40, 72), (72, 12)),        # channels between the tile sizes: two, three and six slabs
    (1, 2, 6, 62, (8, 64, 64), (64, 10)),            # the widest image that a ring of 256 rows holds
    (1, 2, 5, 64, (8, 96, 128), (128, 10)),          # a ring of 512 rows; 96 and 128 channels out, two groups in
    (2, 2, 6, 20, (8, 128, 96, 16), (16, 10)),       # 128 and 96 contraction channels
    (1, 2, 5, 32, (8, 32, 64), (64, 10)),            # 32 pixels wide, a height that the tile kernels for that width refuse
    (1, 2, 6, 10, (8, 136, 24), (24, 10)),           # 136 channels: one side of each layer on the generic kernels
    (1, 1, 3, 150, (8, 16, 48), (48, 10)),           # wide and low
    (1, 40, 1, 1, (8, 32, 32), (32, 10)),            # images of one pixel: margins everywhere
    (1, 16, 28, 28, (8, 128, 128, 128, 128), (128, 10)),     # partial sums of 30 MB per layer: the SGD steps in two launches
]


@pytest.mark.parametrize("P,B,H,W,channels,dims", CASES, ids=["%dx%d-%s" % (c[2], c[3], "-".join(map(str, c[4]))) for c in CASES])
def test_one_step(P, B, H, W, channels, dims):
    """Both sides start from the same state and round at the same points, so they differ by fp32 sums (1e-6 of the step)
    and, rarely, by a value whose rounding to bf16 falls the other way: 2^-8 of one term of a gradient element."""
    g, o, spec = _setup(P, 1, B, H, W, channels, dims, 75, lr=0.5)
    start = g.params().astype(np.float64)
    g.local_steps()
    o.local_steps()
    for j in sorted({0, P - 1}):
        got, want = g.replica(j) - start, np.asarray(o.replica(j)) - start
        for name, sl in conv_slices(spec):
            e = np.max(np.abs(got[sl] - want[sl])) / max(np.max(np.abs(want[sl])), 1e-30)
            print("  learner %d %-8s %.3g" % (j, name, e))
            assert e < 2.0 ** -8, "%s of learner %d: %.3g" % (name, j, e)


LAST = [
    # the last convolution: bits and partial sums in place of its activations
    (2, 9, 1, 2, (8, 16), (16, 10)),                 # images of six positions: 23 of them in the 128 of a wavefront
    (2, 70, 2, 1, (8, 8, 128), (128, 3)),        # more images than a tile holds; two tiles per learner
    (1, 3, 3, 4, (8, 8, 72), (72, 40)),              # a last word of eight channels
    (3, 3, 32, 32, (8, 32), (32, 10)),               # one convolution, 32 pixels wide: its gradient from the bits as well
    (2, 5, 32, 32, (8, 32, 32, 64), (64, 10)),       # an odd batch: the gradients of the kernels for any width
    (2, 4, 16, 32, (8, 64, 64, 128), (128, 17)),     # an even one: those for 32 pixels, from bits
    (1, 2, 13, 47, (8, 40, 104), (104, 10)),
    (1, 2, 3, 80, (8, 48, 64), (64, 10)),            # the widest images whose three slabs come at once
    (1, 3, 2, 468, (8, 16), (16, 10)),               # the widest images of all, four wavefronts side by side
    (1, 2, 2, 596, (8, 16, 72), (72, 10)),           # ... and two
]


@pytest.mark.parametrize("P,B,H,W,channels,dims", LAST, ids=["%dx%d-%s" % (c[2], c[3], "-".join(map(str, c[4]))) for c in LAST])
def test_last_convolution(P, B, H, W, channels, dims):
    test_one_step(P, B, H, W, channels, dims)


@pytest.mark.parametrize("n_conv", [8, 9])
def test_steps_of_many_convolutions(n_conv):
    """The SGD steps of up to eight convolutions run in the launch of the MLP's updates, those of more in launches of their own, and
    with the updates profiled layer by layer eight do as well.  One step of each of two contexts: the same bits.  Tolerance as in
    test_one_step."""
    channels, dims = (8,) + (16,) * n_conv, (16, 8, 10)
    g, o, spec = _setup(2, 1, 6, 5, 7, channels, dims, 79, lr=0.5)
    apart, _, _ = _setup(2, 1, 6, 5, 7, channels, dims, 79, lr=0.5)
    start = g.params().astype(np.float64)
    apart.profile(["update"])
    for c in (g, apart, o):
        c.local_steps()
    apart.profile([])
    for j in range(2):
        got, want = g.replica(j) - start, np.asarray(o.replica(j)) - start
        assert np.array_equal(g.replica(j), apart.replica(j))
        for name, sl in conv_slices(spec):
            assert np.any(want[sl] != 0.0)
            e = np.linalg.norm(got[sl] - want[sl]) / np.linalg.norm(want[sl])
            assert e < 2.0 ** -8, "%s of learner %d: %.3g" % (name, j, e)


LARGE = [
    # the mean over the positions out of many partial sums, one per 64 positions: sixteen and eight at a time
    (2, 2, 60, 40, (8, 16), (16, 10)),               # 40 of them
    (1, 2, 31, 33, (8, 8, 24), (24, 10)),            # 17, images at the ends of wavefronts
    (1, 3, 17, 31, (8, 8, 24), (24, 32, 10)),        # nine, the mean in the launch of the MLP
]


@pytest.mark.parametrize("P,B,H,W,channels,dims", LARGE, ids=["%dx%d-%s" % (c[2], c[3], "-".join(map(str, c[4]))) for c in LARGE])
def test_mean_of_large_images(P, B, H, W, channels, dims):
    test_one_step(P, B, H, W, channels, dims)


MANY = [
    # More than 256 workgroups: whole ones (the cases above have half as many positions each); two learners are checked.
    (257, 3, 5, 6, (8, 16, 40), (40, 10)),           # images across and beside the ends of tiles
    (257, 70, 2, 1, (8, 8, 128), (128, 3)),          # 22 images of six positions to a wavefront
    (130, 5, 9, 13, (8, 72, 64), (64, 10)),          # three slabs at a time; 64 and 128 channels out
    (129, 3, 7, 41, (8, 64, 24), (24, 10)),          # four slabs, the widest images (in 512 positions) that take them
    (257, 1, 3, 80, (8, 48, 128, 40), (40, 10)),
    (512, 2, 32, 32, (8, 64, 64, 128), (128, 17)),   # 32 pixels wide, forward pass and data gradient on the kernels for any width
]


@pytest.mark.parametrize("P,B,H,W,channels,dims", MANY, ids=["%dx%d-%s" % (c[2], c[3], "-".join(map(str, c[4]))) for c in MANY])
def test_whole_workgroups(P, B, H, W, channels, dims):
    """Tolerance as in test_one_step."""
    g, o, spec = _setup(P, 1, B, H, W, channels, dims, 76, lr=0.5)
    start = g.params().astype(np.float64)
    g.local_steps()
    o.local_steps(learners=[0, P - 1])
    for j in (0, P - 1):
        got, want = g.replica(j) - start, np.asarray(o.replica(j)) - start
        for name, sl in conv_slices(spec):
            e = np.max(np.abs(got[sl] - want[sl])) / max(np.max(np.abs(want[sl])), 1e-30)
            print("  learner %d %-8s %.3g" % (j, name, e))
            assert e < 2.0 ** -8, "%s of learner %d: %.3g" % (name, j, e)
    g.close()


@pytest.mark.parametrize("size,bad", [(3, 0), (3, 7), (12, 2)], ids=["first-of-eight", "last-of-eight", "two-tiles"])
def test_an_infinite_activation_stays_in_its_image(size, bad):
    """One image whose first output channel overflows bf16.  Every hidden unit takes that channel with a negative weight, so
    the image's hidden layer is zero and its loss log C, and the losses of the other images, whose sums over the positions are
    formed beside its own, are what they are without it."""
    torch = pytest.importorskip("torch")
    B, channels, dims = 9, (8, 16), (16, 8, 3)
    spec = C.ConvSpec(size, size, channels, dims)
    rng = np.random.default_rng(21)
    X = torch.from_numpy(rng.standard_normal((B, size, size, 8)).astype(np.float32)).to(torch.bfloat16)
    X[bad] = 0.0
    X[bad, :, :, 0] = 3e38
    y = rng.integers(0, 3, size=B).astype(np.int32)
    w = (rng.standard_normal(spec.num_params()) * 0.3).astype(np.float32)
    convs, Ws, bs = C.unpack(w, spec)                        # (views into w)
    convs[0][0][...] *= np.arange(8) > 0                     # input channel 0: the centre tap of output channel 0 alone
    convs[0][0][0, 1, 1, 0] = 4.0
    Ws[0][:, 0] = -0.5
    bs[0][:], bs[1][:] = 1.0, 0.0
    w = w.astype(np.float32)

    g = kavg.MAvg(2, 1, 0.0, 0.0, dims, B, kavg.KAVG_BF16, index_seed=1, conv=(size, size, channels))
    g.set_data(X.cuda(), torch.from_numpy(y).cuda())
    g.set_params(w)
    g.set_indices(torch.arange(B, dtype=torch.int32, device="cuda").repeat(2))
    g.local_steps()
    others = [i for i in range(B) if i != bad]
    loss, _ = C.minibatch_gradient(w.astype(np.float64), spec, X.float().numpy().reshape(B, -1)[others], y[others], bf16=True)
    want = (loss * (B - 1) + np.log(3.0)) / B
    assert abs(loss - np.log(3.0)) > 0.02                    # (what the others would have if their hidden layers were lost)
    assert np.max(np.abs(g.losses() - want)) < 1e-3, (g.losses(), want, loss)
    g.close()


def test_mean_over_more_than_2_to_the_31_outputs():
    """256 learners of 65 536 images of two pixels and 128 channels: 2^31 means."""
    P, B, channels, dims = 256, 65536, (8, 128), (128, 10)
    g, o, spec = _setup(P, 1, B, 1, 2, channels, dims, 78, lr=0.5)
    start = g.params().astype(np.float64)
    g.local_steps()
    sample = [0, 127, 128, P - 1]
    o.local_steps(learners=sample)
    for j in sample:
        got, want = g.replica(j) - start, np.asarray(o.replica(j)) - start
        for name, sl in conv_slices(spec):
            e = np.max(np.abs(got[sl] - want[sl])) / max(np.max(np.abs(want[sl])), 1e-30)
            assert e < 2.0 ** -8, "%s of learner %d: %.3g" % (name, j, e)      # (as above)
    g.close()


def test_profile_counts_the_packing_of_the_weights():
    """A step's forward launches: the packed weights, two convolutions, the mean over the positions (the last layer of ten
    classes runs in the head kernels)."""
    g, _, _ = _setup(2, 2, 4, 9, 28, (8, 32, 64), (64, 10), 77)
    g.profile(["forward"])
    g.local_steps()
    assert g.profile_read()["forward"][1] == 2 * 4
    g.profile([])
    g.local_steps()
    assert np.all(np.isfinite(g.losses()))
