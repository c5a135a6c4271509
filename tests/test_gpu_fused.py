"""Small fp32 models: all K local steps of Algorithm 1 in one launch (kavg_fused) against the oracle
and against the launch-per-layer path of the same library."""
import os
import re

import numpy as np
import pytest

from paper_2110_00625_amd import kavg
from tests.test_gpu_small import TOL_FP32, _pair, _run_and_compare, _torch
from tests.util import flat_error

pytestmark = pytest.mark.gpu

CASES = [
    # P, K, B, dims
    (4, 4, 32, (3072, 64, 10)),        # the shape of the smallest workload: 16 workgroups of 192 columns per learner
    (3, 3, 19, (200, 40, 7)),          # ragged everywhere: odd batch, 40 units (split by units: three groups, the last one 8)
    (2, 2, 64, (64, 64, 16)),          # full batch, every class (four groups of units)
    (5, 3, 7, (132, 8, 3)),            # fewer rows and units than a matrix-instruction block (one group)
    (1, 5, 33, (1000, 33, 2)),         # a single learner, batch one over half the tile
    (2, 3, 64, (4000, 64, 16)),        # 21 chunks of 192 columns (the last one 160 wide), full batch
    (3, 2, 50, (1600, 48, 9)),         # 13 chunks of 128 columns (the last one 64 wide)
]


# shapes that the split by inputs runs (kavg_fused 1), where its chunks, rows and units end
BY_INPUTS = [
    (3, 3, 19, (520, 40, 7)),          # last chunk 8 columns wide, odd batch, 40 units
    (5, 3, 7, (516, 8, 3)),            # last chunk 4 columns wide, fewer rows than a matrix-instruction block
    (20, 2, 64, (64, 64, 16)),         # one workgroup per learner, every limit reached
    (70, 2, 20, (40, 33, 10)),         # one chunk of 40 columns, 70 learners
    (40, 3, 17, (196, 64, 10)),        # 40 learners of four chunks, the last one 4 columns wide
]


@pytest.mark.parametrize("P,K,B,dims", BY_INPUTS, ids=[str(c[3]) for c in BY_INPUTS])
def test_split_by_inputs(P, K, B, dims):
    torch = _torch()
    g, o = _pair(P, K, 0.05, 0.9, dims, B, False, 95)
    assert g.one_launch == 1
    _run_and_compare(g, o, dims, 2, TOL_FP32, "by inputs %s" % (dims,))
    g, o = _pair(P, K, 0.05, 0.9, dims, B, False, 95)
    idx = np.random.default_rng(6).integers(0, 600, size=(P, K, B)).astype(np.int32)
    g.set_indices(torch.from_numpy(idx).cuda())
    o.set_indices(idx)
    _run_and_compare(g, o, dims, 2, TOL_FP32, "by inputs %s, caller's indices" % (dims,))


# four workgroups of 16 units to a chunk of up to 384 columns, where its chunks, rows and units end
QUARTERS = [
    (4, 3, 32, (3072, 64, 10)),        # eight chunks of 384 columns
    (3, 3, 31, (3076, 33, 16)),        # nine chunks, the last one 4 columns wide; 33 units; odd batch
    (2, 4, 1, (580, 64, 2)),           # one row; ten chunks of 64 columns become five of 128, the last one 68 wide
    (5, 2, 17, (1028, 49, 9)),         # one row in the second block of rows; chunks of 256
    (1, 2, 16, (4092, 64, 10)),        # one block of rows
]


@pytest.mark.parametrize("P,K,B,dims", QUARTERS, ids=["B%d-%s" % (c[2], c[3]) for c in QUARTERS])
def test_quarters_of_the_units(P, K, B, dims):
    g, o = _pair(P, K, 0.05, 0.9, dims, B, False, 97)
    assert g.one_launch == 1
    _run_and_compare(g, o, dims, 3, TOL_FP32, "quarters %s" % (dims,))


LINES = [
    # P, B, dims, kernel: on either side of the lines of the rule where both kernels cover a shape
    (48, 16, (256, 64, 10), 2), (49, 16, (256, 64, 10), 1), (200, 9, (64, 64, 10), 2), (128, 9, (64, 64, 10), 1),
    (24, 16, (512, 64, 10), 2), (20, 17, (512, 64, 10), 1),
    (16, 17, (128, 64, 10), 2), (17, 17, (128, 64, 10), 1),
    (2, 32, (384, 64, 10), 2), (2, 32, (388, 64, 10), 1),
    (2, 64, (192, 20, 10), 2), (2, 64, (196, 20, 10), 1),
]


@pytest.mark.parametrize("P,B,dims,kernel", LINES, ids=["P%d-B%d-%d" % (c[0], c[1], c[2][0]) for c in LINES])
def test_where_both_splits_cover_a_shape(P, B, dims, kernel):
    g, o = _pair(P, 2, 0.05, 0.9, dims, B, False, 96)
    assert g.one_launch == kernel
    _run_and_compare(g, o, dims, 2, TOL_FP32, "kernel %d %s" % (kernel, dims))


@pytest.mark.parametrize("P,K,B,dims", CASES, ids=[str(c[3]) for c in CASES])
def test_fused_steps_match_the_oracle(P, K, B, dims):
    g, o = _pair(P, K, 0.05, 0.9, dims, B, False, 91)
    assert g.fused
    _run_and_compare(g, o, dims, 4, TOL_FP32, "fused %s" % (dims,))


@pytest.mark.parametrize("P,K,B,dims", CASES[:3], ids=[str(c[3]) for c in CASES[:3]])
def test_fused_steps_match_the_launch_per_layer_path(P, K, B, dims):
    g, _ = _pair(P, K, 0.05, 0.9, dims, B, False, 92)
    h, _ = _pair(P, K, 0.05, 0.9, dims, B, False, 92)
    h.set_fused(False)
    assert g.fused and not h.fused
    for r in range(3):
        g.local_steps()
        h.local_steps()
        for j in range(P):
            assert flat_error(g.replica(j), h.replica(j)) < 2e-6, (r, j)
        assert np.max(np.abs(g.losses() - h.losses())) < 1e-5
        g.meta_update()
        h.meta_update()
    assert flat_error(g.params(), h.params()) < 2e-6


def test_fused_steps_with_caller_indices():
    torch = _torch()
    P, K, B, dims = 3, 3, 20, (264, 48, 10)
    g, o = _pair(P, K, 0.05, 0.9, dims, B, False, 93)
    assert g.fused
    rng = np.random.default_rng(5)
    for r in range(3):
        idx = rng.integers(0, 600, size=(P, K, B)).astype(np.int32)
        g.set_indices(torch.from_numpy(idx).cuda())
        o.set_indices(idx)
        g.local_steps()
        o.local_steps()
        assert np.array_equal(g.indices(), idx)
        for j in range(P):
            assert flat_error(g.replica(j), o.replica(j)) < TOL_FP32
        g.meta_update()
        o.meta_update()
    assert flat_error(g.params(), o.params()) < TOL_FP32


def test_a_wait_that_gives_up_ends_the_launch_and_is_reported():
    """With a limit of one poll a workgroup does not wait for the others: the launch still runs to its end
    (nothing hangs), a wait that found its data missing is reported once as KAVG_EDEVICE, and the context
    works again after the parameters have been installed anew."""
    P, K, B, dims = 4, 4, 32, (3072, 64, 10)
    g, o = _pair(P, K, 0.05, 0.9, dims, B, False, 94)
    w0 = g.params().copy()
    g.set_wait_limit(1)
    reported = 0
    for _ in range(3):
        g.local_steps()
        try:
            g.losses()
        except kavg.KavgError as e:
            assert e.code == kavg.KAVG_EDEVICE
            reported += 1
    print("launches with a wait that gave up: %d of 3" % reported)
    g.set_wait_limit(1 << 20)
    g.set_state(w0, np.zeros_like(w0), 0)                     # parameters, momentum and the index stream as at the start
    _run_and_compare(g, o, dims, 2, TOL_FP32, "after a wait limit of one poll")


def test_fused_path_is_taken_only_where_it_fits():
    _torch()
    assert kavg.MAvg(2, 2, 0.1, 0.5, (64, 65, 10), 8, kavg.KAVG_FP32).one_launch == 2    # hidden layer too wide for the split by inputs
    assert not kavg.MAvg(2, 2, 0.1, 0.5, (516, 65, 10), 8, kavg.KAVG_FP32).fused         # ... and inputs too long for the split by units
    assert not kavg.MAvg(2, 2, 0.1, 0.5, (64, 1025, 10), 8, kavg.KAVG_FP32).fused        # more than 16 groups of 64 units
    assert not kavg.MAvg(2, 2, 0.1, 0.5, (64, 32, 17), 8, kavg.KAVG_FP32).fused          # too many classes
    assert not kavg.MAvg(2, 2, 0.1, 0.5, (64, 32, 10), 65, kavg.KAVG_FP32).fused         # batch too large
    assert kavg.MAvg(2, 2, 0.1, 0.5, (66, 32, 10), 8, kavg.KAVG_FP32).one_launch == 2    # d_0 not a multiple of 4: split by units only
    assert not kavg.MAvg(2, 2, 0.1, 0.5, (602, 32, 10), 8, kavg.KAVG_FP32).fused         # ... and too long for it
    assert not kavg.MAvg(17, 2, 0.1, 0.5, (3072, 32, 10), 8, kavg.KAVG_FP32).fused       # 17 x 16 workgroups: more than compute units
    assert not kavg.MAvg(2, 2, 0.1, 0.5, (64, 32, 32, 10), 8, kavg.KAVG_FP32).fused      # two hidden layers
    assert not kavg.MAvg(2, 33, 0.1, 0.5, (64, 32, 10), 32, kavg.KAVG_FP32).fused        # K*B beyond the index table
    assert not kavg.MAvg(2, 2, 0.1, 0.5, (64, 32, 10), 8, kavg.KAVG_BF16).fused          # mixed precision
    assert kavg.MAvg(2, 2, 0.1, 0.5, (600, 32, 10), 8, kavg.KAVG_FP32).one_launch == 1
    g = kavg.MAvg(2, 2, 0.1, 0.5, (64, 32, 10), 8, kavg.KAVG_FP32)
    assert g.fused
    g.set_fused(False)
    assert g.one_launch == 0
    g.set_fused(True)
    assert g.fused
    g.set_learner_momentum(0.9)
    assert not g.fused
    g.set_learner_momentum(0.0)
    assert g.fused


def _constant(file, name):
    """A size that the library's sources state, `name = <product>;`."""
    text = open(os.path.join(os.path.dirname(kavg.__file__), "csrc", file)).read()
    return int(np.prod([int(f) for f in re.search(r"\b%s = ([0-9 *]+);" % name, text).group(1).split("*")]))


def test_losses_that_fit_the_pinned_buffer_and_more():
    """As many learners as leave three steps of losses, and the flags in front of them, room in the buffer, and one more: those are read
    the other way.  A learner's losses do not depend on how many others there are."""
    dims, K, B = (8, 4, 2), 3, 2
    P = (_constant("kavg_internal.h", "REPORT_BYTES") - _constant("kavg_api.hip", "ALIGN")) // (4 * K)
    g = [_pair(p, K, 0.05, 0.9, dims, B, False, 98)[0] for p in (P, P + 1, 5)]
    for _ in range(2):
        for c in g:
            c.local_steps()
        fit, more, few = (c.losses() for c in g)
        for got, want in ((fit, more[:, :P]), (fit[:, :5], few)):
            assert np.all(np.isfinite(got)) and np.all(got > 0)
            assert np.max(np.abs(got - want)) < 1e-5             # (fp32, sums of eight terms in another order)
        assert np.isfinite(more[-1, P]) and more[-1, P] > 0
