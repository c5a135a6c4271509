"""fp32 models with a wide hidden layer on short inputs: all K local steps in one launch, the workgroups of a learner
splitting its hidden units (fused_units.hip), against the oracle and against the launch-per-layer path."""
import numpy as np
import pytest

from paper_2110_00625_amd import kavg
from tests.test_gpu_small import TOL_FP32, _pair, _run_and_compare, _torch
from tests.util import flat_error

pytestmark = pytest.mark.gpu

CASES = [
    # P, K, B, dims
    (6, 4, 32, (256, 256, 10)),        # 16 groups of 16 units per learner
    (48, 3, 4, (256, 256, 10)),        # many learners: groups of 64 units, 4 rows of a 16-row block
    (3, 3, 19, (61, 927, 7)),          # inputs no multiple of 4 (word by word), 15 groups of 64, the last one 31 wide
    (2, 2, 64, (64, 200, 16)),         # full batch, every class, last group 8 units
    (5, 3, 7, (5, 70, 3)),             # a contraction shorter than one block
    (1, 5, 33, (500, 65, 2)),          # one unit in the last group, rows one over two blocks, two pieces per row and lane
    (3, 2, 16, (512, 40, 10)),         # the longest inputs
    (130, 2, 16, (20, 33, 10)),        # one workgroup per learner: nothing is exchanged
    (2, 3, 1, (4, 2, 1)),              # the smallest of everything
]
IDS = ["P%d-B%d-%s" % (c[0], c[2], c[3]) for c in CASES]


@pytest.mark.parametrize("P,K,B,dims", CASES, ids=IDS)
def test_steps_match_the_oracle(P, K, B, dims):
    g, o = _pair(P, K, 0.05, 0.9, dims, B, False, 191)
    assert g.one_launch == 2
    _run_and_compare(g, o, dims, 3, TOL_FP32, "units %s" % (dims,))


@pytest.mark.parametrize("P,K,B,dims", CASES, ids=IDS)
def test_steps_match_the_launch_per_layer_path(P, K, B, dims):
    """Same arithmetic, another order of the fp32 sums: a sum of n terms differs by a few times sqrt(n) 2^-24 of its
    largest term, here n <= 927 (about 2e-6); 1e-5 also covers three steps of it."""
    g, _ = _pair(P, K, 0.05, 0.9, dims, B, False, 192)
    h, _ = _pair(P, K, 0.05, 0.9, dims, B, False, 192)
    h.set_fused(False)
    for _ in range(2):
        g.local_steps()
        h.local_steps()
        for j in (0, P - 1):
            assert flat_error(g.replica(j), h.replica(j)) < 1e-5
        assert np.max(np.abs(g.losses() - h.losses())) < 1e-4
        g.meta_update()
        h.meta_update()
    assert flat_error(g.params(), h.params()) < 1e-5


def test_caller_indices():
    torch = _torch()
    P, K, B, dims = 3, 3, 20, (100, 150, 10)
    g, o = _pair(P, K, 0.05, 0.9, dims, B, False, 193)
    idx = np.random.default_rng(5).integers(0, 600, size=(P, K, B)).astype(np.int32)
    g.set_indices(torch.from_numpy(idx).cuda())
    o.set_indices(idx)
    g.local_steps()
    o.local_steps()
    assert np.array_equal(g.indices(), idx)
    for j in range(P):
        assert flat_error(g.replica(j), o.replica(j)) < TOL_FP32


def test_a_wait_that_gives_up_ends_the_launch_and_is_reported():
    P, K, B, dims = 6, 4, 32, (256, 256, 10)
    g, o = _pair(P, K, 0.05, 0.9, dims, B, False, 194)
    w0 = g.params().copy()
    g.set_wait_limit(1)
    for _ in range(3):
        g.local_steps()
        try:
            g.losses()
        except kavg.KavgError as e:
            assert e.code == kavg.KAVG_EDEVICE
    g.set_wait_limit(1 << 20)
    g.set_state(w0, np.zeros_like(w0), 0)
    _run_and_compare(g, o, dims, 2, TOL_FP32, "after a wait limit of one poll")


def test_the_librarys_own_block_takes_a_model_whose_scratch_does_not_fit():
    """400-256-10 with 63 learners: 32.2 MiB with the scratch of the one-launch path, 31.2 without.  A context in the 32 MiB
    block then runs one launch per layer, bit for bit what a caller workspace gives with that path chosen."""
    torch = _torch()
    P, K, B, dims = 63, 2, 16, (400, 256, 10)
    h, _ = _pair(P, K, 0.05, 0.9, dims, B, False, 194)
    h.set_fused(False)
    assert h.workspace.numel() > 32 << 20
    g = kavg.MAvg(P, K, 0.05, 0.9, dims, B, kavg.KAVG_FP32, index_seed=197, static_workspace=True)
    assert g.one_launch == 0
    rng = np.random.default_rng(6)
    X = torch.from_numpy(rng.standard_normal((600, 400), dtype=np.float32)).cuda()
    y = torch.from_numpy(rng.integers(0, 10, 600).astype(np.int32)).cuda()
    w0 = h.params()
    for c in (g, h):
        c.set_data(X, y)
        c.set_params(w0)
        c.local_steps()
    for j in (0, P - 1):
        assert np.array_equal(g.replica(j), h.replica(j))
    g.close()
