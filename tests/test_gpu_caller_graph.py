"""kavg_local_steps recorded by the caller into a graph of their own (torch.cuda.graph on the context's stream): every
replay has to be a meta round on the indices that lie in the caller's array at that moment."""
import numpy as np
import pytest

from tests.test_gpu_small import TOL_BF16, TOL_FP32, _pair, _torch
from tests.util import replica_error

pytestmark = pytest.mark.gpu

CASES = [
    # P, K, B, dims, bf16
    (6, 4, 32, (256, 256, 10), False),       # eagerly one launch, hidden units split over workgroups
    (3, 3, 20, (600, 64, 10), False),        # eagerly one launch, inputs split over workgroups
    (3, 2, 20, (96, 72, 40, 10), False),     # launches per layer
    (4, 2, 24, (264, 200, 136, 10), True),
]


@pytest.mark.parametrize("P,K,B,dims,bf16", CASES, ids=[str(c[3]) for c in CASES])
def test_replays_follow_the_callers_indices(P, K, B, dims, bf16):
    torch = _torch()
    side = torch.cuda.Stream()
    rng = np.random.default_rng(7)
    draw = lambda: rng.integers(0, 600, size=(P, K, B)).astype(np.int32)
    tol = TOL_BF16 if bf16 else TOL_FP32
    with torch.cuda.stream(side):
        g, o = _pair(P, K, 0.05, 0.9, dims, B, bf16, 241)
        idx = torch.zeros(P, K, B, dtype=torch.int32, device="cuda")
        g.set_indices(idx)

        def round_against_the_oracle(tag, go):
            new = draw()
            idx.copy_(torch.from_numpy(new))
            o.set_indices(new)
            go()
            o.local_steps()
            o.meta_update()
            assert np.array_equal(g.indices(), new)
            assert np.max(np.abs(g.losses() - o.losses())) < 1e-2, tag
            e = replica_error(g.params(), o.params(), dims)
            assert e < tol, "%s: %.3g" % (tag, e)

        def eager():
            g.local_steps()
            g.meta_update()

        round_against_the_oracle("eager", eager)
        graph = torch.cuda.CUDAGraph()
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            eager()
        for r in range(3):
            round_against_the_oracle("replay %d" % r, graph.replay)
        round_against_the_oracle("eager after the replays", eager)
        g.close()
