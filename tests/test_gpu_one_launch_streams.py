"""Contexts whose local steps are one launch each (fused_small.hip, fused_units.hip), on streams and threads of their own:
together their workgroups would not find room on the chip, so their launches take turns, and every context has to end
with exactly what it computes alone."""
import threading

import numpy as np
import pytest

from tests.test_gpu_small import _pair, _torch

pytestmark = pytest.mark.gpu

SHAPES = [
    (16, 4, 32, (256, 256, 10)),        # 16 workgroups for each of 16 learners
    (16, 4, 32, (1024, 64, 10)),        # the same, inputs split
    (16, 4, 32, (256, 256, 10)),
]
ROUNDS = 60


def _rounds(g, n):
    for _ in range(n):
        g.local_steps()
        g.meta_update()


@pytest.mark.parametrize("threads", [False, True], ids=["one-thread", "threads"])
def test_contexts_on_streams_of_their_own(threads):
    torch = _torch()
    alone = []
    for i, shape in enumerate(SHAPES):
        P, K, B, dims = shape
        g, _ = _pair(P, K, 0.05, 0.9, dims, B, False, 251 + i)
        _rounds(g, ROUNDS)
        alone.append((g.params(), g.losses()))
        g.close()
    gs = []
    for i, (P, K, B, dims) in enumerate(SHAPES):
        with torch.cuda.stream(torch.cuda.Stream()):
            gs.append(_pair(P, K, 0.05, 0.9, dims, B, False, 251 + i)[0])
    if threads:
        errors = []

        def work(g):
            try:
                _rounds(g, ROUNDS)
            except Exception as e:
                errors.append(e)
        ts = [threading.Thread(target=work, args=(g,)) for g in gs]
        for t in ts:
            t.start()
        for t in ts:
            t.join()
        assert not errors, errors
    else:
        for _ in range(ROUNDS):
            for g in gs:
                _rounds(g, 1)
    for g, (w, losses) in zip(gs, alone):
        assert np.array_equal(g.losses(), losses)
        assert np.array_equal(g.params(), w)
    # the contexts that remain go on as contexts leave and join
    gs[1].close()
    for g in (gs[0], gs[2]):
        _rounds(g, 3)
    gs[0].close()
    _rounds(gs[2], 3)
    P, K, B, dims = SHAPES[0]
    with torch.cuda.stream(torch.cuda.Stream()):
        late, _ = _pair(P, K, 0.05, 0.9, dims, B, False, 251)
    for _ in range(ROUNDS):
        _rounds(gs[2], 1)
        _rounds(late, 1)
    assert np.array_equal(late.params(), alone[0][0])
    assert np.all(np.isfinite(gs[2].losses()))
    late.close()
    gs[2].close()


def test_small_launches_stay_side_by_side():
    """Launches that fit on the chip together (2 x 96 workgroups) do not wait for each other; results as alone."""
    torch = _torch()
    P, K, B, dims = 6, 4, 32, (256, 256, 10)
    alone, _ = _pair(P, K, 0.05, 0.9, dims, B, False, 271)
    _rounds(alone, 20)
    want = alone.params()
    alone.close()
    gs = []
    for _ in range(2):
        with torch.cuda.stream(torch.cuda.Stream()):
            gs.append(_pair(P, K, 0.05, 0.9, dims, B, False, 271)[0])
    for _ in range(20):
        for g in gs:
            _rounds(g, 1)
    for g in gs:
        assert np.array_equal(g.params(), want)
        g.close()


def test_a_launch_that_cannot_be_waited_for_gives_way():
    """The stream of the launch before is being recorded, so no event can be put behind it: the steps run as separate
    launches, with sums in another order."""
    torch = _torch()
    P, K, B, dims = SHAPES[0]
    a, _ = _pair(P, K, 0.05, 0.9, dims, B, False, 261)
    a.set_fused(False)
    _rounds(a, 1)
    want = a.params()
    a.close()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        first, _ = _pair(P, K, 0.05, 0.9, dims, B, False, 262)
        _rounds(first, 1)
    second, _ = _pair(P, K, 0.05, 0.9, dims, B, False, 261)
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    x = torch.zeros(64, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side, capture_error_mode="thread_local"):
        x.add_(1.0)
        _rounds(second, 1)
    graph.replay()
    assert np.array_equal(second.params(), want)
    assert np.all(np.isfinite(first.losses()))
    second.close()
    first.close()
