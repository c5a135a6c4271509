"""The meta step where the parameters per lane change (1, 4 of a float replica; 2, 8 of one in planes), with ragged ends and
numbers of replicas around the sixteen (eight) whose loads go out together, against 64-bit arithmetic."""
import numpy as np
import pytest
import torch

from paper_2110_00625_amd import kavg
from tests.test_gpu_small import _pair

pytestmark = pytest.mark.gpu


def _expected(w, v, reps, mu):
    w, v, reps = (np.asarray(a, dtype=np.float64) for a in (w, v, reps))
    vn = mu * v + (reps.mean(axis=0) - w)
    return w + vn, vn


def _close(got, want, terms):
    """A sum of `terms` differences of the size of `want` in fp32, and two roundings."""
    bound = (terms + 3) * 2.0 ** -24 * max(float(np.max(np.abs(want))), 1e-30) * 4
    assert np.max(np.abs(np.asarray(got, dtype=np.float64) - want)) <= bound


@pytest.mark.parametrize("n", [1, 3, 255, 20001, 196607, 196610, 262143, 262145, 524287, 524290])
@pytest.mark.parametrize("P,shadow", [(1, False), (15, True), (17, False), (26, True), (33, True)])
def test_float_replicas(n, P, shadow):
    gen = torch.Generator(device="cuda").manual_seed(n + P)
    stride = (n + 63) // 64 * 64
    w = torch.randn(n, generator=gen, device="cuda") * 0.05
    v = torch.randn(n, generator=gen, device="cuda") * 1e-2
    reps = torch.zeros(P, stride, device="cuda")
    reps[:, :n] = w + torch.randn(P, n, generator=gen, device="cuda") * 1e-2
    sh = torch.zeros(P, stride, dtype=torch.bfloat16, device="cuda") if shadow else None
    wn, vn = _expected(w.cpu(), v.cpu(), reps[:, :n].cpu(), 0.9)
    kavg.kavg_meta_update_flat(w, v, reps, 0.9, shadow=sh)
    _close(v.cpu(), vn, P)
    _close(w.cpu(), wn, P)
    assert torch.equal(reps[:, :n], w.expand(P, n)) and not reps[:, n:].any()
    if shadow:
        bits = (w.view(torch.int32) + 0x8000) >> 16              # nearest, ties away from zero
        assert torch.equal(sh[:, :n].contiguous().view(torch.int16), bits.to(torch.int16).expand(P, n))


@pytest.mark.parametrize("P", [1, 7, 17])
@pytest.mark.parametrize("dims", [(8, 8, 3), (256, 1000, 8, 5), (512, 600, 8, 6), (512, 1016, 8, 6), (1024, 512, 7), (1024, 1016, 8, 9)], ids=lambda d: "-".join(map(str, d)))
def test_replicas_in_planes(P, dims):
    g, _ = _pair(P, 1, 0.05, 0.9, dims, 8, True, 31)
    for _ in range(2):
        g.local_steps()
        wn, vn = _expected(g.params(), g.momentum(), np.stack([g.replica(j) for j in range(P)]), 0.9)
        g.meta_update()
        _close(g.momentum(), vn, P)
        _close(g.params(), wn, P)
        for j in (0, P - 1):
            assert np.array_equal(g.replica(j), g.params())
    g.close()
