"""The end of an update (its FP64 sums, r_k, the stop, the iteration count) runs with the next
update's column or class pass, or as a launch of its own before the host reads the state
(every check_every updates).  Both sum in the same order, so a solve does not depend on
check_every: volume, history and count are bitwise equal, at the cap and when the tolerance
stops it in the middle of a run of updates."""
import numpy as np
import pytest

from paper_2503_13802_amd import inputs
from gpu_util import announce, torch_cuda

pytestmark = pytest.mark.gpu

PLANS = {
    # compile-time passes, separable passes (few and many blocks), padding; user PSFs: one and
    # two workgroups per plane, components, 2D, padding
    "fast": lambda m, t: m.Plan((32, 32, 32), range(2, 6), 1.0, (2, 4, 4), 8.0, 1e-3),
    "sep": lambda m, t: m.Plan((48, 64, 36), (2, 3, 4), 1.0, (2, 2, 3), 8.0, 1e-3),
    "sep many": lambda m, t: m.Plan((128, 16, 8), (2, 3), 1.0, (2, 4, 2), 8.0, 1e-3),
    "padded": lambda m, t: m.Plan((24, 16, 12), (2, 3, 4), 1.0, (2, 2, 2), 6.0, 1e-3, pad=(4, 2, 2)),
    "user": lambda m, t: _user(m, t, (16, 12, 8), (2, 2, 2), 3, 1),
    "vector": lambda m, t: _user(m, t, (16, 12, 8), (2, 2, 2), 3, 3),
    "image": lambda m, t: _user(m, t, (32, 1, 48), (2, 1, 4), 4, 2),
    "user padded": lambda m, t: _user(m, t, (16, 12, 8), (2, 2, 2), 3, 2, pad=(4, 2, 2)),
}


def _user(m, torch, shape, ds, K, C, **kw):
    h, b = inputs.vector_psfs(C, K, shape, 61), inputs.vector_sensitivity(C, shape, 62)
    f32 = lambda v: torch.tensor(np.ascontiguousarray(v), dtype=torch.float32)
    return m.Plan(shape, range(2, K + 2), 1.0, ds, 1.0, 1e-2, psf=f32(h if C > 1 else h[0]), sens=f32(b if C > 1 else b[0]), **kw)


def _same(torch, a, b):
    assert a[1]["iters"] == b[1]["iters"]
    assert list(a[1]["history"]) == list(b[1]["history"])
    assert torch.equal(a[0], b[0])


@pytest.mark.parametrize("kind", sorted(PLANS))
def test_solve_does_not_depend_on_where_updates_finish(kind):
    torch = torch_cuda()
    from paper_2503_13802_amd import mh3d
    announce("finish of updates: %s" % kind)
    p = PLANS[kind](mh3d, torch)
    d = p.forward(torch.tensor(np.abs(inputs.random_field(p.shape, 63)), dtype=torch.float32))
    own = p.solve(d, max_iter=23, tol=0.0, check_every=1)      # a finish of its own after each
    assert own[1]["iters"] == 23
    for every in (2, 7, 25):
        _same(torch, own, p.solve(d, max_iter=23, tol=0.0, check_every=every))
    # r_k falls: stop at its value after 10 updates, inside a run of 25
    tol = float(own[1]["history"][9])
    first = int(np.argmax(np.asarray(own[1]["history"]) <= tol)) + 1
    got = p.solve(d, max_iter=23, tol=tol, check_every=25)
    assert got[1]["iters"] == first
    _same(torch, p.solve(d, max_iter=23, tol=tol, check_every=1), got)


def test_batch_does_not_depend_on_where_updates_finish():
    torch = torch_cuda()
    from paper_2503_13802_amd import mh3d
    announce("finish of updates: batch")
    plans = [PLANS[k](mh3d, torch) for k in ("sep", "padded", "sep many")]
    ds = [p.forward(torch.tensor(np.abs(inputs.random_field(p.shape, 64 + i)), dtype=torch.float32)) for i, p in enumerate(plans)]
    r1, i1 = mh3d.Batch(plans).solve(ds, max_iter=60, tol=2e-2, check_every=1)
    r2, i2 = mh3d.Batch(plans).solve(ds, max_iter=60, tol=2e-2, check_every=20)
    assert [i["iters"] for i in i1] == [i["iters"] for i in i2]
    assert all(torch.equal(a, b) for a, b in zip(r1, r2))
