"""The general column pass (more than four x aliases, more than sixteen y residues): its aliases go through the registers in runs of
four, two and one, and the threads of a block share the products of a frequency where there are
more of them; the residues' shares are added eight at a time.  Every remainder, one to several threads per frequency with and without
idle ones, harmonics in one and several groups, with and without padding, against the FP64
oracle; volumes of such plans in one batch equal their own solves."""
import numpy as np
import pytest

from oracle import model as om
from oracle import solver as osv
from paper_2503_13802_amd import inputs
from gpu_util import announce, rel_l2, torch_cuda

pytestmark = pytest.mark.gpu
TOL = 1e-5   # FP32 applications, as for the other plans

CASES = [
    # grid, ds, harmonics, pad
    ((16, 4, 4), (8, 2, 2), (2,), (0, 0, 0)),                        # two samples along x
    ((12, 6, 4), (6, 2, 1), (2, 3, 4), (0, 0, 0)),                   # 4 + 2, idle threads
    ((36, 8, 8), (9, 2, 2), (2, 3), (0, 0, 0)),                      # 4 + 4 + 1
    ((216, 4, 8), (18, 1, 2), (2, 3, 5), (0, 0, 0)),                 # 16 + 2
    ((96, 8, 4), (12, 1, 1), tuple(range(2, 8)), (0, 0, 0)),
    ((256, 4, 4), (64, 1, 1), (2, 3, 4), (0, 0, 0)),                 # four samples, 64 aliases
    ((64, 8, 8), (16, 1, 1), tuple(range(2, 10)), (0, 0, 0)),        # several threads per frequency
    ((256, 4, 8), (8, 1, 1), tuple(range(2, 22)), (0, 0, 0)),        # 20 harmonics in two groups
    ((144, 8, 8), (9, 2, 2), (2, 3, 4), (18, 2, 2)),                 # padded: forward and adjoint alone
    ((72, 12, 8), (6, 3, 1), (2, 4), (6, 3, 1)),
    ((8, 72, 4), (2, 18, 1), (2, 3), (0, 0, 0)),                     # 18 residues: 4 + 8 + 6
    ((8, 128, 4), (2, 64, 1), (2, 3, 4), (0, 0, 0)),
    ((16, 96, 8), (8, 32, 2), (2, 3), (0, 0, 0)),                    # both
]


@pytest.mark.parametrize("shape,ds,harm,pad", CASES)
def test_operator_and_updates(shape, ds, harm, pad):
    torch = torch_cuda()
    from paper_2503_13802_amd import mh3d
    announce("x aliases %s ds=%s K=%d pad=%s" % (shape, ds, len(harm), pad))
    op = osv.Operator(om.psf_bank(shape, list(harm), 0.9), om.sensitivity(shape, 6.0), ds, 1e-2, pad=pad)
    p = mh3d.Plan(shape, harm, 0.9, ds, 6.0, 1e-2, pad=pad)
    f32 = lambda v: torch.tensor(v, dtype=torch.float32)
    x = inputs.random_field(shape, 91)
    d_ref = op.A(x)
    d, back = p.forward_adjoint(f32(x))
    assert rel_l2(d.cpu().numpy(), d_ref) <= TOL
    assert rel_l2(back.cpu().numpy(), op.AT(d_ref)) <= TOL
    assert torch.equal(p.forward(f32(x)), d)
    r = inputs.random_field(d_ref.shape, 92)
    assert rel_l2(p.adjoint(f32(r)).cpu().numpy(), op.AT(r)) <= TOL
    assert rel_l2(p.normal(f32(x)).cpu().numpy(), op.normal(x)) <= TOL
    tau = osv.step_size(osv.power_iteration(op, np.ones(shape), 20))
    want, _, _ = osv.fista(op, d_ref, tau, max_iter=8)
    got, info = p.solve(f32(d_ref), max_iter=8, tol=0.0, tau=tau)
    assert info["iters"] == 8
    assert rel_l2(got.cpu().numpy(), want) <= 1e-4


def test_batch_equals_own_solves():
    torch = torch_cuda()
    from paper_2503_13802_amd import mh3d
    announce("batch of %d volumes with many x aliases" % len(CASES))
    plans = [mh3d.Plan(s, h, 0.9, ds, 6.0, 1e-2, pad=pad) for s, ds, h, pad in CASES]
    data = [p.forward(torch.tensor(inputs.random_field(p.shape, 93 + i), dtype=torch.float32).abs()) for i, p in enumerate(plans)]
    own = [p.solve(d, max_iter=7, tol=0.0, tau=0.0)[0] for p, d in zip(plans, data)]
    rhos, _ = mh3d.Batch(plans).solve(data, max_iter=7, tol=0.0, tau=0.0)
    for v, (a, b) in enumerate(zip(own, rhos)):
        assert torch.equal(a, b), v
