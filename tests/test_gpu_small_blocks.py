"""Small-grid blocks of many short lines: one to three decimated y samples against thousands of
half-spectrum columns in the block, where the division that deals the run-time transforms'
elements leaves the range of the plain multiply-high.  Every call against the FP64 oracle."""
import numpy as np
import pytest

from oracle import model as om
from oracle import solver as osv
from paper_2503_13802_amd import inputs
from gpu_util import announce, rel_l2, torch_cuda

pytestmark = pytest.mark.gpu
TOL = 1e-5   # FP32 applications, as for the other plans

CASES = [
    # shape, decimation, padding, x'-block
    ((32, 4, 192), (1, 2, 1), (0, 0, 0), 32),     # my = 2
    ((32, 6, 192), (1, 2, 1), (0, 0, 0), 32),     # my = 3
    ((48, 6, 128), (1, 2, 1), (0, 0, 0), 48),
    ((36, 6, 144), (1, 2, 1), (2, 0, 4), 36),     # the padded volumes' pass back into the spectra
    ((64, 1, 256), (1, 1, 1), (0, 0, 0), 64),     # an image (user PSFs): my = 1
]


@pytest.mark.parametrize("shape,ds,pad,xb", CASES)
def test_many_short_lines_in_a_block(shape, ds, pad, xb):
    torch = torch_cuda()
    from paper_2503_13802_amd import mh3d
    announce("small-grid block %s ds=%s pad=%s xb=%d" % (shape, ds, pad, xb))
    harm, a, sig, lam = (2, 3), 0.9, 6.0, 1e-2
    f32 = lambda v: torch.tensor(np.ascontiguousarray(v), dtype=torch.float32)
    if shape[1] == 1:
        h, b = inputs.vector_psfs(1, 2, shape, 71)[0], inputs.vector_sensitivity(1, shape, 72)[0]
        p = mh3d.Plan(shape, harm, a, ds, sig, lam, psf=f32(h), sens=f32(b))
    else:
        h, b = om.psf_bank(shape, list(harm), a), om.sensitivity(shape, sig)
        p = mh3d.Plan(shape, harm, a, ds, sig, lam, pad=pad)
    op = osv.Operator(h, b, ds, lam, pad=pad)
    x = inputs.random_field(shape, 73)
    d_ref = op.A(x)
    r = inputs.random_field(d_ref.shape, 74)

    p.set_tiles(0, 0, xb, 0)
    assert p.tiles()[2] == xb
    d, back = p.forward_adjoint(f32(x))
    assert rel_l2(d.cpu().numpy(), d_ref) <= TOL
    assert rel_l2(back.cpu().numpy(), op.AT(d_ref)) <= TOL
    assert torch.equal(p.forward(f32(x)), d)
    assert rel_l2(p.adjoint(f32(r)).cpu().numpy(), op.AT(r)) <= TOL
    assert rel_l2(p.normal(f32(x)).cpu().numpy(), op.normal(x)) <= TOL
    c = p.backproject(f32(r)).cpu().numpy()
    for k in range(len(harm)):
        only = np.zeros_like(r)
        only[k] = r[k]
        assert rel_l2(c[k], op.AT(only)) <= TOL, k
    tau = osv.step_size(osv.power_iteration(op, np.ones(shape), 20))
    want, _, _ = osv.fista(op, d_ref, tau, max_iter=5)
    got, info = p.solve(f32(d_ref), max_iter=5, tol=0.0, tau=tau)
    assert rel_l2(got.cpu().numpy(), want) <= 1e-4   # solver updates, as for the other plans
