"""Passes of user-PSF plans where their shapes can go wrong: lengths without compiled stages,
odd rows, planes whose components do not fit a workgroup together (rounds of one), several
workgroups per plane with uneven shares, every number of spectrum elements per thread, harmonics
around the depth of the spectra's ring, zero component blocks, 2D grids of up to three
components.  A, A^T, A then A^T, the normal operator and solver updates against the oracle."""
import numpy as np
import pytest

from oracle import model as om
from oracle import solver as osv
from paper_2503_13802_amd import inputs
from gpu_util import announce, rel_l2, torch_cuda

pytestmark = pytest.mark.gpu
TOL = 1e-5   # FP32 applications, as for the other plans

CASES = [
    # shape, decimation, harmonics, components, tiles (E, cpw, xb, ps) or None
    ((4, 4, 4), (1, 1, 1), 1, 1, None),
    ((81, 6, 4), (3, 3, 1), 2, 2, None),             # nx = 81: the run-time engine
    ((6, 81, 54), (2, 3, 3), 3, 3, None),            # ny = 81 and odd rows
    ((8, 128, 64), (2, 4, 2), 2, 3, None),           # three components take rounds
    ((8, 128, 64), (2, 4, 2), 2, 2, (2, 1, 1, 4)),   # two fit; uneven quarters of the columns
    ((8, 18, 12), (2, 2, 2), 5, 3, (8, 1, 2, 2)),    # E = 8: class passes in rounds
    ((8, 18, 12), (2, 2, 2), 4, 2, (4, 1, 1, 1)),
    ((8, 18, 12), (2, 2, 2), 7, 2, (1, 9, 4, 2)),
    ((18, 12, 6), (3, 3, 1), 9, 2, (9, 2, 1, 2)),
    ((12, 6, 12), (2, 3, 2), 6, 3, (3, 1, 1, 3)),
    ((16, 1, 48), (2, 1, 4), 4, 3, None),            # 2D
    ((12, 1, 162), (3, 1, 3), 3, 2, None),           # 2D, nz = 162
]


@pytest.mark.parametrize("shape,ds,K,C,tiles", CASES)
def test_user_psf_passes_vs_oracle(shape, ds, K, C, tiles):
    torch = torch_cuda()
    from paper_2503_13802_amd import mh3d
    announce("user PSF %s ds=%s K=%d C=%d tiles=%s" % (shape, ds, K, C, tiles))
    h = inputs.vector_psfs(C, K, shape, 51)
    if C > 1 and K > 2:
        h[1, K - 1] = 0.0                             # a zero block: skipped
        h[0, 0] = 0.0
    b = inputs.vector_sensitivity(C, shape, 52)
    f32 = lambda v: torch.tensor(np.ascontiguousarray(v), dtype=torch.float32)
    p = mh3d.Plan(shape, range(2, K + 2), 1.0, ds, 1.0, 1e-2, psf=f32(h if C > 1 else h[0]), sens=f32(b if C > 1 else b[0]))
    if tiles:
        p.set_tiles(*tiles)
    fwd = lambda v: om.forward_vector(h, b, v, ds)
    adj = lambda v: om.adjoint_vector(h, b, v, ds)
    rho = inputs.random_field(shape, 53)
    d_ref = fwd(rho)
    r = inputs.random_field(d_ref.shape, 54)
    d = p.forward(f32(rho))
    assert rel_l2(d.cpu().numpy(), d_ref) <= TOL
    assert rel_l2(p.adjoint(f32(r)).cpu().numpy(), adj(r)) <= TOL
    d2, x2 = p.forward_adjoint(f32(rho))
    assert torch.equal(d2, d)
    assert rel_l2(x2.cpu().numpy(), adj(d_ref)) <= TOL
    normal = lambda v: adj(fwd(v)) + 1e-2 * om.reg_normal(v)
    assert rel_l2(p.normal(f32(rho)).cpu().numpy(), normal(rho)) <= TOL
    # three updates written out: y, gradient, projection
    lmax = p.power_iteration(30, 0)
    tau = 0.9 / lmax
    want = prev = np.zeros(shape)
    for k in range(1, 4):
        y = want + (k - 1.0) / (k + 2.0) * (want - prev)
        g = adj(fwd(y) - d_ref) + 1e-2 * om.reg_normal(y)
        prev, want = want, np.maximum(y - tau * g, 0.0)
    got, info = p.solve(f32(d_ref), max_iter=3, tol=0.0, tau=tau)
    assert info["iters"] == 3
    assert rel_l2(got.cpu().numpy(), want) <= 3 * TOL
