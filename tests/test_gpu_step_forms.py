"""The two register forms of the solver's step: which one a batch runs follows from how many of
its blocks the chip holds at once, a volume's own solve of few blocks runs the first.  Batches on
either side of that, by blocks of 512 and 128 threads, equal the volumes' own solves bitwise."""
import numpy as np
import pytest

from paper_2503_13802_amd import inputs
from gpu_util import announce, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,count", [((64, 64, 64), 4), ((64, 64, 64), 5),      # 512 blocks, 640: a second round
                                         ((32, 32, 32), 40), ((32, 32, 32), 41)])   # 2560 blocks, 2624
def test_batch_equals_own_solves(shape, count):
    torch = torch_cuda()
    from paper_2503_13802_amd import mh3d
    announce("step forms: %d of %s" % (count, shape))
    plans = [mh3d.Plan(shape, (2, 3), 1.0, (2, 2, 2), 20.0, 1e-3) for _ in range(count)]
    x = torch.tensor(np.abs(inputs.random_field(shape, 81)), dtype=torch.float32, device="cuda")
    data = [p.forward(x * (1.0 + 0.1 * i)) for i, p in enumerate(plans)]
    rhos, _ = mh3d.Batch(plans).solve(data, max_iter=6, tol=0.0, tau=0.05)
    for i in sorted({0, 1, count // 2, count - 1}):
        own, _ = plans[i].solve(data[i], max_iter=6, tol=0.0, tau=0.05)
        assert torch.equal(own, rhos[i]), i
