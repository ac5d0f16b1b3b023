"""The folded FP32 sweep with one and with two blocks per CU.

A 16-row schedule whose folded sweep has 512 or more blocks runs it on
three-plane rings whatever the schedule's pipe, below that the pipe decides.
The red-black order does not depend on the rings, so at one z chunk the iterate
of a mixed solve is the same, bit for bit, on both sides of that line (2-plane
chunks: 512 and 896 blocks, 4-plane ones: 256 and 448) and for every tile height;
the second shape ends in partial tiles along x.
"""
import numpy as np
import pytest

from paper_1303_0008_amd import inputs as I

pytestmark = pytest.mark.gpu



@pytest.mark.parametrize("zc", [2, 4])
@pytest.mark.parametrize("n", [(128, 128, 64), (96, 112, 128)])
def test_folded_sweep_rings_agree(n, zc):
    import torch
    from paper_1303_0008_amd import vmg as V
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    delta = torch.from_numpy(I.lognormal(n, 71, sigma=1.0)).to("cuda")
    outs = []
    for sched in ((16, zc, 1), (16, zc, 0), (8, zc, 1), (4, zc, 0)):
        with V.Plan([V.make_grid(n, h=1.0 / 128)], V.make_params(0.1, 1.5, 1e-30, 2, V.MIXED)) as plan:
            plan.set_schedule(0, *sched)
            assert plan.schedule(0) == sched
            phi = torch.zeros_like(delta)
            plan.solve(delta, phi, allow_noconv=True)
            outs.append(phi.cpu().numpy())
    assert np.isfinite(outs[0]).all() and np.abs(outs[0]).max() > 0
    for o in outs[1:]:
        assert np.array_equal(o, outs[0])
