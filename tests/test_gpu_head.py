"""The one-launch head of a small periodic level (residual, averages, coarse
right-hand side) and cbar left in its block sums: solves on grids with partial
bricks and uneven levels reach the oracle's answer, for every taker of the sums
(bricks with and without the folded prolongation, marches, the tail, levels
without pre- or post-sweeps)."""
import numpy as np
import pytest

from paper_1303_0008_amd import inputs as I

pytestmark = pytest.mark.gpu

SHAPES = [(8, 8, 8), (10, 12, 14), (16, 16, 16), (20, 24, 28), (28, 16, 20), (64, 48, 56)]


@pytest.fixture(scope="module")
def refs():
    return {}


@pytest.mark.parametrize("n", SHAPES)
@pytest.mark.parametrize("prec,tol,bound", [("fp64", 1e-11, 1e-10), ("mixed", 1e-10, 1e-8)])
@pytest.mark.parametrize("how", ["default", "no_tail", "no_pre", "no_post", "march", "source"])
def test_head_solves(oracle_mod, refs, n, prec, tol, bound, how):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1303_0008_amd import vmg as V
    key = (n, how == "source")
    if key not in refs:
        delta = I.lognormal(n, 31, sigma=0.8)
        src = 0.2 * I.gaussian_field(n, -2.0, 32) if how == "source" else None
        refs[key] = (delta, src, oracle_mod.solve(delta, 0.1, 1.5, source=src)[0])
    delta, src, ref = refs[key]
    d = torch.from_numpy(delta).to("cuda")
    s = None if src is None else torch.from_numpy(np.ascontiguousarray(src)).to("cuda")
    p = {"fp64": V.FP64, "mixed": V.MIXED}[prec]
    with V.Plan([V.make_grid(n)], V.make_params(0.1, 1.5, tol, 80, p, flags=V.GRAPH)) as plan:
        if how == "no_tail":
            plan.set_cycle(coarse_tail=0)
        elif how == "no_pre":
            plan.set_cycle(nu1=0, nu2=3)
        elif how == "no_post":
            plan.set_cycle(nu1=3, nu2=0)
        elif how == "march":
            for l in range(plan.level_count()):
                plan.set_schedule(l, 4, 4, l & 1)
        for _ in range(2):                     # both ping-pong parities of the recorded graphs
            phi = torch.zeros_like(d)
            plan.solve(d, phi, source=s)
            err = np.abs(phi.cpu().numpy() - ref).max() / np.abs(ref).max()
            assert err <= bound, err
