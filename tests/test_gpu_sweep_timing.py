"""Timing of the finest sweeps (vmg_plan_time_sweeps) counts launches and changes
nothing: a launch of bricks holds up to two sweeps, a march one, and a timed
solve issues the launches of an untimed one, so its iterate is the same, bit for
bit.  The launch that prolongs the coarse correction and the mixed path's launch
from a zero correction are not counted, with whatever sweeps they hold."""
import numpy as np
import pytest

from paper_1303_0008_amd import inputs as I

pytestmark = pytest.mark.gpu


def expected_launches(mixed, per, nu, cycles, inner=2):
    """Counted launches of a solve on a periodic grid of at most 2^18 cells, whose
    finest schedule holds `per` sweeps in a launch and folds the prolongation."""
    n = lambda k: (k + per - 1) // per   # noqa: E731
    post = n(nu[1] - min(nu[1], per))
    if not mixed:        # shifted cycles: one more head than tails
        return (cycles + 1) * n(nu[0]) + cycles * post
    first = n(nu[0] - min(nu[0], per))
    return cycles * (first + (inner - 1) * n(nu[0]) + inner * post)


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n", [(32, 32, 32), (20, 24, 28)])
@pytest.mark.parametrize("nu", [(2, 2), (3, 1), (1, 3), (0, 4)])
@pytest.mark.parametrize("march", [False, True])
def test_launches_of_timed_solves(prec, n, nu, march):
    import torch
    from paper_1303_0008_amd import vmg as V
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    delta = torch.from_numpy(I.lognormal(n, 61, sigma=1.0)).to("cuda")
    p = V.MIXED if prec == "mixed" else V.FP64
    with V.Plan([V.make_grid(n)], V.make_params(0.1, 1.5, 1e-30, 4, p, *nu)) as plan:
        if march:
            plan.set_schedule(0, 16, 8, 1)
        out = []
        for timed in (False, True):
            plan.time_sweeps(timed)
            phi = torch.zeros_like(delta)
            r = plan.solve(delta, phi, allow_noconv=True)[0]
            out.append(phi.cpu().numpy())
        us, launches = plan.sweep_time()
    assert np.array_equal(out[0], out[1]) and np.abs(out[0]).max() > 0
    assert launches == expected_launches(p == V.MIXED, 1 if march else 2, nu, r["cycles"])
    assert us > 0
