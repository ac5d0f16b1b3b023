"""A plan reports the sweep schedules it runs and accepts them back.

Installing what vmg_plan_schedule reports changes neither the reports nor the
launches nor a bit of the iterate, on plans whose finest level runs bricks (at
most 2^18 cells) and on larger ones; a schedule installed on the finest level
leaves the coarser ones alone; a tuned plan runs the finest schedule its tuner
chose.  What a finest level runs shows in the launches of its timed sweeps: two
sweeps each on bricks, one on a march."""
import numpy as np
import pytest
from test_gpu_sweep_timing import expected_launches

from paper_1303_0008_amd import inputs as I

pytestmark = pytest.mark.gpu
NU = (3, 4)    # launches differ between one and two sweeps a launch, before and after the coarse cycle


@pytest.fixture(scope="module")
def V():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1303_0008_amd import vmg
    vmg.load()
    return vmg


def timed_solve(V, plan, n):
    """Iterate after a few cycles, cycles, counted launches of finest sweeps."""
    import torch
    delta = torch.from_numpy(I.lognormal(n, 63, sigma=1.0)).to("cuda")
    phi = torch.zeros_like(delta)
    plan.time_sweeps(True)
    r = plan.solve(delta, phi, allow_noconv=True)[0]
    _, launches = plan.sweep_time()
    plan.time_sweeps(False)
    return phi.cpu().numpy(), r["cycles"], launches


def reports(plan):
    return [plan.schedule(l) for l in range(plan.level_count())]


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n", [(8, 8, 8), (32, 32, 32), (64, 40, 56), (64, 64, 64), (80, 64, 64), (128, 96, 64)])
def test_installing_the_reported_schedules_changes_nothing(V, prec, n):
    mixed = prec == "mixed"
    p = V.make_params(0.1, 1.5, 1e-30, 2, V.MIXED if mixed else V.FP64, *NU)
    with V.Plan([V.make_grid(n)], p) as plan:
        before = reports(plan)
        assert before[0][2] == (2 if n[0] * n[1] * n[2] <= 1 << 18 else 1)
        phi, cycles, launches = timed_solve(V, plan, n)
        if before[0][2] == 2:
            assert launches == expected_launches(mixed, 2, NU, cycles)
        for l, s in enumerate(before):
            plan.set_schedule(l, *s)
            assert reports(plan) == before
        again, _, launches2 = timed_solve(V, plan, n)
    assert np.array_equal(phi, again) and launches == launches2


@pytest.mark.parametrize("n", [(48, 48, 48), (128, 96, 64)])
def test_a_finest_schedule_leaves_the_coarser_levels(V, n):
    with V.Plan([V.make_grid(n)], V.make_params(0.1, 1.5, 1e-8)) as plan:
        before = reports(plan)
        plan.set_schedule(0, 4, 8, 0)
        assert reports(plan) == [(4, 8, 0)] + before[1:]


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n", [(40, 32, 48), (64, 64, 64)])
def test_a_tuned_plan_runs_its_schedule(V, prec, n):
    mixed = prec == "mixed"
    p = V.make_params(0.1, 1.5, 1e-30, 2, V.MIXED if mixed else V.FP64, *NU, V.AUTOTUNE)
    with V.Plan([V.make_grid(n)], p) as plan:
        s = plan.schedule(0)
        c = plan.cycle()
        _, cycles, launches = timed_solve(V, plan, n)
    assert (c["nu1"], c["nu2"]) == NU
    inner = c["inner_cycles"] if mixed else 2
    assert launches == expected_launches(mixed, 2 if s[2] == 2 else 1, NU, cycles, inner), s


def test_refused_finest_bricks(V):
    for n, s in (((32, 32, 32), (8, 16, 2)), ((32, 32, 32), (16, 8, 2)), ((80, 64, 64), (8, 8, 2)),
                 ((6, 6, 6), (8, 8, 2))):
        with V.Plan([V.make_grid(n)], V.make_params(0.1, 1.5, 1e-8)) as plan:
            with pytest.raises(V.VmgError) as ei:
                plan.set_schedule(0, *s)
            assert ei.value.status == V.VMG_EINVAL
