"""Schedules a plan takes by default: the finest level of a small periodic grid runs
bricks and gives the march's iterate bit for bit (both precisions, with and
without a source, partial bricks, odd sweep counts), an installed schedule takes
their place, and batches on default schedules solve the oracle's equations."""
import numpy as np
import pytest

from paper_1303_0008_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def V():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1303_0008_amd import vmg
    vmg.load()
    return vmg


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).to("cuda")


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n", [(8, 8, 8), (16, 16, 16), (20, 24, 28), (32, 32, 32), (64, 40, 56), (64, 64, 64)])
@pytest.mark.parametrize("nu,flags,source", [((2, 2), 1, False), ((1, 3), 0, True), ((3, 1), 1, True)])
def test_finest_bricks_equal_march(V, prec, n, nu, flags, source):
    import torch
    delta = I.lognormal(n, 7, sigma=1.0)
    f = 0.1 * I.gaussian_field(n, -2.0, 8) if source else None
    p = {"fp64": V.FP64, "mixed": V.MIXED}[prec]
    out = []
    for march in (None, (16, 8, 1), (4, 2, 0)):
        with V.Plan([V.make_grid(n)], V.make_params(0.1, 1.5, 1e-30, 3, p, *nu, flags)) as plan:
            if march is not None:
                coarse = [plan.schedule(l) for l in range(1, plan.level_count())]
                plan.set_schedule(0, *march)
                assert plan.schedule(0) == march
                for l, c in enumerate(coarse):
                    plan.set_schedule(l + 1, *c)
            phi = torch.zeros(n[::-1], dtype=torch.float64, device="cuda")
            plan.solve(dev(delta), phi, source=None if f is None else dev(f), allow_noconv=True)
            out.append(phi.cpu().numpy())
    assert np.abs(out[0]).max() > 0
    for o in out[1:]:
        assert np.array_equal(out[0], o)


@pytest.mark.parametrize("sizes", [[(16, 16, 16)] * 3, [(24, 40, 32), (64, 64, 64), (64, 64, 64), (6, 6, 6)]])
def test_default_batch_parity(V, oracle_mod, sizes):
    """A batch below and one above the cell count at which the finest level marches."""
    import torch
    rng = np.random.Generator(np.random.PCG64(11))
    h, off, goff = 1.0 / 512, 0, 0
    grids, deltas, ghosts = [], [], []
    for i, n in enumerate(sizes):
        deltas.append(I.lognormal(n, 300 + i, sigma=1.5))
        ghosts.append(2e-5 * rng.standard_normal(oracle_mod.ghost_count(n)))
        grids.append(V.make_grid(n, h, V.DIRICHLET, off, goff))
        off += deltas[-1].size
        goff += ghosts[-1].size
    refs = [oracle_mod.solve(d, 0.1, 1.5, h=h, ghost=g)[0] for d, g in zip(deltas, ghosts)]
    for prec, bound in ((V.FP64, 1e-10), (V.MIXED, 1e-8)):
        phi = torch.zeros(off, dtype=torch.float64, device="cuda")
        with V.Plan(grids, V.make_params(0.1, 1.5, 1e-12, 100, prec, flags=V.GRAPH)) as plan:
            plan.solve(dev(np.concatenate([d.ravel() for d in deltas])), phi, ghost=dev(np.concatenate(ghosts)),
                       allow_noconv=True)
        phi_n = phi.cpu().numpy()
        for g, ref in zip(grids, refs):
            got = phi_n[g.offset:g.offset + ref.size].reshape(ref.shape)
            assert np.abs(got - ref).max() <= bound * np.abs(ref).max(), (prec, ref.shape)
