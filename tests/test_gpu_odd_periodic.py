"""Periodic levels whose x rows hold an odd number of cells.

A level that coarsens has an even n0, but the coarsest one may have 5 or 7 cells
along x: a grid of one level (residual and norm passes, the mixed path's outer
pass), or level 1 of a grid with n0 = 10 or 14 (the truncation-error estimate).
The passes move x pairs; the cell past such a row is the next row's first, or
past the array, and must neither enter a sum nor be written.  Bounds: the residual
field 1e-12 of its largest value (same operations, same precision), tau's RMS
1e-9 (two formulas of values of size |L phi|), solutions 1e-10 (FP64) and 1e-8
(mixed) of the largest value against the oracle solved to its rounding floor, as
elsewhere in this suite.
"""
import numpy as np
import pytest

from paper_1303_0008_amd import inputs as I

pytestmark = pytest.mark.gpu
PAD = 64
ONE_LEVEL = [(5, 5, 5), (5, 8, 8), (7, 5, 6), (7, 6, 4)]


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


def guarded(a):
    """A device copy of `a` between guard elements: the buffer and the view."""
    import torch
    buf = torch.full((a.size + 2 * PAD,), 7.0, dtype=torch.float64, device="cuda")
    view = buf[PAD:PAD + a.size].view(a.shape)
    view.copy_(dev(a))
    return buf, view


def guards_intact(buf):
    b = buf.cpu().numpy()
    return bool((b[:PAD] == 7.0).all() and (b[-PAD:] == 7.0).all())


@pytest.mark.parametrize("source", [False, True])
@pytest.mark.parametrize("n", ONE_LEVEL)
def test_residual(V, oracle_mod, n, source):
    rng = np.random.Generator(np.random.PCG64(181))
    shape, h = n[::-1], 1.0 / 64
    delta, phi = rng.standard_normal(shape), 1e-3 * rng.standard_normal(shape)
    src = rng.standard_normal(shape) if source else None
    d_ref, info = oracle_mod.residual(delta, phi, 0.1, 1.5, h=h, source=src)
    buf, d = guarded(np.zeros(shape))
    with V.Plan([V.make_grid(n, h=h)], V.make_params(0.1, 1.5, 1e-8)) as p:
        r = p.residual(0, dev(delta), dev(phi), d=d, source=None if src is None else dev(src))
    assert guards_intact(buf)
    assert np.abs(d.cpu().numpy() - d_ref).max() <= 1e-12 * np.abs(d_ref).max()
    assert abs(r["rms"] - info["rms"]) <= 1e-12 * info["rms"]


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n", ONE_LEVEL)
def test_solve_of_one_level(V, oracle_mod, n, prec):
    delta, h = I.lognormal(n, 41, sigma=1.0), 1.0 / 8
    src = 0.1 * np.random.Generator(np.random.PCG64(182)).standard_normal(delta.shape)
    for source in (None, src):
        ref, _ = oracle_mod.solve(delta, 0.1, 1.5, h=h, source=source)
        buf, phi = guarded(np.zeros_like(delta))
        with V.Plan([V.make_grid(n, h=h)], V.make_params(0.1, 1.5, 1e-12 if prec == "fp64" else 1e-11, 60,
                                                         {"fp64": V.FP64, "mixed": V.MIXED}[prec])) as p:
            r = p.solve(dev(delta), phi, source=None if source is None else dev(source))[0]
        assert r["status"] == V.VMG_OK and guards_intact(buf)
        err = np.abs(phi.cpu().numpy() - ref).max() / np.abs(ref).max()
        print(n, prec, source is not None, r["cycles"], f"{err:.1e}", flush=True)
        assert err <= (1e-10 if prec == "fp64" else 1e-8)


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n", [(10, 10, 10), (14, 12, 16), (10, 16, 16)])
def test_tau_rms(V, oracle_mod, n, prec):
    import torch
    delta = I.lognormal(n, 43, sigma=1.0)
    phi = torch.zeros(delta.shape, dtype=torch.float64, device="cuda")
    factor = 1.0 / 3.0
    with V.Plan([V.make_grid(n)], V.make_params(0.1, 1.5, 1e-12, 80, {"fp64": V.FP64, "mixed": V.MIXED}[prec],
                                                tau_factor=factor)) as p:
        r = p.solve(dev(delta), phi)[0]
    _, tau = oracle_mod.truncation_error(delta, phi.cpu().numpy(), 0.1, 1.5)
    print(n, prec, r["rms"], r["tau_rms"], tau, flush=True)
    assert r["status"] == V.VMG_OK and r["rms"] <= factor * r["tau_rms"]
    assert abs(r["tau_rms"] - tau) <= 1e-9 * tau
