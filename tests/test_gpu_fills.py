"""Refinement fills of many grids in one call on the GPU against the oracle: more
fills than one launch's argument table holds, block edges (fills of exactly one
block's values, one more, one less, a single cell), ragged and wrapping places."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# 16 x 16 x 4 = 1024 values = one block of the fill kernel
SHAPES = [(16, 16, 4), (16, 16, 16), (1, 1, 1), (41, 25, 1), (31, 33, 1), (5, 3, 7), (1, 9, 2), (24, 24, 24), (2, 1, 30)]


@pytest.mark.parametrize("count", [1, 40, 41, 85])
@pytest.mark.parametrize("parent_shape,ratio", [((12, 10, 14), 2), ((1, 8, 5), 1), ((16, 16, 16), 4)])
def test_fills_of_many_grids(oracle_mod, count, parent_shape, ratio):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1303_0008_amd import vmg as V
    rng = np.random.Generator(np.random.PCG64(100 * count + ratio))
    parent = rng.standard_normal(parent_shape[::-1])
    H = 1.0 / 16
    h = H / ratio
    grids, origins, off, goff = [], [], 0, 0
    for i in range(count):
        n = SHAPES[i % len(SHAPES)]
        grids.append(V.make_grid(n, h, V.DIRICHLET, off, goff))
        origins.append(tuple(int(v) for v in rng.integers(-40, 60, size=3)))
        off += int(np.prod(n))
        goff += V.ghost_count(n)
    dev = dict(dtype=torch.float64, device="cuda")
    p_t = torch.from_numpy(parent).to("cuda")
    ghost, phi = torch.full((goff,), float("nan"), **dev), torch.full((off,), float("nan"), **dev)
    V.fill_ghosts(p_t, H, grids, origins, ghost)
    V.fill_interior(p_t, H, grids, origins, phi)
    ghost, phi = ghost.cpu().numpy(), phi.cpu().numpy()
    # a place is rounded by a few eps of its index (|u| < 128 parent cells), which
    # moves a value by that times the slope along three axes (2 max|parent| each)
    bound = 3 * 2 * np.abs(parent).max() * 8 * 128 * np.finfo(np.float64).eps
    for g, o in zip(grids, origins):
        n = tuple(g.n)
        ref = oracle_mod.fill_ghosts(parent, n, h, o, H=H)
        assert np.abs(ghost[g.ghost_offset:g.ghost_offset + ref.size] - ref).max() <= bound, (n, o)
        ref = oracle_mod.fill_interior(parent, n, h, o, H=H).ravel()
        assert np.abs(phi[g.offset:g.offset + ref.size] - ref).max() <= bound, (n, o)
