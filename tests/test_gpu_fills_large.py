"""More values to fill in one call than one launch has threads for: 38 refinements of
768^3 cells (all written to one place, with the same values) need 2^24 blocks,
which is 2^32 threads, the end of a launch's range; then a small one of its own."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_fills_of_more_than_a_launch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1303_0008_amd import vmg as V
    rng = np.random.Generator(np.random.PCG64(17))
    parent = torch.from_numpy(rng.standard_normal((40, 48, 32))).to("cuda")
    H = 1.0 / 32
    n, small, origin, last = (768, 768, 768), (20, 12, 36), (3, -7, 50), (-5, 9, 1)
    cells = 768 ** 3
    assert 38 * ((cells + 1023) // 1024) > 1 << 24
    big = V.make_grid(n, H / 2, V.DIRICHLET, 0, 0)
    tail = V.make_grid(small, H / 2, V.DIRICHLET, cells, 0)
    nan = float("nan")
    one = torch.full((cells + 20 * 12 * 36,), nan, dtype=torch.float64, device="cuda")
    for g, o in ((big, origin), (tail, last)):
        V.fill_interior(parent, H, [g], [o], one)
    many = torch.full_like(one, nan)
    V.fill_interior(parent, H, [big] * 38 + [tail], [origin] * 38 + [last], many)
    assert not bool(torch.isnan(one).any())
    assert torch.equal(one, many)
