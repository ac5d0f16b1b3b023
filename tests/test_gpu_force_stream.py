"""Total force on grids whose outputs fill the last-level cache.

From 2^23 cells on, grids whose rows are whole 128-byte lines store their outputs
past the caches; just below, and with other rows, they do not.  Either way Psi is
the oracle's bit for bit and the force within 4 ulp of its largest value (the GPU
multiplies by 1/(2h), the oracle divides by 2h).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(256, 128, 256), (256, 128, 255), (240, 190, 187), (250, 190, 187)])
def test_streamed_force(oracle_mod, n):
    import torch
    from paper_1303_0008_amd import vmg as V
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(5151)
    phi_n, phi = (rng.standard_normal(n[::-1]) for _ in range(2))
    h = 1.0 / 256
    a, b = (torch.from_numpy(x).to("cuda") for x in (phi_n, phi))
    psi, g = V.total_force(a, b, h, psi=torch.empty_like(a))
    psi_o, g_o = oracle_mod.total_force(phi_n, phi, h)
    assert np.array_equal(psi.cpu().numpy(), psi_o)
    assert np.abs(g.cpu().numpy() - g_o).max() <= 4 * np.finfo(np.float64).eps * np.abs(g_o).max()
    _, g2 = V.total_force(a, b, h)
    assert torch.equal(g2, g)
