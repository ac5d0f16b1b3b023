"""Mass assignment at the ends of its counting tables: the most bricks an LDS table
holds (16384, 64 KB of counters beside the kernel's own LDS) and one brick more
(counted in hashed chunks), in the box and in a region; and more than 128 bricks
with over 4096 particles each, which several workgroups share, heaviest bricks
first for the triangular-shaped cloud.  Reference and bound as for the other paths."""
import numpy as np
import pytest
from test_gpu_assign_paths import deposit

pytestmark = pytest.mark.gpu


def bricks(n):
    return int(np.prod([-(-m // 16) for m in n]))


@pytest.mark.parametrize("tsc", [False, True])
@pytest.mark.parametrize("ordered", [False, True])
@pytest.mark.parametrize("n,nb,count,region", [((512, 512, 256), 16384, 300000, False),
                                               ((512, 512, 256), 16384, 300000, True),
                                               ((77, 460, 1801), 16385, 300000, False),
                                               ((460, 77, 1801), 16385, 300000, True),
                                               ((112, 112, 48), 147, 900000, False)])
def test_table_limits(n, nb, count, region, ordered, tsc):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1303_0008_amd import vmg as V
    assert bricks(n) == nb
    g = torch.Generator(device="cuda").manual_seed(count + nb)
    pos = torch.rand((count, 3), generator=g, dtype=torch.float64, device="cuda")
    pos[: count // 3] = 0.4 + 0.05 * pos[: count // 3]          # a dense clump
    if ordered:
        pos = pos[torch.argsort(pos[:, 2])].contiguous()
    scheme = V.ASSIGN_TSC if tsc else V.ASSIGN_CIC
    if region:
        h, corner = 1.0 / 2048, [0.38, 0.41, 0.95]
        mean = count * h ** 3
        got = V.mass_assign_region(pos, n, h, corner, mean, scheme)
        mass, hits = deposit(torch, pos, n, tsc, (h, corner))
        places = 2048
        assert float(hits.sum()) > 100
    else:
        mean = count / (n[0] * n[1] * n[2])
        got = V.mass_assign(pos, n, scheme)
        mass, hits = deposit(torch, pos, n, tsc)
        places = max(n)
    eps = np.finfo(np.float64).eps
    bound = hits / mean * (2.0 ** -41 + 16 * places * eps) + eps * hits * (mass / mean + 1.0) + 4 * eps
    assert bool((torch.abs(got - (mass / mean - 1.0)) <= bound).all())
