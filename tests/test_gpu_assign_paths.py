"""Paths of the mass assignment that a call's sizes choose, against a plain torch
deposit: small and large bricks, several workgroups per brick, the hashed count of
grids with more bricks than an LDS table holds, block ranges of particles with and
without members of a region, and a workspace that only has room for large bricks."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def V():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1303_0008_amd import vmg
    vmg.load()
    return vmg


def deposit(torch, pos, n, tsc, region=None):
    """(mass, number of contributions) per cell; region = (h, corner) or None."""
    axes = []
    for a in range(3):
        if region is None:
            u = torch.remainder(pos[:, a], 1.0) * n[a]
        else:
            h, corner = region
            off = torch.remainder(pos[:, a] - corner[a], 1.0)
            u = torch.where(off > (n[a] + 2) * h, off - 1.0, off) / h
        if tsc:
            c = torch.floor(u)
            d = u - c - 0.5
            axes.append((c.long() - 1, (0.5 * (0.5 - d) ** 2, 0.75 - d * d, 0.5 * (0.5 + d) ** 2)))
        else:
            c = torch.floor(u - 0.5)
            t = u - 0.5 - c
            axes.append((c.long(), (1.0 - t, t)))
    # (many particles on few cells are summed on the host: torch's double adds to one
    # address from half a million threads are retried for minutes)
    cells = n[0] * n[1] * n[2]
    on_host = pos.shape[0] > cells
    mass = torch.zeros(cells, dtype=torch.float64, device=pos.device)
    hits = torch.zeros_like(mass)
    for k, wz in enumerate(axes[2][1]):
        for j, wy in enumerate(axes[1][1]):
            for i, wx in enumerate(axes[0][1]):
                cell = [axes[a][0] + o for a, o in enumerate((i, j, k))]
                one = torch.ones_like(wx)
                if region is not None:
                    for a in range(3):
                        one = torch.where((cell[a] >= 0) & (cell[a] < n[a]), one, 0.0)
                e = [torch.remainder(cell[a], n[a]) for a in range(3)]
                e = (e[2] * n[1] + e[1]) * n[0] + e[0]
                if on_host:
                    e = e.cpu().numpy()
                    for out, v in ((mass, wx * wy * wz * one), (hits, one)):
                        out += torch.from_numpy(np.bincount(e, v.cpu().numpy(), minlength=cells)).to(pos.device)
                else:
                    mass.index_add_(0, e, wx * wy * wz * one)
                    hits.index_add_(0, e, one)
    return mass.view(n[::-1]), hits.view(n[::-1])


# (cells, particles, ordered): small bricks; large ones; 27 bricks of 60000 particles
# (shared by workgroups); 8 of 8; one cell; more bricks than the table (33 x 33 x
# 65535 cells); ranges that do not end on a whole iteration
CASES = [((64, 64, 64), 100000, False), ((130, 128, 129), 300000, True), ((20, 24, 17), 1700000, False),
         ((16, 16, 16), 3000, True), ((1, 1, 1), 5000, False), ((33, 33, 65535), 20000, False),
         ((40, 9, 100), 2049, True), ((25, 70, 8), 1, False)]


@pytest.mark.parametrize("tsc", [False, True])
@pytest.mark.parametrize("where", ["box", "region", "small_workspace"])
@pytest.mark.parametrize("n,count,ordered", CASES)
def test_assign_paths(V, n, count, ordered, where, tsc):
    import torch
    if where == "region" and max(n) > 200:
        pytest.skip("a region is smaller than the box")
    g = torch.Generator(device="cuda").manual_seed(count + sum(n))
    pos = torch.rand((count, 3), generator=g, dtype=torch.float64, device="cuda")
    pos[: count // 3] = 0.4 + 0.05 * pos[: count // 3]          # a dense clump
    if ordered:
        pos = pos[torch.argsort(pos[:, 2])].contiguous()
    scheme = V.ASSIGN_TSC if tsc else V.ASSIGN_CIC
    if where == "region":
        h, corner = 1.0 / 256, [0.37, 0.39, 0.95]
        mean = count * h ** 3
        got = V.mass_assign_region(pos, n, h, corner, mean, scheme)
        mass, hits = deposit(torch, pos, n, tsc, (h, corner))
        places = 256
    else:
        mean = count / (n[0] * n[1] * n[2])
        work = None
        if where == "small_workspace":
            # room for bricks of 16^3 cells only: the smallest workspace a call accepts
            need = V.mass_assign_workspace(count, n)
            bricks = int(np.prod([-(-m // 16) for m in n]))
            least = sum(-(-b // 256) * 256 for b in (64 * bricks, 64 * bricks, 64 * bricks + 4,
                                                      -(-16 * bricks // 4096) * 4, 4 * count, 4 * count,
                                                      18 ** 3 * 8 * bricks, 4 * bricks))
            assert least <= need
            work = torch.empty(least, dtype=torch.uint8, device="cuda")
            with pytest.raises(V.VmgError):
                V.mass_assign(pos, n, scheme, workspace=work[: least - 256])
        got = V.mass_assign(pos, n, scheme, workspace=work)
        mass, hits = deposit(torch, pos, n, tsc)
        places = max(n)
    eps = np.finfo(np.float64).eps
    # each contribution is rounded once to 2^-40 and its weights come from a place
    # rounded by a few eps of its index on either side; the reference's sum rounds too
    bound = hits / mean * (2.0 ** -41 + 16 * places * eps) + eps * hits * (mass / mean + 1.0) + 4 * eps
    assert bool((torch.abs(got - (mass / mean - 1.0)) <= bound).all())
