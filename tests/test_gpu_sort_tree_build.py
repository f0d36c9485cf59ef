"""Cell and tree builds of shuffled lattices at the edges of the sort's tiles
(4,096 pairs), tile groups (64 tiles) and scanned groups (more than 64 of
them), and of the trees whose last levels one workgroup orders: neighbours at
distance 1 are counted exactly."""
import pytest

from paper_2301_12557_amd import fcfc

pytestmark = pytest.mark.gpu


def _lattice(m, seed):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    i = torch.randperm(m ** 3, generator=g, device="cuda")
    return torch.stack([i // (m * m), i // m % m, i % m], dim=1).to(torch.float64).contiguous()


@pytest.mark.parametrize("m", [1, 2, 15, 16, 17, 64, 65, 257])
def test_lattice_on_the_grid(m):
    x = _lattice(m, m)
    plan = fcfc.Plan("s", [0.0, 0.5, 1.2], box=float(max(m, 3)), n_hint=m ** 3)
    c = plan.build_cells(x)
    got, _ = plan.count(c)
    n = m ** 3
    want = 3 * n if m >= 3 else 3 * (n - m * m)
    assert got.cpu().tolist() == [0, want]
    c.close()
    plan.close()


@pytest.mark.parametrize("m,leaf", [(1, 32), (3, 32), (15, 32), (16, 32), (16, 128), (17, 128), (33, 32), (33, 101),
                                    (65, 77), (100, 128)])
def test_lattice_in_a_tree(m, leaf):
    x = _lattice(m, m + 1) + 5.0
    plan = fcfc.Plan("s", [0.0, 0.5, 1.2], n_hint=m ** 3, tree_leaf=leaf)
    plan.set_bounds((4.0,) * 3, (6.0 + m,) * 3)
    c = plan.build_cells(x)
    got, _ = plan.count(c)
    assert got.cpu().tolist() == [0, 3 * (m ** 3 - m * m)]
    c.close()
    plan.close()
