"""Subgrid scale at the sizes where its launches can go wrong: one element, one
less and one more than a workgroup of every family, alone (the family's own
kernel) and next to another family (the common kernel), and both sides of the
common kernel's limits; against the CPU oracle within the bound that
test_gpu_subscale derives, and bit for bit between the two kernels."""
import numpy as np
import pytest

import meshgen as mg
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1805_03949_amd as fea  # noqa: E402
from tests.test_gpu_subscale import check  # noqa: E402

EPW = (256, 32, 42, 32)  # elements per workgroup: tet4, pyr5, pen6, hex8


@pytest.mark.parametrize("model", [oracle.POISSON, oracle.ELASTIC])
@pytest.mark.parametrize("family", [0, 1, 2, 3])
@pytest.mark.parametrize("groups,extra", [(0, 1), (1, -1), (1, 0), (1, 1), (3, 2)])
def test_group_remainders(family, groups, extra, model):
    n = groups * EPW[family] + extra
    side = max(3, int(np.ceil((-(-n // int(mg.SUBELEMS[family])) + 1) ** (1 / 3))))
    other = (family + 1) % 4
    cells = np.full(side ** 3, family, dtype=np.uint8)
    cells[-1] = other
    full = mg.cube_mesh(side, cells, jitter=0.2, seed=10 * n + family)
    alone = np.flatnonzero(full.types == family)[:n]
    both = np.concatenate([np.flatnonzero(full.types == other), alone])
    got = []
    for ids in (alone, both):
        m = mg.submesh(full, ids)
        u = mg.smooth_field(full, 1 if model == oracle.POISSON else 3, seed=7, noise=0.3)
        B = u.size // full.n_nodes
        nodes = mg.submesh(full, ids, return_nodes=True)[1]
        dm = fea.DeviceMesh(m)
        got.append(check(m, dm, dm.graph(), np.ascontiguousarray(u.reshape(-1, B)[nodes].reshape(-1)), model)[0])
    assert np.array_equal(got[0], got[1][-len(got[0]):])


# hex8 in nearly all cells: n^3 / 32 workgroups, the common kernel's limit for
# such meshes is 4096
@pytest.mark.parametrize("n", [50, 52])
def test_both_sides_of_the_rule(n):
    cells = np.full(n ** 3, mg.HEX8, dtype=np.uint8)
    cells[::1000] = mg.PEN6
    m = mg.cube_mesh(n, cells)
    dm = fea.DeviceMesh(m)
    check(m, dm, dm.graph(), mg.smooth_field(m, 3, seed=7, noise=0.3), oracle.ELASTIC)
