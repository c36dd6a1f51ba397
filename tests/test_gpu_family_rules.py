"""The neo-Hookean forms on both sides of the tile counts from which on every
family has a launch of its own, two families in equal halves: the tangent and
the Newton residual, upper triangle and row-owner, against the CPU oracle."""
import numpy as np
import pytest

import meshgen as mg
import oracle
from tests.helpers import fp64_errors

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1805_03949_amd as fea  # noqa: E402


# hex8 and tet4: 0.1914 n^3 tiles of the upper triangle, 0.3125 n^3 of the
# row-owner form; the lines are at 3400 (tangent), 2150 and 6000 (residual)
@pytest.mark.parametrize("n,variant,residual", [(26, fea.ROWSYM, False), (27, fea.ROWSYM, False), (22, fea.ROWSYM, True),
                                                (23, fea.ROWSYM, True), (26, fea.ROWOWNER, True),
                                                (27, fea.ROWOWNER, True)])
def test_both_sides(n, variant, residual):
    cells = np.where(np.arange(n ** 3) < n ** 3 // 2, mg.HEX8, mg.TET4).astype(np.uint8)
    m = mg.cube_mesh(n, cells, jitter=0.2, seed=n)
    rng = np.random.default_rng(n)
    m.nh_flag = (rng.random(len(m.types)) < 0.3).astype(np.uint8)
    m.u = mg.smooth_field(m, 3, seed=n) * 0.5
    dm = fea.DeviceMesh(m)
    g = dm.graph()
    og = oracle.mesh_graph(m)
    ref, rrhs = oracle.assemble(m, og, model=oracle.ELASTIC, use_nh=True)
    if residual:
        rrhs = oracle.residual(m, use_nh=True)
    vals, rhs, st = dm.assemble(g, model=fea.ELASTIC, variant=variant, use_nh=True, residual=residual)
    assert int(st.item()) == -1
    ev, er = fp64_errors(vals.cpu().numpy(), ref, og.row_ptr, 3, rhs.cpu().numpy(), rrhs)
    assert ev <= 1e-12 and er <= 1e-12
