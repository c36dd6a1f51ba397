"""Upper-triangle element tiles at the sizes where they can go wrong: one
element, one less and one more than a tile, several tiles and a remainder,
for every family, model and precision, against the CPU oracle."""
import numpy as np
import pytest

import meshgen as mg
import oracle
from tests.helpers import fp32_bound_L, fp64_errors, row_scale, within_fp32_bound

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1805_03949_amd as fea  # noqa: E402

EPB = (25, 17, 12, 7)  # elements per tile: tet4, pyr5, pen6, hex8


@pytest.mark.parametrize("family", [0, 1, 2, 3])
@pytest.mark.parametrize("tiles,extra", [(0, 1), (1, -1), (1, 0), (1, 1), (3, 2)])
def test_tile_remainders(family, tiles, extra):
    n = tiles * EPB[family] + extra
    cells = -(-n // int(mg.SUBELEMS[family]))
    side = max(2, int(np.ceil(cells ** (1 / 3))))
    full = mg.cube_mesh(side, np.full(side ** 3, family, dtype=np.uint8), jitter=0.2, seed=10 * n + family)
    mesh = mg.submesh(full, np.arange(n))
    dm = fea.DeviceMesh(mesh)
    g = dm.graph()
    og = oracle.mesh_graph(mesh)
    for model, B in ((fea.ELASTIC, 3), (fea.POISSON, 1)):
        om = oracle.ELASTIC if model == fea.ELASTIC else oracle.POISSON
        if model == fea.POISSON:
            mesh.source = mesh.source[:, :1].copy()
            mesh.source[:] = 1.0
            dm = fea.DeviceMesh(mesh, dofs=1)
        ref, rrhs, T, _ = oracle.assemble(mesh, og, model=om, with_terms=True)
        vals, rhs, status = dm.assemble(g, model=model, variant=fea.ROWSYM)
        assert int(status.item()) == -1
        ev, er = fp64_errors(vals.cpu().numpy(), ref, og.row_ptr, B, rhs.cpu().numpy(), rrhs)
        assert ev <= 1e-12 and er <= 1e-12, (family, n, model, ev, er)
        mv, _, _ = dm.assemble(g, model=model, variant=fea.ROWSYM, precision=fea.MIXED, out_dtype=fea.F32)
        floor = 1e-12 * row_scale(ref, og.row_ptr, B)
        assert within_fp32_bound(mv.cpu().numpy(), ref, T, fp32_bound_L(mesh.types), floor) <= 1.0
