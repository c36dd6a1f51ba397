"""Batches at their edges: meshes that leave out the neo-Hookean flags or the
displacement next to one that gives them."""
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


@pytest.mark.parametrize("variant", [fea.ROWOWNER, fea.ROWSYM, fea.ROWGATHER])
@pytest.mark.parametrize("precision", [fea.FP64, fea.MIXED])
def test_flags_and_field_may_be_left_out(variant, precision):
    """Equal, bit for bit, to the batch in which the missing flags and fields
    are zeros; in FP64 also within 1e-12 of the oracle."""
    meshes = [mg.hybrid_bands(5, seed=1, jitter=0.2), mg.heterogeneous(6, seed=2, brick=2, jitter=0.1),
              mg.hybrid_bands(4, seed=3, jitter=0.2), mg.hybrid_bands(7, seed=4, jitter=0.2)]
    missing = [("nh_flag", "u"), (), ("nh_flag",), ("nh_flag", "u")]
    assert meshes[1].nh_flag.any()
    full, part = [], []
    for m, names in zip(meshes, missing):
        for name in names:
            getattr(m, name)[:] = 0
        full.append(fea.DeviceMesh(m))
        part.append(fea.DeviceMesh(m))
        for name in names:
            setattr(part[-1], name, None)
    out = fea.F64 if precision == fea.FP64 else fea.F32
    b = fea.Batch(part, use_nh=True)
    got = b.assemble(precision=precision, out_dtype=out, variant=variant)
    ref = fea.Batch(full, use_nh=True).assemble(precision=precision, out_dtype=out, variant=variant)
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(got, ref))
    assert np.all(got[2].cpu().numpy() == -1)
    if precision == fea.FP64:
        for m, mesh in enumerate(meshes):
            og = oracle.mesh_graph(mesh)
            ov, orr = oracle.assemble(mesh, og, model=oracle.ELASTIC, use_nh=True)
            ev, er = fp64_errors(got[0][b.vals_off[m]:b.vals_off[m + 1]].cpu().numpy(), ov, og.row_ptr, 3,
                                 got[1][b.rhs_off[m]:b.rhs_off[m + 1]].cpu().numpy(), orr)
            assert ev <= 1e-12 and er <= 1e-12, (m, ev, er)
