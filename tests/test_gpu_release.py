"""Memory of destroyed graphs, kept for later ones, goes back on request."""
import pytest

import meshgen as mg

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1805_03949_amd as fea  # noqa: E402


def test_release_memory():
    dm = fea.DeviceMesh(mg.hybrid_bands(24, seed=1))
    keep, gone = dm.graph(), dm.graph()
    ref = [x.clone() for x in dm.assemble(keep, variant=fea.ROWSYM)]
    dm.assemble(gone, variant=fea.ROWSYM)
    gone.destroy()
    before = torch.cuda.mem_get_info()[0]
    fea.release_memory()
    assert torch.cuda.mem_get_info()[0] > before
    got = dm.assemble(keep, variant=fea.ROWSYM)  # the graph in use is untouched
    assert all(torch.equal(a, b) for a, b in zip(got, ref))
    keep.destroy()
