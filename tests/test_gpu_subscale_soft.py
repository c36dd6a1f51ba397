"""Subgrid scale of elements without stiffness: Young's modulus 0 (tau is
infinite) or 1e-300 in every second element; against the CPU oracle, infinities
and NaN included."""
import numpy as np
import pytest

import meshgen as mg
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1805_03949_amd as fea  # noqa: E402
from tests.test_gpu_subscale import _scale  # noqa: E402


@pytest.mark.parametrize("family", [0, 1, 2, 3])
@pytest.mark.parametrize("young", [0.0, 1e-300])
def test_soft_elements(family, young):
    m = mg.cube_mesh(4, np.full(64, family, dtype=np.uint8), jitter=0.2, seed=family)
    rng = np.random.default_rng(5)
    m.source[:, :3] = rng.uniform(0.5, 1.5, (m.n_elems, 3)) * rng.choice([-1, 1], (m.n_elems, 3))
    m.source[::3, 1] = 0.0
    m.young[::2] = young
    u = mg.smooth_field(m, 3, seed=7, noise=0.3)
    with np.errstate(all="ignore"):
        gp, ref = oracle.subscale(m, u, model=oracle.ELASTIC)
        dm = fea.DeviceMesh(m)
        out, status = dm.subscale(dm.graph(), torch.from_numpy(u).to("cuda:0"))
        assert int(status.item()) == -1
        got = out.cpu().numpy()
        assert np.array_equal(np.isnan(got), np.isnan(ref))
        assert np.array_equal(np.isinf(got) * np.sign(got), np.isinf(ref) * np.sign(ref), equal_nan=True)
        assert young or np.isinf(ref).any()
        ok = np.isfinite(ref)
        # the part of L, 1e-11 of the scale that the subgrid-scale tests derive,
        # and as much of the value itself
        bound = 1e-11 * (np.abs(ref) + np.nan_to_num(_scale(m, u, 3, gp, oracle.ELASTIC))[:, None])
        assert np.all(np.abs(got - ref)[ok] <= bound[ok])
