"""A graph cache of the right sizes whose incidence lists hold entries out of
range is refused, and read without following them."""
import numpy as np
import pytest

import meshgen as mg

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1805_03949_amd as fea  # noqa: E402


@pytest.mark.parametrize("array,value", [(9, -1), (9, 1 << 40), (10, -1), (10, 0x7fffffff), (10, None)])
def test_incidence_lists_out_of_range(array, value, tmp_path):
    """array 9: the lists' bounds (int64), 10: the lists (int32); None: the
    number of elements, one beyond the last."""
    mesh = mg.hybrid_bands(6, seed=2, jitter=0.2)
    dm = fea.DeviceMesh(mesh)
    g = dm.graph()
    path = tmp_path / "g"
    g.save(path)
    g.destroy()
    raw = bytearray(path.read_bytes())
    off = 256 + 8 * int(np.frombuffer(raw, np.int64, 1, 248)[0])
    for _ in range(array):
        off += 8 + int(np.frombuffer(raw, np.int64, 1, off)[0])
    nb = int(np.frombuffer(raw, np.int64, 1, off)[0])
    dtype = np.int64 if array == 9 else np.int32
    n = nb // dtype().itemsize
    assert n == (mesh.n_nodes + 1 if array == 9 else mesh.conn.size)
    raw[off + 8:off + 8 + nb] = np.full(n, mesh.n_elems if value is None else value, dtype).tobytes()
    if array == 9 and value > 0:  # ascending bounds beyond the lists
        raw[off + 8:off + 8 + nb] = (np.arange(n, dtype=dtype) * value).tobytes()
    path.write_bytes(raw)
    with pytest.raises(fea.FeaError) as e:
        dm.graph(cache=path)
    assert e.value.code == -1 and "out of range" in str(e.value)
