"""Batches at their edges: meshes that leave out the neo-Hookean flags or the
displacement next to one that gives them, and numbers of items around the
number of workgroups, from which on there is a queue."""
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


EPB = (25, 17, 12, 7)  # elements per tile and least item: tet4, pyr5, pen6, hex8


def _items(full, family, n):
    """Two meshes of one family with n items of one tile, the last item of each
    a partial one."""
    a = max(1, n // 3)
    return [mg.submesh(full, np.arange(k * EPB[family] - 1)) for k in (a, n - a) if k]


@pytest.mark.parametrize("variant", [fea.ROWOWNER, fea.ROWSYM])
@pytest.mark.parametrize("family", [0, 1, 2, 3])
def test_item_counts_around_the_workgroups(family, variant):
    """One item less than the family's workgroups, as many, one more (the
    queue starts) and three times as many: in type-sorted and in permuted
    order, in a static partition and in replays of a captured launch the
    results equal, bit for bit, those of items of many tiles (fewer items than
    workgroups, no queue), and to 1e-13 of the row scale one mesh's."""
    def batch(meshes, tile):
        return fea.Batch(meshes, tile=[tile] * 4)

    side = int(np.ceil((3 * 2048 * EPB[family] / int(mg.SUBELEMS[family])) ** (1 / 3))) + 1
    full = mg.cube_mesh(side, np.full(side ** 3, family, dtype=np.uint8), jitter=0.2, seed=family)
    # the family's workgroups, from the records of a launch that has three items for each
    b = batch([fea.DeviceMesh(m) for m in _items(full, family, 3 * 2048)], 1)
    b.assemble(variant=variant)
    assert b.n_items >= 3 * b.workers()
    w = int(b.cycles()[1].max()) + 1
    assert 256 <= w <= b.workers()
    rng = np.random.default_rng(family)
    for n in (w - 1, w, w + 1, 3 * w + 1):
        meshes = _items(full, family, n)
        dms = [fea.DeviceMesh(m) for m in meshes]
        ref = batch(dms, 64 * EPB[family]).assemble(variant=variant)
        b = batch(dms, 1)
        assert b.n_items == n
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            out = b.outputs()

            def same(what):
                assert all(torch.equal(x, y) for x, y in zip(out, ref)), (n, w, what)
                for x in out:
                    x.fill_(123)

            def run(what):
                b.assemble(vals=out[0], rhs=out[1], status=out[2], variant=variant)
                same(what)

            run("type-sorted")
            b.set_order(rng.permutation(n))
            run("permuted")
            b.capture(*out, variant=variant)
            for k in range(3):
                b.replay(1)
                same("replay")
                run("between replays")
            b.partition(fea.TYPE_SORTED)
            run("static partition")
        for m, dm in enumerate(dms):
            g = dm.graph()
            v1, r1, _ = dm.assemble(g, variant=variant)
            ev, er = fp64_errors(ref[0][b.vals_off[m]:b.vals_off[m + 1]].cpu().numpy(), v1.cpu().numpy(),
                                 g.export()["row_ptr"].cpu().numpy(), 3,
                                 ref[1][b.rhs_off[m]:b.rhs_off[m + 1]].cpu().numpy(), r1.cpu().numpy())
            assert ev <= 1e-13 and er <= 1e-13, (m, ev, er)
