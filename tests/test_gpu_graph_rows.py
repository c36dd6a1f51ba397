"""Rows of the graph at the sizes where the build changes its way: rows of
up to 64, 128, 256 and 512 slots, rows of 64, 65 and 200 elements, nodes of no
element and meshes of few nodes (long block lists), in shuffled order, every
exported and stored array equal to the one the definitions give."""
import threading

import numpy as np
import pytest

import meshgen as mg
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1805_03949_amd as fea  # noqa: E402

NODES = np.array([4, 5, 6, 8])


def _mesh(n_nodes, types, rng, hub):
    """Random connectivity without repeated nodes; the first `hub` elements
    hold node 0 (at any place), no other element does."""
    rows = []
    for e, t in enumerate(types):
        v = rng.choice(np.arange(1, n_nodes), NODES[t], replace=False)
        if e < hub:
            v[rng.integers(NODES[t])] = 0
        rows.append(v)
    order = rng.permutation(len(rows))
    rows, types = [rows[i] for i in order], types[order]
    cp = np.concatenate([[0], np.cumsum(NODES[types])]).astype(np.int64)
    return types.astype(np.uint8), cp, np.concatenate(rows).astype(np.int32)


CASES = [  # nodes, elements, families, elements at node 0
    (9, 1, [3], 1), (40, 8, [3], 8), (60, 16, [0], 16), (60, 17, [0], 17), (60, 12, [1], 12), (60, 13, [1], 13),
    (60, 10, [2], 10), (60, 11, [2], 11), (80, 9, [3], 9), (90, 25, [1], 25), (90, 26, [1], 26), (90, 32, [3], 32),
    (90, 33, [3], 33), (300, 51, [1], 51), (300, 52, [1], 52), (300, 64, [0, 1, 2, 3], 64), (300, 64, [3], 64),
    (300, 65, [0, 1, 2, 3], 65), (500, 200, [0, 1, 2, 3], 200), (10, 60, [0, 1, 2, 3], 40), (700, 600, [0, 2], 3),
]


@pytest.mark.parametrize("n,elems,fams,hub", CASES)
def test_rows(n, elems, fams, hub, tmp_path):
    rng = np.random.default_rng(1000 * n + elems)
    types, cp, conn = _mesh(n, rng.choice(fams, elems), rng, hub)
    n += 2  # two nodes of no element at the end
    dev = [torch.from_numpy(a).to("cuda:0") for a in (types, cp, conn)]
    g = fea.Graph(n, *dev)
    ex = {k: v.cpu().numpy() if torch.is_tensor(v) else v for k, v in g.export().items()}
    og = oracle.graph(n, types, cp, conn)
    for k in ("row_ptr", "col", "map_ptr", "e2nnz", "inv_ptr", "inv"):
        assert np.array_equal(ex[k], np.asarray(getattr(og, k))), k
    perm = np.argsort(types, kind="stable")
    assert np.array_equal(ex["type_perm"], perm)
    assert ex["type_seg"] == [int((types < t).sum()) for t in range(5)]
    # the stored arrays: type-sorted node lists and places, incidence lists
    g.save(str(tmp_path / "g"))
    raw = (tmp_path / "g").read_bytes()
    off = 256 + 8 * int(np.frombuffer(raw, np.int64, 1, 248)[0])
    arr = []
    while off < len(raw):
        nb = int(np.frombuffer(raw, np.int64, 1, off)[0])
        arr.append(raw[off + 8:off + 8 + nb])
        off += 8 + nb
    pnodes, pdest, prdest, n2e = (np.frombuffer(arr[i], np.int32) for i in (6, 7, 8, 10))
    n2e_ptr, n2a = np.frombuffer(arr[9], np.int64), np.frombuffer(arr[11], np.uint8)
    entries = np.concatenate([np.arange(cp[e], cp[e + 1]) for e in perm])
    slots = np.concatenate([np.arange(ex["map_ptr"][e], ex["map_ptr"][e + 1]) for e in perm])
    elem = np.repeat(np.arange(elems), NODES[types])
    inc = np.lexsort((elem, conn))  # incidence order: node, then element
    place = np.empty_like(inc)
    place[inc] = np.arange(len(inc))
    back = np.empty(len(ex["inv"]), np.int64)
    back[ex["inv"]] = np.arange(len(back))
    assert np.array_equal(n2e_ptr, np.concatenate([[0], np.cumsum(np.bincount(conn, minlength=n))]))
    assert np.array_equal(n2e, elem[inc])
    assert np.array_equal(n2a, (np.arange(len(conn)) - cp[elem])[inc])
    assert np.array_equal(pnodes, conn[entries])
    assert np.array_equal(prdest, place[entries])
    assert np.array_equal(pdest, back[slots])
    g.destroy()


@pytest.mark.parametrize("elems,hub", [(65536, 1), (65537, 1), (131075, 1), (70000, 70)])
def test_colouring_in_chunks(elems, hub):
    """Meshes of one chunk of the colouring's connectivity stream, one element
    more, two chunks and a remainder, and one that needs the wide masks: the
    colours are the first fit in element order."""
    rng = np.random.default_rng(elems)
    types = rng.choice([0, 0, 1, 2, 3], elems)
    cp = np.concatenate([[0], np.cumsum(NODES[types])]).astype(np.int64)
    # nodes 7 k + (0 .. n - 1) from a random k: distinct, neighbours by chance
    first = 1 + 7 * rng.integers(0, 30000, elems)
    conn = (np.repeat(first - cp[:-1], NODES[types]) + np.arange(cp[-1])).astype(np.int32)
    conn[cp[np.sort(rng.choice(elems, hub, replace=False))]] = 0
    n = int(conn.max()) + 1
    dev = [torch.from_numpy(a).to("cuda:0") for a in (types.astype(np.uint8), cp, conn)]
    g = fea.Graph(n, *dev)
    colour, nc = oracle.colour_greedy(n, cp, conn)
    assert g.n_colours == nc and (hub < 65 or nc > 64)
    assert np.array_equal(g.export()["colour"].cpu().numpy(), colour)
    g.destroy()


def test_graphs_of_two_threads_share_freed_memory():
    """Two threads, each on a stream of its own, build, assemble and destroy
    graphs of changing sizes, so that each takes memory that the other gave
    back: every result equals the one of a graph that lives alone."""
    cells = [6, 9, 12, 9, 6, 12]
    meshes = {n: fea.DeviceMesh(mg.hybrid_bands(n, seed=n, jitter=0.2)) for n in set(cells)}
    ref = {}
    for n, dm in meshes.items():
        g = dm.graph()
        ref[n] = [x.clone() for x in dm.assemble(g, variant=fea.ROWSYM)]
        torch.cuda.synchronize()
        g.destroy()
    wrong = []

    def work(order):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for n in order * 3:
                    g = meshes[n].graph()
                    got = meshes[n].assemble(g, variant=fea.ROWSYM)
                    torch.cuda.current_stream().synchronize()
                    wrong.extend(n for a, b in zip(got, ref[n]) if not torch.equal(a, b))
                    g.destroy()
        except Exception as e:  # noqa: BLE001
            wrong.append(e)

    threads = [threading.Thread(target=work, args=(o,)) for o in (cells, cells[::-1])]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
