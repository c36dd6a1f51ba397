"""Timed workloads of the assembly library, through its Python entry points.

A case is a dict of plain values; `prepare` makes what a program holds before
the call (mesh, material, sparsity graph or batch, output buffers, on the
GPU, from the seed alone), `run` is one pass, `work` what a pass cannot do
without, `exact` the same outputs in 64 bits by plain torch.

Meshes tile the unit cube with n^3 cells, each one hex8, two pen6, six tet4
or six pyr5 around a centre node; interior nodes are moved by up to 5% of a
cell, Poisson's ratio is drawn per element. `mix` says how the cells get
their families: one family everywhere, "bands" (four equal layers), "split"
(40 / 30 / 20 / 10 % hex8 / tet4 / pen6 / pyr5 layers) or "random" (drawn cell
by cell, so that nearly every row touches several families).

kind "assemble"  one mesh, matrix and right-hand side, graph already built;
                 "nh" is the share of 8^3-cell bricks with the neo-Hookean
                 tangent, "residual" asks for the Newton residual
kind "batch"     many meshes of different sizes in one persistent launch
kind "subscale"  the element-wise subgrid scale of a nodal field
kind "build"     a new mesh: sparsity graph and its exported maps, then the
                 first assembly on it
kind "cost"      the learned cost model: standardise, train, predict
"""
import math
import types as _types

import numpy as np
import torch

import paper_1805_03949_amd as fea

TET4, PYR5, PEN6, HEX8 = 0, 1, 2, 3
NODES = (4, 5, 6, 8)
POINTS = (1, 8, 6, 8)
DEV = "cuda"

# corners 0 c000, 1 c100, 2 c110, 3 c010, 4 .. 7 the same at the top, 8 centre
CORNERS = ((0, 0, 0), (1, 0, 0), (1, 1, 0), (0, 1, 0), (0, 0, 1), (1, 0, 1), (1, 1, 1), (0, 1, 1))
CELL = {
    HEX8: ((0, 1, 2, 3, 4, 5, 6, 7),),
    PEN6: ((0, 1, 2, 4, 5, 6), (0, 2, 3, 4, 6, 7)),
    TET4: ((0, 1, 2, 6), (0, 2, 3, 6), (0, 5, 1, 6), (0, 4, 5, 6), (0, 3, 7, 6), (0, 7, 4, 6)),
    PYR5: ((0, 1, 2, 3, 8), (4, 7, 6, 5, 8), (0, 4, 5, 1, 8), (3, 2, 6, 7, 8), (0, 3, 7, 4, 8), (1, 5, 6, 2, 8)),
}
FAMILY = {"tet4": TET4, "pyr5": PYR5, "pen6": PEN6, "hex8": HEX8}


def listed():
    def asm(name, n, mix, model="elastic", precision="fp64", variant="rowsym", nh=0.0, residual=False):
        return dict(name=name, kind="assemble", n=n, mix=mix, model=model, precision=precision, variant=variant,
                    nh=nh, residual=residual)

    return [
        # a scalar problem on a small grid, the smallest call: launches and latency count
        asm("poisson_hex16", 16, "hex8", model="poisson"),
        # a small hybrid solid, one call of a time loop on a coarse mesh
        asm("small_hybrid10", 10, "bands"),
        # a hybrid mesh of ordinary size, plain double precision
        asm("hybrid96_fp64", 96, "bands"),
        # the same in mixed precision with single-precision output
        asm("hybrid96_mixed", 96, "bands", precision="mixed"),
        # a production-sized mesh of one GPU (13 million elements, 95 million blocks)
        asm("large160_fp64", 160, "split"),
        # default options (row-owner scatter) on a mesh of odd size whose cells mix families at random
        asm("default_random47", 47, "random", variant="rowowner"),
        # a Newton step of the solid: tangent and residual, 30% of the bricks neo-Hookean
        asm("newton64", 64, "split", nh=0.3, residual=True),
        # the neo-Hookean tangent in mixed precision on a larger mesh
        asm("hetero96_mixed", 96, "split", precision="mixed", nh=0.3),
        # many independent meshes in one persistent launch, mixed precision
        dict(name="batch24_mixed", kind="batch", meshes=24, lo=8, hi=36, precision="mixed"),
        # the element loop after an assembly that scatters nothing
        dict(name="subscale96", kind="subscale", n=96, mix="bands", model="elastic"),
        # a mesh that has just changed: graph, maps and the first assembly on it
        dict(name="remesh48", kind="build", n=48, mix="bands"),
        # learning the cost of work items from one recorded assembly
        dict(name="cost_train60k", kind="cost", items=60000, steps=10),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["assemble"] * 5 + ["batch", "subscale", "build", "cost"])
    mix = rng.choice(["bands", "split", "random", "hex8", "tet4", "pen6", "pyr5"])
    if kind == "assemble":
        model = rng.choice(["elastic", "elastic", "elastic", "poisson"])
        nh = rng.choice([0.0, 0.0, 0.3]) if model == "elastic" else 0.0
        residual = nh > 0 and rng.random() < 0.5
        precision = "fp64" if residual else rng.choice(["fp64", "mixed"])
        return dict(kind=kind, n=_log_int(rng, 8, 100), mix=mix, model=model, precision=precision,
                    variant=rng.choice(["rowsym", "rowsym", "rowowner"]), nh=nh, residual=residual)
    if kind == "batch":
        return dict(kind=kind, meshes=_log_int(rng, 3, 30), lo=rng.randint(4, 12), hi=rng.randint(14, 36),
                    precision=rng.choice(["fp64", "mixed"]))
    if kind == "subscale":
        return dict(kind=kind, n=_log_int(rng, 8, 100), mix=mix, model=rng.choice(["elastic", "poisson"]))
    if kind == "build":
        return dict(kind=kind, n=_log_int(rng, 8, 60), mix=mix)
    return dict(kind=kind, items=_log_int(rng, 2000, 100000), steps=rng.randint(4, 10))


# ------------------------------------------------------------------ inputs
def _cell_types(n, mix, draw):
    if mix in FAMILY:
        return torch.full((n ** 3,), FAMILY[mix], dtype=torch.int64, device=DEV)
    if mix == "random":  # the connectivity belongs to the case: only values come from the seed
        gen = torch.Generator(device=DEV)
        gen.manual_seed(1000 * n + draw)
        p = torch.rand(4, generator=gen, device=DEV) + 0.1
        return torch.multinomial(p, n ** 3, replacement=True, generator=gen)
    if mix == "bands":
        q = n // 4
        lay = [(HEX8, q), (PEN6, q), (TET4, q), (PYR5, n - 3 * q)]
    else:
        nh, nt, npn = round(0.4 * n), round(0.3 * n), round(0.2 * n)
        lay = [(HEX8, nh), (TET4, nt), (PEN6, npn), (PYR5, n - nh - nt - npn)]
    t = torch.tensor([f for f, k in lay for _ in range(k)], dtype=torch.int64, device=DEV)
    return t.repeat_interleave(n * n)


def _mesh(n, mix, seed, dofs=3, nh=0.0, draw=0):
    """A mesh with its material, source and a smooth displacement, on the GPU."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    m = n + 1
    ct = _cell_types(n, mix, draw)
    cell = torch.arange(n ** 3, device=DEV)
    ci, cj, ck = cell % n, (cell // n) % n, cell // (n * n)
    pyr = (ct == PYR5).nonzero().flatten()
    n_nodes = m ** 3 + pyr.numel()
    centre = torch.zeros(n ** 3, dtype=torch.int64, device=DEV)
    centre[pyr] = m ** 3 + torch.arange(pyr.numel(), device=DEV)
    nodes = torch.stack([ci + dx + m * (cj + dy + m * (ck + dz)) for dx, dy, dz in CORNERS] + [centre], dim=1)
    per_cell = torch.tensor([len(CELL[t]) for t in range(4)], device=DEV)[ct]
    first = torch.cumsum(per_cell, 0) - per_cell
    n_elems = int(per_cell.sum())
    types = ct.repeat_interleave(per_cell).to(torch.uint8)
    conn_ptr = torch.zeros(n_elems + 1, dtype=torch.int64, device=DEV)
    conn_ptr[1:] = torch.cumsum(torch.tensor(NODES, device=DEV)[types.long()], 0)
    conn = torch.empty(int(conn_ptr[-1]), dtype=torch.int32, device=DEV)
    for t in range(4):
        cells = (ct == t).nonzero().flatten()
        for s, corners in enumerate(CELL[t]):
            base = conn_ptr[first[cells] + s]
            for a, lab in enumerate(corners):
                conn[base + a] = nodes[cells, lab].to(torch.int32)
    h = 1.0 / n
    idx = torch.arange(m ** 3, device=DEV)
    g = torch.stack([idx % m, (idx // m) % m, idx // (m * m)], dim=1)
    inside = ((g > 0) & (g < n)).all(dim=1)
    X = torch.cat([g.double(), torch.stack([ci, cj, ck], dim=1)[pyr].double() + 0.5])
    inside = torch.cat([inside, torch.ones(pyr.numel(), dtype=torch.bool, device=DEV)])
    X = (X + inside[:, None] * (torch.rand(n_nodes, 3, generator=gen, device=DEV, dtype=torch.float64) - 0.5) * 0.1) * h
    nu = 0.2 + 0.15 * torch.rand(n_elems, generator=gen, device=DEV, dtype=torch.float64)
    source = torch.zeros(n_elems, dofs, dtype=torch.float64, device=DEV)
    source[:, dofs - 1] = 1.0 if dofs == 1 else -1.0
    # smooth field of three sine modes, gradient bound about 0.1
    k = torch.randint(1, 3, (3, 3), generator=gen, device=DEV).double()
    amp = (torch.rand(3, dofs, generator=gen, device=DEV, dtype=torch.float64) - 0.5) * 0.01
    phase = 6.28 * torch.rand(3, generator=gen, device=DEV, dtype=torch.float64)
    wave = torch.sin(2 * math.pi * (X[:, None, :] * k).sum(2) + phase)
    u = (wave[:, :, None] * amp).sum(1).reshape(-1).contiguous()
    nh_flag = torch.zeros(n_elems, dtype=torch.uint8, device=DEV)
    if nh:
        nb = (n + 7) // 8
        brick = torch.rand(nb ** 3, generator=gen, device=DEV) < nh
        of = ci // 8 + nb * (cj // 8 + nb * (ck // 8))
        nh_flag = brick[of].repeat_interleave(per_cell).to(torch.uint8)
    return _types.SimpleNamespace(
        n_nodes=n_nodes, n_elems=n_elems, types=types, conn_ptr=conn_ptr, conn=conn, x=X[:, 0].contiguous(),
        y=X[:, 1].contiguous(), z=X[:, 2].contiguous(), young=torch.ones(n_elems, dtype=torch.float64, device=DEV),
        nu=nu, nh_flag=nh_flag, u=u, source=source)


def _dofs(case):
    return 1 if case.get("model") == "poisson" else 3


def _batch_meshes(case, seed):
    sizes = np.round(np.linspace(case["lo"], case["hi"], case["meshes"])).astype(int)
    sizes = np.random.default_rng(3).permutation(sizes)
    return [_mesh(int(n), "random", seed + 7919 * k, draw=k) for k, n in enumerate(sizes)]


def _cost_inputs(case, seed):
    """Item features and log-cycles shaped as recorded ones: family one-hot,
    shares, logarithms of counts and sizes; cost by family and count."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    n = case["items"]
    f = torch.rand(n, fea.N_FEATURES, generator=gen, device=DEV)
    fam = torch.randint(0, 4, (n,), generator=gen, device=DEV)
    f[:, :4] = torch.nn.functional.one_hot(fam, 4).float()
    f[:, 5] = 3.5 + 2.5 * f[:, 5]
    f[:, 6] = 4 * f[:, 6]
    f[:, 10] = -6 + f[:, 10]
    f[:, 11] = 0.0
    t = 9.0 + 0.3 * fam + 0.69 * f[:, 5] + 0.8 * f[:, 4] + 0.1 * torch.randn(n, generator=gen, device=DEV)
    return f.contiguous(), t.float().contiguous()


def _outputs(case, nnz, n_nodes):
    B = _dofs(case)
    odt = torch.float32 if case.get("precision") == "mixed" else torch.float64
    return (torch.empty(nnz * B * B, dtype=odt, device=DEV), torch.empty(n_nodes * B, dtype=odt, device=DEV),
            torch.empty(1, dtype=torch.int32, device=DEV))


def prepare(case, seed):
    s = _types.SimpleNamespace(case=case)
    kind = case["kind"]
    if kind == "cost":
        s.feats, s.target = _cost_inputs(case, seed)
        return s
    if kind == "batch":
        s.meshes = _batch_meshes(case, seed)
        s.batch = fea.Batch(s.meshes, model=fea.ELASTIC)
        s.out = s.batch.outputs(fea.F32 if case["precision"] == "mixed" else fea.F64)
        return s
    s.mesh = m = _mesh(case["n"], case["mix"], seed, dofs=_dofs(case), nh=case.get("nh", 0.0))
    if kind == "build":
        return s
    s.graph = fea.Graph(m.n_nodes, m.types, m.conn_ptr, m.conn)
    if kind == "subscale":
        n_points, _ = s.graph.gauss_points()
        s.out = (torch.empty(n_points, _dofs(case), dtype=torch.float64, device=DEV),
                 torch.empty(1, dtype=torch.int32, device=DEV))
    else:
        s.out = _outputs(case, s.graph.nnz, m.n_nodes)
    return s


# ------------------------------------------------------------------- a pass
def _assemble(case, m, graph, out):
    poisson = case.get("model") == "poisson"
    nh = case.get("nh", 0.0) > 0
    mixed = case.get("precision") == "mixed"
    return fea.assemble(graph, m.x, m.y, m.z, m.types, m.conn_ptr, m.conn, m.source,
                        model=fea.POISSON if poisson else fea.ELASTIC, young=m.young, nu=None if poisson else m.nu,
                        nh_flag=m.nh_flag if nh else None, u=m.u if nh else None,
                        precision=fea.MIXED if mixed else fea.FP64, out_dtype=fea.F32 if mixed else fea.F64,
                        variant=case.get("variant", "rowsym"), residual=bool(case.get("residual", False)),
                        vals=out[0], rhs=out[1], status=out[2])


def run(s):
    case, kind = s.case, s.case["kind"]
    if kind == "assemble":
        return _assemble(case, s.mesh, s.graph, s.out)
    if kind == "batch":
        mixed = case["precision"] == "mixed"
        return s.batch.assemble(precision=fea.MIXED if mixed else fea.FP64, out_dtype=fea.F32 if mixed else fea.F64,
                                vals=s.out[0], rhs=s.out[1], status=s.out[2], variant=fea.ROWSYM)
    if kind == "subscale":
        m, poisson = s.mesh, case["model"] == "poisson"
        return fea.subscale(s.graph, m.x, m.y, m.z, m.u, m.source, model=fea.POISSON if poisson else fea.ELASTIC,
                            young=m.young, nu=None if poisson else m.nu, out=s.out[0], status=s.out[1])
    if kind == "build":
        m = s.mesh
        g = fea.Graph(m.n_nodes, m.types, m.conn_ptr, m.conn)
        vals, rhs, status = _assemble(case, m, g, _outputs(case, g.nnz, m.n_nodes))
        return dict(g.export(), colours=g.n_colours, vals=vals, rhs=rhs, status=status)
    cm = fea.CostModel(seed=7)
    cm.fit_norm(s.feats)
    loss = cm.train(s.feats, s.target, steps=case["steps"])
    return cm.predict(s.feats), loss


# ------------------------------------------------------- what it cannot avoid
def _counts(n, mix):
    """(elements per family, nodes) of a mesh, for "random" on average."""
    if mix in FAMILY:
        cells = [n ** 3 if t == FAMILY[mix] else 0 for t in range(4)]
    elif mix == "random":
        cells = [n ** 3 / 4] * 4
    elif mix == "bands":
        q = n // 4
        cells = [q * n * n, (n - 3 * q) * n * n, q * n * n, q * n * n]
    else:
        nh, nt, npn = round(0.4 * n), round(0.3 * n), round(0.2 * n)
        cells = [nt * n * n, (n - nh - nt - npn) * n * n, npn * n * n, nh * n * n]
    return [c * len(CELL[t]) for t, c in enumerate(cells)], (n + 1) ** 3 + cells[PYR5], cells


def _blocks(n, mix):
    """Nonzero blocks, from the neighbours of a node in each family's grid."""
    _, _, cells = _counts(n, mix)
    return sum(c * k for c, k in zip(cells, (15, 36, 21, 27)))  # tet4, pyr5 (corner and centre), pen6, hex8


def work(case):
    kind = case["kind"]
    if kind == "cost":
        n = case["items"]
        mac = 12 * 64 + 64 * 64 + 64
        return {"bytes": n * 4 * (fea.N_FEATURES + 2) + 4 * fea.N_PARAMS, "flops": 2.0 * mac * n * (3 * case["steps"] + 1)}
    if kind == "batch":
        one = [work(dict(case, kind="assemble", n=int(round(k)), mix="random", model="elastic"))
               for k in np.linspace(case["lo"], case["hi"], case["meshes"])]
        return {"bytes": sum(w["bytes"] for w in one), "flops": sum(w["flops"] for w in one)}
    B = _dofs(case)
    elems, nodes, _ = _counts(case["n"], case["mix"])
    E = sum(elems)
    conn = sum(e * NODES[t] for t, e in enumerate(elems))
    size = 4 if case.get("precision") == "mixed" else 8
    read = nodes * 24 + conn * 4 + E * (8 + 8 * (B == 3) + 8 * B) + (24 * nodes if case.get("nh") or kind == "subscale" else 0)
    if kind == "subscale":
        pts = sum(e * POINTS[t] for t, e in enumerate(elems))
        return {"bytes": read + pts * 8 * B, "flops": pts * (150.0 if B == 1 else 480.0)}
    blocks = _blocks(case["n"], case["mix"])
    written = (blocks * B * B + nodes * B) * size
    if kind == "build":
        slots = sum(e * NODES[t] ** 2 for t, e in enumerate(elems))
        written += 4 * blocks + 8 * (blocks + 2 * nodes + E) + 8 * slots + 6 * E
    # geometry per point, then the blocks a <= b: an outer product per point
    flops = 0.0
    for t, e in enumerate(elems):
        n, q = NODES[t], POINTS[t]
        flops += e * (q * (18 * n + 60 + 15 * n) + n * (n + 1) / 2 * q * (2 * B * B + 3))
    return {"bytes": read + written, "flops": flops * (1 + 1.5 * case.get("nh", 0.0))}


# ------------------------------------------------------------ 64-bit results
def _reference(t):
    """Shape functions, first and second derivatives at the Gauss points, and
    the weights: N [q, n], dN [q, n, 3], d2 [q, n, 3] (pairs 01, 02, 12), w."""
    g = 1.0 / math.sqrt(3.0)
    if t == TET4:
        N = np.full((1, 4), 0.25)
        dN = np.array([[[-1, -1, -1], [1, 0, 0], [0, 1, 0], [0, 0, 1]]], dtype=float)
        return N, dN, np.zeros((1, 4, 3)), np.array([1 / 6])
    if t == PEN6:
        tri = ((1 / 6, 1 / 6), (2 / 3, 1 / 6), (1 / 6, 2 / 3))
        pts = [(r, s, z) for z in (-g, g) for r, s in tri]
        N, dN, d2 = np.zeros((6, 6)), np.zeros((6, 6, 3)), np.zeros((6, 6, 3))
        dL = ((-1, -1), (1, 0), (0, 1))
        for q, (r, s, z) in enumerate(pts):
            L = (1 - r - s, r, s)
            for a in range(6):
                k, sg = a % 3, -1.0 if a < 3 else 1.0
                f = 0.5 * (1 + sg * z)
                N[q, a] = L[k] * f
                dN[q, a] = (dL[k][0] * f, dL[k][1] * f, 0.5 * sg * L[k])
                d2[q, a] = (0.0, 0.5 * sg * dL[k][0], 0.5 * sg * dL[k][1])
        return N, dN, d2, np.full(6, 1 / 6)
    sg = np.array(CORNERS, dtype=float) * 2 - 1
    pts = np.array([(x, y, z) for z in (-g, g) for y in (-g, g) for x in (-g, g)])
    f = 0.5 * (1 + sg[None] * pts[:, None])  # [q, 8, 3]
    N = f.prod(2)
    dN = np.stack([0.5 * sg[:, 0] * f[..., 1] * f[..., 2], 0.5 * sg[:, 1] * f[..., 0] * f[..., 2],
                   0.5 * sg[:, 2] * f[..., 0] * f[..., 1]], axis=2)
    d2 = np.stack([0.25 * sg[:, 0] * sg[:, 1] * f[..., 2], 0.25 * sg[:, 0] * sg[:, 2] * f[..., 1],
                   0.25 * sg[:, 1] * sg[:, 2] * f[..., 0]], axis=2)
    if t == PYR5:  # the top four corners are the apex
        N, dN, d2 = (np.concatenate([v[:, :4], v[:, 4:].sum(1, keepdims=True)], axis=1) for v in (N, dN, d2))
    return N, dN, d2, np.ones(8)


def _families(m, chunk=150000):
    for t in range(4):
        ids = (m.types == t).nonzero().flatten()
        for e in ids.split(chunk):
            yield t, e, m.conn[m.conn_ptr[e][:, None] + torch.arange(NODES[t], device=DEV)].long()


def _geometry(m, t, c):
    N, dN, d2, w = (torch.from_numpy(np.ascontiguousarray(v)).to(DEV) for v in _reference(t))
    X = torch.stack([m.x, m.y, m.z], dim=1)[c]                                  # [E, n, 3]
    J = (X[:, None, :, :, None] * dN[None, :, :, None, :]).sum(2)               # [E, q, 3, 3]: dx_i / dxi_j
    det = torch.linalg.det(J)
    inv = torch.linalg.inv(J)
    G = (dN[None, :, :, :, None] * inv[:, :, None]).sum(3)                      # [E, q, n, 3]
    return X, N, d2, inv, G, w * det


def _lame(m, e):
    E, nu = m.young[e], m.nu[e]
    return E * nu / ((1 + nu) * (1 - 2 * nu)), E / (2 * (1 + nu))


def _element(m, t, e, c, B, nh, residual):
    """Element matrices [E, n, n, B, B] and right-hand sides [E, n, B]."""
    _, N, _, _, G, wd = _geometry(m, t, c)
    f = (wd[:, :, None] * N).sum(1)[:, :, None] * m.source[e][:, None, :]
    n = NODES[t]
    if B == 1:
        K = (wd[:, :, None, None, None] * G[:, :, :, None, :] * G[:, :, None, :, :]).sum((1, 4))
        return K[..., None, None], f
    lam, mu = _lame(m, e)
    eye = torch.eye(3, dtype=torch.float64, device=DEV)
    flat = G.reshape(len(e), POINTS[t], 3 * n)
    S = ((wd[:, :, None] * flat).transpose(1, 2).contiguous() @ flat).reshape(-1, n, 3, n, 3).permute(0, 1, 3, 2, 4)
    lam_, mu_ = lam[:, None, None, None, None], mu[:, None, None, None, None]
    K = lam_ * S + mu_ * S.transpose(3, 4) + mu_ * S.diagonal(dim1=3, dim2=4).sum(-1)[..., None, None] * eye
    U = None
    if nh or residual:
        U = m.u.reshape(-1, 3)[c]
        H = (U[:, None, :, :, None] * G[:, :, :, None, :]).sum(2)               # du_i / dx_j
    if residual:
        sig = lam[:, None, None, None] * H.diagonal(dim1=2, dim2=3).sum(-1)[..., None, None] * eye \
            + mu[:, None, None, None] * (H + H.transpose(2, 3))
    if nh:
        on = m.nh_flag[e].bool()
        F = eye + H
        Fi, lnJ = torch.linalg.inv(F), torch.log(torch.linalg.det(F))
        h = (G[..., :, None] * Fi[:, :, None]).sum(3)                           # F^-T grad N
        hf = h.reshape(len(e), POINTS[t], 3 * n)

        def outer(wt, a, b):
            r = (wt[:, :, None] * a).transpose(1, 2).contiguous() @ b
            return r.reshape(-1, n, 3, n, 3).permute(0, 1, 3, 2, 4)

        c2 = mu[:, None] - lam[:, None] * lnJ
        Kn = outer(wd * lam[:, None], hf, hf) + outer(wd * c2, hf, hf).transpose(3, 4)
        tr = (wd[:, :, None, None, None] * G[:, :, :, None, :] * G[:, :, None, :, :]).sum((1, 4)) * mu[:, None, None]
        Kn = Kn + tr[..., None, None] * eye
        K = torch.where(on[:, None, None, None, None], Kn, K)
        if residual:
            P = mu[:, None, None, None] * F - c2[..., None, None] * Fi.transpose(2, 3)
            sig = torch.where(on[:, None, None, None], P, sig)
    if residual:
        f = f - (wd[:, :, None, None, None] * sig[:, :, None] * G[:, :, :, None, :]).sum((1, 4))
    return K, f


def _exact_system(m, B, nh=False, residual=False):
    N = m.n_nodes
    keys = []
    for t, e, c in _families(m, 1 << 62):
        keys.append(torch.unique((c[:, :, None] * N + c[:, None, :]).reshape(-1)))
    keys = torch.unique(torch.cat(keys))
    vals = torch.zeros(keys.numel(), B * B, dtype=torch.float64, device=DEV)
    rhs = torch.zeros(N, B, dtype=torch.float64, device=DEV)
    for t, e, c in _families(m):
        K, f = _element(m, t, e, c, B, nh, residual)
        at = torch.searchsorted(keys, (c[:, :, None] * N + c[:, None, :]).reshape(-1))
        vals.index_add_(0, at, K.reshape(-1, B * B))
        rhs.index_add_(0, c.reshape(-1), f.reshape(-1, B))
    return vals.reshape(-1), rhs.reshape(-1)


def _exact_subscale(m, B):
    q = torch.tensor(POINTS, device=DEV)[m.types.long()]
    ptr = torch.cumsum(q, 0) - q
    out = torch.zeros(int(q.sum()), B, dtype=torch.float64, device=DEV)
    pairs = ((0, 1), (0, 2), (1, 2))
    for t, e, c in _families(m):
        X, _, d2, inv, G, wd = _geometry(m, t, c)
        U = m.u.reshape(-1, B)[c]
        g = (U[:, None, :, :, None] * G[:, :, :, None, :]).sum(2)               # [E, q, B, 3]
        Hu = (U[:, None, :, :, None] * d2[None, :, :, None, :]).sum(2)          # [E, q, B, 3 pairs]
        Hx = (X[:, None, :, :, None] * d2[None, :, :, None, :]).sum(2)
        M3 = Hu - (g[..., None] * Hx[:, :, None]).sum(3)
        M = torch.zeros(*M3.shape[:3], 3, 3, dtype=torch.float64, device=DEV)
        for k, (i, j) in enumerate(pairs):
            M[..., i, j] = M[..., j, i] = M3[..., k]
        i5 = inv[:, :, None]
        H = i5.transpose(3, 4) @ M @ i5                                         # second derivatives in x
        V = wd.sum(1)
        r = m.source[e][:, None, :]
        lap = H.diagonal(dim1=3, dim2=4).sum(-1)
        if B == 1:
            k, L = torch.ones_like(V), lap
        else:
            lam, mu = _lame(m, e)
            div = torch.stack([sum(H[:, :, a, i, a] for a in range(3)) for i in range(3)], dim=2)
            k, L = mu, mu[:, None, None] * lap + (lam + mu)[:, None, None] * div
        tau = V ** (2.0 / 3.0) / (4 * k)
        at = ptr[e][:, None] + torch.arange(POINTS[t], device=DEV)
        out[at.reshape(-1)] = (tau[:, None, None] * (r + L)).reshape(-1, B)
    return out


def _initial_weights(seed):
    """He-normal weights and zero biases of the 12-64-64-1 model: Box-Muller
    normals of a SplitMix64 stream, rounded to single precision."""
    x, full = seed, (1 << 64) - 1

    def uniform():
        nonlocal x
        x = (x + 0x9e3779b97f4a7c15) & full
        z = ((x ^ (x >> 30)) * 0xbf58476d1ce4e5b9) & full
        z = ((z ^ (z >> 27)) * 0x94d049bb133111eb) & full
        return (z ^ (z >> 31)) >> 11

    def normal(fan_in):
        u1, u2 = (uniform() + 1.0) * 2.0 ** -53, uniform() * 2.0 ** -53
        return math.sqrt(-2.0 * math.log(u1)) * math.cos(2.0 * math.pi * u2) * math.sqrt(2.0 / fan_in)

    w = [normal(12) for _ in range(64 * 12)] + [0.0] * 64 + [normal(64) for _ in range(64 * 64)] + [0.0] * 64
    w += [normal(64) for _ in range(64)] + [0.0]
    return torch.tensor(w, dtype=torch.float32).double().to(DEV)


def _exact_cost(case, seed):
    """The same training in 64 bits, from the same initial weights."""
    f, t = (v.double() for v in _cost_inputs(case, seed))
    start = _initial_weights(7)
    shapes = ((64, 12), (64,), (64, 64), (64,), (64,), (1,))
    P = [p.reshape(s).clone().requires_grad_() for p, s in zip(start.split([math.prod(s) for s in shapes]), shapes)]
    mean, sd = f.mean(0), f.std(0, correction=0)
    z = (f - mean) / torch.where(sd > 1e-12, sd, torch.ones_like(sd))

    def model():
        a = torch.relu(z @ P[0].T + P[1])
        return torch.relu(a @ P[2].T + P[3]) @ P[4] + P[5]

    M, V, hist = [torch.zeros_like(p) for p in P], [torch.zeros_like(p) for p in P], []
    for k in range(1, case["steps"] + 1):
        loss = ((model() - t) ** 2).mean()
        hist.append(loss.detach())
        grads = torch.autograd.grad(loss, P)
        with torch.no_grad():
            for p, g, m1, v1 in zip(P, grads, M, V):
                m1.mul_(0.9).add_(0.1 * g)
                v1.mul_(0.999).add_(0.001 * g * g)
                p -= 1e-3 * (m1 / (1 - 0.9 ** k)) / ((v1 / (1 - 0.999 ** k)).sqrt() + 1e-8)
    with torch.no_grad():
        return model(), torch.stack(hist)


def exact(case, seed):
    kind = case["kind"]
    if kind == "cost":
        return _exact_cost(case, seed)
    if kind == "batch":
        got = [_exact_system(m, 3) for m in _batch_meshes(case, seed)]
        return torch.cat([v for v, _ in got]), torch.cat([r for _, r in got]), None
    m = _mesh(case["n"], case["mix"], seed, dofs=_dofs(case), nh=case.get("nh", 0.0))
    if kind == "subscale":
        return _exact_subscale(m, _dofs(case)), None
    vals, rhs = _exact_system(m, _dofs(case), case.get("nh", 0.0) > 0, bool(case.get("residual", False)))
    return {"vals": vals, "rhs": rhs} if kind == "build" else (vals, rhs, None)
