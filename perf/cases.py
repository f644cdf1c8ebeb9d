"""Neighbor builds as programs that use this library run them, from the
smallest mesh, where launches and host work count, to the largest batch.

Meshes are the lattices of the package's generators (triangle, quadrilateral,
Kuhn tetrahedra, hexahedra, wedges, pyramids, hybrids of four types), built on
the GPU.  Vertex labels and the element order are random permutations
("shuffled", as the benchmark has them: no locality at all), or permuted
within a sliding window ("local", as a mesh generator or a renumbering leaves
them).  All outputs are int32 CSR arrays with one right answer.
"""
import math

import torch

import paper_1604_04689_amd as nb
from paper_1604_04689_amd import meshgen

TRI3, TET4, HEX8, QUAD4, WEDGE6, PYRAMID5 = 0, 1, 2, 3, 4, 5
NPE = {TRI3: 3, TET4: 4, HEX8: 8, QUAD4: 4, WEDGE6: 6, PYRAMID5: 5}
EDGES = {
    TRI3: ((0, 1), (1, 2), (2, 0)),
    TET4: ((0, 1), (0, 2), (0, 3), (1, 2), (1, 3), (2, 3)),
    HEX8: ((0, 1), (1, 2), (2, 3), (3, 0), (4, 5), (5, 6), (6, 7), (7, 4), (0, 4), (1, 5), (2, 6), (3, 7)),
    QUAD4: ((0, 1), (1, 2), (2, 3), (3, 0)),
    WEDGE6: ((0, 1), (1, 2), (2, 0), (3, 4), (4, 5), (5, 3), (0, 3), (1, 4), (2, 5)),
    PYRAMID5: ((0, 1), (1, 2), (2, 3), (3, 0), (0, 4), (1, 4), (2, 4), (3, 4)),
}
ETYPE = {"tri": TRI3, "quad": QUAD4, "tet": TET4, "hex": HEX8, "wedge": WEDGE6, "pyramid": PYRAMID5}
BATCH_SEED = meshgen.BASE_SEED + 3  # the size draw of the 512-mesh batch
WINDOW = 256  # how far a "local" label lies from its lattice place
BYTES = 4  # int32 throughout


def listed():
    return [
        # a program that rebuilds the neighbors of a small surface again and
        # again on kept buffers: launches and host work only
        mesh("tri64_both", "tri", 64, "both", options="tuned"),
        # the same through a captured graph, as latency-bound loops run it
        mesh("tri64_graph", "tri", 64, "both", call="graph", options="tuned"),
        # one call on a small volume mesh met once: workspace, outputs, the
        # build, and the sizes read back
        mesh("tet12_oneshot", "tet", 12, "both", call="oneshot"),
        # smoothing and fairing want the node relation alone: a surface of
        # about half a million triangles, sizes off every power of two
        mesh("tri513_node", "tri", 513, "node"),
        # gathering element data at nodes wants the element relation alone
        mesh("tet37_elem", "tet", 37, "elem"),
        # half a million hexahedra: the widest elements
        mesh("hex80_both", "hex", 80, "both"),
        # a renumbered surface of 2.1 M triangles: labels with locality
        mesh("tri1025_local", "tri", 1025, "both", order="local"),
        # hexahedra, wedges, pyramids and tetrahedra in one mesh
        mesh("hybrid48_mixed", "hybrid", 48, "both", call="mixed"),
        # what one step of the server builds: a batch of 64 queued meshes
        batch("batch64_both", 64),
        # the large surface and the large volume
        mesh("tri2048_both", "tri", 2048, "both", options="tuned"),
        mesh("tet96_both", "tet", 96, "both", options="tuned"),
        # the whole batch of 512 meshes of three types in one call
        batch("batch512_both", 512),
    ]


def mesh(name, shape, size, relation, call="build", order="shuffled", options="default"):
    c = {"call": call, "shape": shape, "size": size, "relation": relation, "order": order, "options": options}
    return dict(c, name=name) if name else c


def batch(name, n_mesh, spec_seed=BATCH_SEED, options="tuned"):
    c = {"call": "batch", "n_mesh": n_mesh, "spec_seed": spec_seed, "relation": "both", "options": options}
    return dict(c, name=name) if name else c


# connectivity slots (ids) of a lattice of one cell or vertex squared, and the power it grows with
SLOTS = {"tri": (6, 2), "quad": (4, 2), "tet": (24, 3), "hex": (8, 3), "wedge": (3, 3), "pyramid": (30, 3),
         "hybrid": (18.5, 3)}


def draw(rng):
    call = rng.choices(("build", "graph", "oneshot", "mixed", "batch"), (12, 1, 3, 2, 4))[0]
    if call == "batch":
        n = int(round(math.exp(rng.uniform(math.log(8), math.log(256)))))
        return batch(None, n, spec_seed=rng.randrange(1 << 30))
    most = {"build": 2.5e7, "graph": 3e5, "oneshot": 3e6, "mixed": 4e6}[call]
    shape = "hybrid" if call == "mixed" else rng.choice(("tri", "tri", "tet", "tet", "hex", "quad", "wedge", "pyramid"))
    a, p = SLOTS[shape]
    slots = math.exp(rng.uniform(math.log(1.5e4), math.log(most)))
    size = max(4, int(round((slots / a) ** (1 / p))))
    relation = "both" if call in ("oneshot", "mixed") else rng.choice(("both", "both", "node", "elem"))
    order = rng.choice(("shuffled", "shuffled", "local"))
    options = "default" if call in ("oneshot", "mixed") else rng.choice(("default", "tuned"))
    return mesh(None, shape, size, relation, call, order, options)


# ---- meshes ------------------------------------------------------------------

def _axes(*n, device):
    g = torch.meshgrid(*[torch.arange(k, device=device) for k in n], indexing="ij")
    return [x.reshape(-1) for x in g]


HEX_CORNERS = ((0, 0, 0), (1, 0, 0), (1, 1, 0), (0, 1, 0), (0, 0, 1), (1, 0, 1), (1, 1, 1), (0, 1, 1))
FACES = (((0, 0, 0), (0, 1, 0), (1, 1, 0), (1, 0, 0)), ((0, 0, 1), (1, 0, 1), (1, 1, 1), (0, 1, 1)),
         ((0, 0, 0), (1, 0, 0), (1, 0, 1), (0, 0, 1)), ((0, 1, 0), (0, 1, 1), (1, 1, 1), (1, 1, 0)),
         ((0, 0, 0), (0, 0, 1), (0, 1, 1), (0, 1, 0)), ((1, 0, 0), (1, 1, 0), (1, 1, 1), (1, 0, 1)))
KUHN = []
for _o in ((0, 1, 2), (0, 2, 1), (1, 0, 2), (1, 2, 0), (2, 0, 1), (2, 1, 0)):
    _p, _path = [0, 0, 0], [(0, 0, 0)]
    for _ax in _o:
        _p[_ax] = 1
        _path.append(tuple(_p))
    KUHN.append(tuple(_path))
CELL_WEDGES = tuple(tuple((a, b, z) for z in (0, 1) for a, b in t)
                    for t in (((0, 0), (1, 0), (1, 1)), ((0, 0), (1, 1), (0, 1))))


def _cells(m, device):
    x, y, z = _axes(m, m, m, device=device)
    s = m + 1
    return lambda c: ((x + c[0]) * s + (y + c[1])) * s + (z + c[2])


def _lattice(shape, n, gen, device):
    """(connectivity [elements, nodes], vertices) before relabelling."""
    if shape in ("tri", "quad"):
        i, j = _axes(n - 1, n - 1, device=device)
        a, b, c, d = i * n + j, i * n + j + 1, (i + 1) * n + j, (i + 1) * n + j + 1
        if shape == "quad":
            return torch.stack([a, c, d, b], 1), n * n
        flip = torch.randint(0, 2, a.shape, generator=gen, device=device).bool()[:, None]
        t1 = torch.where(flip, torch.stack([a, b, c], 1), torch.stack([a, b, d], 1))
        t2 = torch.where(flip, torch.stack([b, d, c], 1), torch.stack([a, d, c], 1))
        return torch.stack([t1, t2], 1).reshape(-1, 3), n * n
    if shape == "wedge":
        layers = max(1, n // 2)
        i, j, k = _axes(n - 1, n - 1, layers, device=device)
        vid = lambda a, b, c: ((i + a) * n + (j + b)) * (layers + 1) + k + c  # noqa: E731
        w = [torch.stack([vid(a, b, c) for c in (0, 1) for a, b in t], 1)
             for t in (((0, 0), (0, 1), (1, 1)), ((0, 0), (1, 1), (1, 0)))]
        return torch.stack(w, 1).reshape(-1, 6), n * n * (layers + 1)
    at = _cells(n, device)
    s = n + 1
    if shape == "hex":
        return torch.stack([at(c) for c in HEX_CORNERS], 1), s ** 3
    if shape == "tet":
        return torch.stack([torch.stack([at(c) for c in t], 1) for t in KUHN], 1).reshape(-1, 4), s ** 3
    centre = s ** 3 + torch.arange(n ** 3, device=device)
    p = [torch.stack([at(c) for c in f] + [centre], 1) for f in FACES]
    return torch.stack(p, 1).reshape(-1, 5), s ** 3 + n ** 3


def _order(n, order, gen, device):
    if order == "local":
        at = torch.arange(n, device=device, dtype=torch.float64)
        return torch.argsort(at + WINDOW * torch.rand(n, generator=gen, device=device, dtype=torch.float64))
    return torch.randperm(n, generator=gen, device=device)


def _one_mesh(shape, n, order, gen, device):
    conn, nv = _lattice(shape, n, gen, device)
    label = torch.empty(nv, dtype=torch.int64, device=device)
    label[_order(nv, order, gen, device)] = torch.arange(nv, device=device)
    conn = label[conn][_order(conn.shape[0], order, gen, device)]
    return conn.to(torch.int32).contiguous(), nv


def _hybrid(m, order, gen, device):
    """(ids, types, vertices): every cell one hexahedron, two wedges, six
    pyramids or six tetrahedra (a draw that goes with the size, so that a
    size has one count of edges), the elements in a random order."""
    at = _cells(m, device)
    s = m + 1
    kind = torch.randint(0, 4, (m ** 3,), generator=_gen(m, "cpu")).to(device)
    centre = s ** 3 + torch.arange(m ** 3, device=device)
    groups = [(HEX8, [torch.stack([at(c) for c in HEX_CORNERS], 1)], 0),
              (WEDGE6, [torch.stack([at(c) for c in w], 1) for w in CELL_WEDGES], 1),
              (PYRAMID5, [torch.stack([at(c) for c in f] + [centre], 1) for f in FACES], 2),
              (TET4, [torch.stack([at(c) for c in t], 1) for t in KUHN], 3)]
    ids, types = [], []
    for et, parts, k in groups:
        e = torch.stack(parts, 1)[kind == k].reshape(-1, NPE[et])
        ids.append(torch.nn.functional.pad(e, (0, 8 - NPE[et]), value=-1))
        types.append(torch.full((e.shape[0],), et, dtype=torch.uint8, device=device))
    ids, types = torch.cat(ids), torch.cat(types)
    nv = s ** 3 + m ** 3
    label = torch.full((nv + 1,), -1, dtype=torch.int64, device=device)
    label[_order(nv, order, gen, device)] = torch.arange(nv, device=device)
    o = torch.randperm(ids.shape[0], generator=gen, device=device)
    ids, types = label[ids[o]], types[o]
    return ids[ids >= 0].to(torch.int32).contiguous(), types.contiguous(), nv


def _edge_count(shape, n):
    """Undirected edges of a lattice: half the entries of the node relation."""
    s = n + 1
    if shape == "tri":
        return 2 * n * (n - 1) + (n - 1) ** 2
    if shape == "quad":
        return 2 * n * (n - 1)
    if shape == "wedge":
        layers = max(1, n // 2)
        return (2 * n * (n - 1) + (n - 1) ** 2) * (layers + 1) + n * n * layers
    axis = 3 * n * s * s
    return axis + {"hex": 0, "tet": 3 * n * n * s + n ** 3, "pyramid": 8 * n ** 3}[shape]


def _counts(shape, n):
    """(elements, vertices) of a lattice."""
    if shape in ("tri", "quad"):
        return (2 if shape == "tri" else 1) * (n - 1) ** 2, n * n
    if shape == "wedge":
        layers = max(1, n // 2)
        return 2 * (n - 1) ** 2 * layers, n * n * (layers + 1)
    return ({"hex": 1, "tet": 6, "pyramid": 6}[shape] * n ** 3,
            (n + 1) ** 3 + (n ** 3 if shape == "pyramid" else 0))


def _specs(case):
    """[(shape, size)] of a batch: the generators' size and type draw."""
    name = {v: k for k, v in ETYPE.items()}
    return [(name[s.etype], s.size) for s in meshgen.batch_specs(case["n_mesh"], case["spec_seed"])]


def _gen(seed, device):
    return torch.Generator(device=device).manual_seed(int(seed) * 2654435761 % (1 << 62) + 1)


def _inputs(case, seed, device):
    gen = _gen(seed, device)
    if case["call"] == "mixed":
        return _hybrid(case["size"], case["order"], gen, device)
    if case["call"] == "batch":
        return [_one_mesh(shape, n, "shuffled", gen, device) for shape, n in _specs(case)]
    return _one_mesh(case["shape"], case["size"], case["order"], gen, device)


# ---- the calls ---------------------------------------------------------------

def prepare(case, seed):
    device = torch.device("cuda", torch.cuda.current_device())
    options = "tuned" if case["options"] == "tuned" else None
    call, rel = case["call"], case["relation"]
    s = {"call": call, "relation": rel}
    if call == "mixed":
        conn, types, nv = _inputs(case, seed, device)
        off, n_ids, n_pairs = nb.mixed_layout(types.cpu().numpy())
        off = torch.as_tensor(off).to(device)
        s.update(args=(conn, off, types), build=nb.MixedBuild(types.numel(), n_ids, n_pairs, nv, device))
        return s
    if call == "batch":
        meshes = _inputs(case, seed, device)
        specs = _specs(case)
        b = nb.BatchBuild(rel, [(c.shape[0], ETYPE[sh], nv) for (c, nv), (sh, _) in zip(meshes, specs)], device,
                          options=options)
        s.update(args=(torch.cat([c.reshape(-1) for c, _ in meshes]),), build=b,
                 node_nnz=sum(2 * _edge_count(sh, n) for sh, n in specs), elem_nnz=sum(c.numel() for c, _ in meshes))
        return s
    conn, nv = _inputs(case, seed, device)
    et = ETYPE[case["shape"]]
    s.update(args=(conn,), etype=et, n_vert=nv, elem_nnz=conn.numel(),
             node_nnz=2 * _edge_count(case["shape"], case["size"]))
    if call == "oneshot":
        return s
    s["build"] = nb.NeighborBuild(rel, conn.shape[0], et, nv, device, options=options)
    if call == "graph":
        s["graph"] = s["build"].capture(conn)
    return s


def run(s):
    if s["call"] == "oneshot":
        return nb.neighbors(s["args"][0], s["etype"], s["n_vert"])
    b = s["build"]
    if s["call"] == "mixed":  # a program that does not know the sizes reads them back
        b.launch(*s["args"])
        return b.result()
    if s["call"] == "graph":
        s["graph"].launch()
    else:
        b.launch(*s["args"])
    # lattices: the program knows how long its rows are in all, and waits for nothing
    if s["relation"] == "both":
        return (b.row_ptr, b.cols[:s["node_nnz"]]), (b.elem_row_ptr, b.elem_cols[:s["elem_nnz"]])
    return b.row_ptr, b.cols[:s[s["relation"] + "_nnz"]]


def work(case):
    """Connectivity in, the relations' row starts and columns out."""
    if case["call"] == "mixed":
        m = case["size"]
        ids = 18.5 * m ** 3  # a quarter of the cells of each kind: 8, 12, 30 and 24 ids
        nv = (m + 1) ** 3 + m ** 3
        # axis edges, and what the kinds add: the wedges' diagonals, the spokes, the Kuhn diagonals
        nnz = 2 * (3 * m * (m + 1) ** 2 + m ** 3 * (2 + 8 + 5.5) / 4)
        return {"bytes": BYTES * (2 * ids + nnz + 2 * (nv + 1) + ids / 5), "flops": 0}
    total = 0
    specs = _specs(case) if case["call"] == "batch" else [(case["shape"], case["size"])]
    for shape, n in specs:
        ne, nv = _counts(shape, n)
        slots = ne * NPE[ETYPE[shape]]
        total += slots
        if case["relation"] in ("node", "both"):
            total += nv + 1 + 2 * _edge_count(shape, n)
        if case["relation"] in ("elem", "both"):
            total += nv + 1 + slots
    return {"bytes": BYTES * total, "flops": 0}


# ---- the answers, in 64-bit integers -------------------------------------------

def _csr(key, n_rows, n_cols):
    """CSR of the distinct (row, column) keys row * n_cols + column."""
    key = torch.unique(key)
    row = torch.div(key, n_cols, rounding_mode="floor")
    rp = torch.zeros(n_rows + 1, dtype=torch.int64, device=key.device)
    rp[1:] = torch.cumsum(torch.bincount(row, minlength=n_rows), 0)
    return rp, key - row * n_cols


def _node_keys(conn, et, nv):
    c = conn.to(torch.int64)
    out = []
    for a, b in EDGES[et]:
        out += [c[:, a] * nv + c[:, b], c[:, b] * nv + c[:, a]]
    return torch.cat(out)


def _both(parts, nv, n_elem):
    """parts: (type, connectivity, element ids)."""
    node = _csr(torch.cat([_node_keys(c, et, nv) for et, c, _ in parts]), nv, nv)
    elem = _csr(torch.cat([(c.to(torch.int64) * n_elem + e[:, None]).reshape(-1) for _, c, e in parts]), nv, n_elem)
    return node, elem


def exact(case, seed):
    device = torch.device("cuda", torch.cuda.current_device())
    if case["call"] == "mixed":
        ids, types, nv = _inputs(case, seed, device)
        npe = torch.tensor([NPE[t] for t in range(6)], device=device)[types.long()]
        off = torch.cumsum(npe, 0) - npe
        parts = []
        for et in (HEX8, WEDGE6, PYRAMID5, TET4):
            e = torch.nonzero(types == et).reshape(-1)
            parts.append((et, ids[off[e][:, None] + torch.arange(NPE[et], device=device)], e))
        return _both(parts, nv, types.numel())
    if case["call"] == "batch":
        nrp, ncol, erp, ecol, nb0, eb0 = [], [], [], [], 0, 0
        for (c, nv), (shape, _) in zip(_inputs(case, seed, device), _specs(case)):
            (r, k), (er, ek) = _both([(ETYPE[shape], c, torch.arange(c.shape[0], device=device))], nv, c.shape[0])
            nrp.append(r[:-1] + nb0), erp.append(er[:-1] + eb0)
            ncol.append(k), ecol.append(ek)
            nb0, eb0 = nb0 + k.numel(), eb0 + ek.numel()
        end = lambda v, n: torch.cat(v + [torch.tensor([n], device=device)])  # noqa: E731
        return (end(nrp, nb0), torch.cat(ncol)), (end(erp, eb0), torch.cat(ecol))
    conn, nv = _inputs(case, seed, device)
    both = _both([(ETYPE[case["shape"]], conn, torch.arange(conn.shape[0], device=device))], nv, conn.shape[0])
    return both if case["relation"] == "both" else both[0 if case["relation"] == "node" else 1]
