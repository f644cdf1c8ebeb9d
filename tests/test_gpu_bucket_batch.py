"""The vertex buckets of a batch (the library's choice for a batch of meshes
of a useful size) where they can go wrong: tile and bucket edges, meshes of
every type and record form side by side, empty meshes, more meshes than the
planning block takes at once, overfull buckets and long rows, repeated ids,
both bucket sizes, gapped connectivity, inconsistent records.  Exact integer
work with one answer: bit equality with the sort-based pipeline, which the
oracle tests cover, and with the oracle."""
import numpy as np
import pytest

from paper_1604_04689_amd import binding
from paper_1604_04689_amd import meshgen as mg

SORTED = {"node_sort": 3}  # the element-rows pipeline, asked for by name
NPE = {0: 3, 1: 4, 2: 8, 3: 4, 4: 6, 5: 5}


def rand_mesh(rng, etype, n_elem, n_vert, used=None):
    """(conn, etype, n_vert): random ids (some elements repeat one)."""
    c = rng.integers(0, used or n_vert, size=(n_elem, NPE[etype])) if n_elem else np.zeros((0, NPE[etype]))
    return c.astype(np.int32), etype, n_vert


def grid(m):
    return m.conn, m.etype, m.n_vert


def fan(m, n_vert, hub):
    i = np.arange(m)
    rim = np.delete(np.arange(m + 1), hub)
    return np.stack([np.full(m, hub), rim[i], rim[(i + 1) % m]], 1).astype(np.int32), 0, n_vert


def _cases():
    rng = np.random.default_rng(5)
    small = [rand_mesh(rng, et, n, max(1, n // 3)) for n in (1, 255, 256, 257, 511, 513, 1025) for et in range(6)]
    yield "small_all_types", small
    empty = [rand_mesh(rng, 0, 0, 0), rand_mesh(rng, 1, 0, 5000), rand_mesh(rng, 2, 700, 300), rand_mesh(rng, 3, 0, 1),
             rand_mesh(rng, 4, 900, 1), rand_mesh(rng, 5, 800, 40000, 90), rand_mesh(rng, 1, 0, 0)]
    yield "empty_and_unused", empty
    yield "one_mesh", [grid(mg.kuhn_tet_grid(9, 3))]
    yield "many_meshes", [grid(mg.tri_grid(int(n), "coin", int(n))) for n in rng.integers(12, 30, 2100)]
    # an uneven mesh (buckets of far more records than they hold), hubs and their long rows
    i = np.arange(20000) % 500
    dense = np.stack([i, (i * 7 + 1) % 500, (i * 13 + 2) % 500, (i * 3 + 5) % 500], 1).astype(np.int32)
    yield "overfull", [grid(mg.tri_grid(70, "main", 1)), (dense, 1, 4000), fan(9000, 9001, 17), fan(300, 301, 300),
                       grid(mg.hex_grid(12, 4))]
    yield "large", [grid(mg.kuhn_tet_grid(30, 6)), grid(mg.tri_grid(500, "coin", 3)), rand_mesh(rng, 5, 70001, 30000),
                    grid(mg.hex_grid(25, 5)), rand_mesh(rng, 4, 1, 7), grid(mg.tri_grid(333, "main", 9)),
                    fan(40000, 40001, 5), rand_mesh(rng, 3, 60001, 59000)]


CASES = dict(_cases())


def test_choice_does_not_change_sizes():
    """Which pipeline a batch takes shows in its time only."""
    import ctypes
    lib = binding.lib()
    for n_mesh, pairs, slots, vert, most in ((1, 0, 0, 0, 0), (3, 6000, 3000, 900, 500), (64, 5_000_000, 2_000_000, 400_000, 9000),
                                             (512, 300_000_000, 130_000_000, 12_000_000, 250_000), (2, 8, 4, 9, 9),
                                             (4, 60_000_000, 24_000_000, 4_000_000, 3_900_000)):
        got = []
        for o in (None, SORTED):
            opts = binding.make_options(o)
            for name, n_out in (("mesh_batch_neighbors_query", 3), ("mesh_batch_node_neighbors_query", 2)):
                out = [ctypes.c_size_t(0), ctypes.c_int64(0), ctypes.c_int64(0)][:n_out]
                st = getattr(lib, name)(n_mesh, pairs, slots, vert, most, ctypes.byref(opts), *[ctypes.byref(x) for x in out])
                got.append((st, [x.value for x in out]))
        assert got[:2] == got[2:]


def _build(meshes, kind, options, conn_offs=None, conn=None):
    import torch

    import paper_1604_04689_amd as nb
    desc = [(len(c), et, nv) for c, et, nv in meshes]
    b = nb.BatchBuild(kind, desc, "cuda:0", conn_offs=conn_offs, options=options)
    if conn is None:
        conn = np.concatenate([c.ravel() for c, _, _ in meshes]).astype(np.int32)
    b.launch(torch.as_tensor(conn).to("cuda:0"))
    got = b.result()
    pairs = got if kind == "both" else (got,)
    return b, [x.cpu().numpy() for p in pairs for x in p]


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(CASES))
def test_batch_buckets_equal_sorts(name):
    meshes = CASES[name]
    print(f"[batch buckets] {name}: {len(meshes)} meshes, {sum(c.size for c, _, _ in meshes)} slots", flush=True)
    want = _build(meshes, "both", SORTED)[1]
    got = _build(meshes, "both", None)[1]
    node = _build(meshes, "node", None)[1]
    for g, w, k in zip(got + node, want + want[:2], ("node row_ptr", "node cols", "elem row_ptr", "elem cols") * 2):
        assert g.shape == w.shape and np.array_equal(g, w), (name, k)


@pytest.mark.gpu
def test_batch_buckets_equal_oracle():
    import oracle
    meshes = CASES["small_all_types"]
    nr, nc, er, ec = _build(meshes, "both", None)[1]
    v0 = 0
    for c, et, nv in meshes:
        for rp, cols, want in ((nr, nc, oracle.node_neighbors(c, et, nv)), (er, ec, oracle.elem_neighbors(c, et, nv))):
            r = rp[v0:v0 + nv + 1]
            assert np.array_equal(r - r[0], want[0]) and np.array_equal(cols[r[0]:r[-1]], want[1]), (et, len(c))
        v0 += nv


@pytest.mark.gpu
def test_batch_buckets_gapped_connectivity():
    """Meshes anywhere in the connectivity, in any order."""
    meshes = CASES["large"]
    offs, at = [0] * len(meshes), 5
    for i in reversed(range(len(meshes))):
        offs[i] = at
        at += meshes[i][0].size + 3
    conn = np.full(at, -7, np.int32)
    for o, (c, _, _) in zip(offs, meshes):
        conn[o:o + c.size] = c.ravel()
    want = _build(meshes, "both", SORTED)[1]
    got = _build(meshes, "both", None, conn_offs=offs, conn=conn)[1]
    for g, w in zip(got, want):
        assert np.array_equal(g, w)


@pytest.mark.gpu
def test_batch_buckets_leave_out_bad_records():
    """A record that reaches outside the batch is reported; the others' rows
    are right, its own are empty."""
    import torch

    import paper_1604_04689_amd as nb
    meshes = [grid(mg.tri_grid(40, "main", 1)), grid(mg.kuhn_tet_grid(6, 2)), grid(mg.hex_grid(8, 3))]
    want = _build(meshes, "both", None)[1]
    conn = torch.as_tensor(np.concatenate([c.ravel() for c, _, _ in meshes]).astype(np.int32)).to("cuda:0")
    nv = [m[2] for m in meshes]
    for field, value in (("etype", 17), ("n_elem", 1 << 40), ("n_vert", -4), ("slot_off", -1)):
        b = nb.BatchBuild("both", [(len(c), et, v) for c, et, v in meshes], "cuda:0")
        seg = b.seg_host.copy()
        seg[1][field] = value
        b.segs[:seg.nbytes].copy_(torch.as_tensor(seg.view("u1")).to("cuda:0"))
        b.launch(conn)
        with pytest.raises(nb.MeshError) as e:
            b.result()
        assert e.value.status == nb.Status.INDEX_RANGE, field
        for rp, cols, w_rp, w_cols in ((b.row_ptr, b.cols, *want[:2]), (b.elem_row_ptr, b.elem_cols, *want[2:])):
            rp, cols = rp.cpu().numpy(), cols.cpu().numpy()
            deg, w_deg = np.diff(rp), np.diff(w_rp)
            a, z = nv[0], nv[0] + nv[1]
            assert rp[0] == 0 and np.array_equal(deg[:a], w_deg[:a]) and np.array_equal(deg[z:], w_deg[z:]), field
            assert not deg[a:z].any(), field
            keep = np.concatenate([w_cols[:w_rp[a]], w_cols[w_rp[z]:]])
            assert np.array_equal(cols[:len(keep)], keep), field


@pytest.mark.gpu
def test_batch_buckets_need_no_pair_offsets():
    """Only pipelines that sort pairs read pair_off: as in the sort of the
    elements, a batch whose records leave it out is built, and one of more
    pairs than the batch is said to have is not."""
    import torch

    import paper_1604_04689_amd as nb
    meshes = [grid(mg.tri_grid(40, "main", 1)), grid(mg.kuhn_tet_grid(6, 2)), grid(mg.hex_grid(8, 3))] * 5
    conn = torch.as_tensor(np.concatenate([c.ravel() for c, _, _ in meshes]).astype(np.int32)).to("cuda:0")
    want = _build(meshes, "both", SORTED)[1]
    for options in (None, SORTED):
        b = nb.BatchBuild("both", [(len(c), et, v) for c, et, v in meshes], "cuda:0", options=options)
        seg = b.seg_host.copy()
        seg["pair_off"] = 0
        b.segs[:seg.nbytes].copy_(torch.as_tensor(seg.view("u1")).to("cuda:0"))
        b.launch(conn)
        got = [x.cpu().numpy() for rel in b.result() for x in rel]
        for g, w in zip(got, want):
            assert np.array_equal(g, w), options
    b = nb.BatchBuild("both", [(len(c), et, v) for c, et, v in meshes], "cuda:0")
    b.totals["pairs"] -= 2
    b.launch(conn)
    with pytest.raises(nb.MeshError) as e:
        b.result()
    assert e.value.status == nb.Status.INDEX_RANGE


@pytest.mark.gpu
def test_batch_buckets_take_any_type_of_an_empty_mesh():
    import torch

    import paper_1604_04689_amd as nb
    empty = np.zeros((0, 3), np.int32)
    meshes = [(empty, 0, 7), grid(mg.tri_grid(40, "main", 1)), (empty, 0, 900), grid(mg.hex_grid(8, 3)), (empty, 0, 0)]
    conn = torch.as_tensor(np.concatenate([c.ravel() for c, _, _ in meshes]).astype(np.int32)).to("cuda:0")
    want = _build(meshes, "both", SORTED)[1]
    for options in (SORTED, None):
        b = nb.BatchBuild("both", [(len(c), et, v) for c, et, v in meshes], "cuda:0", options=options)
        seg = b.seg_host.copy()
        seg["etype"][[0, 2, 4]] = (99, -5, 6)
        b.segs[:seg.nbytes].copy_(torch.as_tensor(seg.view("u1")).to("cuda:0"))
        b.launch(conn)
        got = [x.cpu().numpy() for rel in b.result() for x in rel]
        for g, w in zip(got, want):
            assert np.array_equal(g, w), options
