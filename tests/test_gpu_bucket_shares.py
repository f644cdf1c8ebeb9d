"""Vertex buckets with far more records than a block's LDS holds: several
blocks share such a bucket, rows beyond the LDS are cut into windows of ids,
and nobody's wait for the rows before its own may fail while those are being
made.  Exact integer work with one answer: bit equality with the sort-based
pipeline, which the oracle tests cover, or with the oracle."""
import numpy as np
import pytest

SORTED = {"node_sort": 3}  # the element-rows pipeline, asked for by name
NPE = np.array([3, 4, 8, 4, 6, 5])
EDGES = np.array([3, 6, 12, 4, 9, 8])
KEYS = ("node row_ptr", "node cols", "elem row_ptr", "elem cols")


def concentrated(etype, n_elem, n_vert, power, seed, repeats):
    """Ids n_vert * x^power, x uniform: rows of every length, the longest side
    by side.  Without `repeats` no element has an id twice."""
    rng = np.random.default_rng(seed)
    c = (n_vert * rng.random((n_elem, NPE[etype])) ** power).astype(np.int32)
    if not repeats:
        s = np.sort(c, 1)
        c = c[(s[:, 1:] != s[:, :-1]).all(1)]
    return np.ascontiguousarray(c)


def hubs(n_vert, first, count, size, rest, seed):
    """`count` vertices from label `first` on in `size` triangles each, and
    `rest` triangles over all vertices."""
    rng = np.random.default_rng(seed)
    rim = rng.integers(first + count, n_vert, count * size) if first == 0 else rng.integers(0, first, count * size)
    c = np.stack([np.repeat(np.arange(first, first + count), size), rim, np.roll(rim, 1)], 1)
    c = np.concatenate([c, rng.integers(0, n_vert, (rest, 3))])
    c = c[(c[:, 1] != c[:, 2]) & (c[:, 0] != c[:, 1]) & (c[:, 0] != c[:, 2])]
    return c[rng.permutation(len(c))].astype(np.int32)


def _builds(conn, etype, n_vert, options=None):
    import torch

    import paper_1604_04689_amd as nb
    c = torch.as_tensor(conn).to("cuda:0")
    both = nb.neighbors(c, etype, n_vert, options=options)
    node = nb.node_neighbors(c, etype, n_vert, options=options)
    elem = nb.elem_neighbors(c, etype, n_vert, options=options)
    return [*both[0], *both[1]], [*node, *elem]


def _equal(got, want, what):
    import torch
    for g, w, k in zip(got, want, KEYS):
        assert g.shape == w.shape and torch.equal(g, w), (what, k)


def _check(conn, etype, n_vert, what):
    print(f"[shares] {what} etype={etype} n_elem={len(conn)} n_vert={n_vert}", flush=True)
    want, _ = _builds(conn, etype, n_vert, SORTED)
    for got in _builds(conn, etype, n_vert):
        _equal(got, want, what)


@pytest.mark.gpu
@pytest.mark.parametrize("repeats", [False, True], ids=["distinct", "repeats"])
@pytest.mark.parametrize("etype,n_elem,n_vert,power", [
    (0, 3000, 1000, 5), (0, 60_000, 30_000, 3), (0, 900_000, 500_000, 2.5), (1, 300_000, 200_000, 3),
    (2, 40_000, 30_000, 3), (2, 200_000, 300_000, 2), (3, 250_000, 100_000, 4), (4, 90_000, 60_000, 2.5),
    (5, 150_000, 90_000, 3)])
def test_concentrated_elements(etype, n_elem, n_vert, power, repeats):
    _check(concentrated(etype, n_elem, n_vert, power, n_elem, repeats), etype, n_vert, f"concentrated {power}")


@pytest.mark.gpu
@pytest.mark.parametrize("n_elem,n_vert,power", [(574, 583, 6), (995, 1352, 8), (25_521, 94_310, 5), (64_941, 10_213, 2)])
def test_no_room_for_shares(n_elem, n_vert, power):
    """Pyramid meshes whose workspace (that of the sorts) just holds the records:
    one block does an overfull bucket."""
    _check(concentrated(5, n_elem, n_vert, power, n_elem, True), 5, n_vert, "no room for shares")


@pytest.mark.gpu
@pytest.mark.parametrize("n_vert,first,count,size", [
    (1_200_000, 0, 1, 60_000),          # one row over several windows of ids, the first bucket
    (1_200_000, 1_199_997, 3, 30_000),  # the last bucket ends with such rows
    (300_000, 0, 60, 3000), (40_000, 39_000, 1000, 40), (700_000, 350_000, 7, 9000)])
def test_hubs(n_vert, first, count, size):
    _check(hubs(n_vert, first, count, size, 200_000, size), 0, n_vert, f"{count} hubs of {size}")


@pytest.mark.gpu
@pytest.mark.parametrize("n_vert,first,count,size", [(1_200_000, 0, 1, 60_000), (300_000, 0, 60, 3000),
                                                     (700_000, 699_993, 7, 9000)])
def test_hubs_with_repeated_ids(n_vert, first, count, size):
    """The shares' element rows are then counted before they have a place."""
    conn = hubs(n_vert, first, count, size, 200_000, size + 1)
    conn[::97, 1] = conn[::97, 0]
    conn[5::1001, 2] = conn[5::1001, 1]
    _check(conn, 0, n_vert, f"{count} hubs of {size}, repeated ids")


@pytest.mark.gpu
def test_hubs_vs_oracle(oracle_mod):
    conn = hubs(50_000, 20_000, 40, 2500, 30_000, 4)
    want = [*oracle_mod.node_neighbors(conn, 0, 50_000), *oracle_mod.elem_neighbors(conn, 0, 50_000)]
    for got in _builds(conn, 0, 50_000):
        for g, w, k in zip(got, want, KEYS):
            assert np.array_equal(g.cpu().numpy(), w), k


@pytest.mark.gpu
def test_a_long_bucket_does_not_fail_the_others():
    """250 vertices side by side in 24,000 triangles each: one bucket has all
    6 million of them, and every other waits for its rows."""
    import torch

    import paper_1604_04689_amd as nb
    n_vert, count, size = 3_000_000, 250, 24_000
    gen = torch.Generator(device="cuda:0").manual_seed(8)
    hub = torch.arange(count * size, device="cuda:0") // size
    rim = torch.randint(count, n_vert, (count * size,), generator=gen, device="cuda:0")
    c = torch.stack([hub, rim, torch.roll(rim, 1)], 1)
    c = c[torch.randperm(count * size, generator=gen, device="cuda:0")].to(torch.int32).contiguous()
    print(f"[shares] {count} hubs of {size}", flush=True)
    want, got = (nb.neighbors(c, 0, n_vert, options=o) for o in (SORTED, None))
    _equal([*got[0], *got[1]], [*want[0], *want[1]], "long bucket")


@pytest.mark.gpu
def test_capacity_too_small_and_a_clean_call_after():
    import torch

    import paper_1604_04689_amd as nb
    conn = hubs(100_000, 0, 20, 5000, 50_000, 6)
    c = torch.as_tensor(conn).to("cuda:0")
    want = nb.node_neighbors(c, 0, 100_000, options=SORTED)
    b = nb.NeighborBuild("node", len(conn), 0, 100_000, "cuda:0", cols_capacity=want[1].numel() - 1)
    b.launch(c)
    with pytest.raises(nb.MeshError) as e:
        b.result()
    assert e.value.status == nb.Status.CAPACITY
    b = nb.NeighborBuild("node", len(conn), 0, 100_000, "cuda:0", cols_capacity=want[1].numel())
    for _ in range(2):
        b.launch(c)
        _equal(b.result(), want, "exact capacity")


@pytest.mark.gpu
def test_batch_with_shared_buckets():
    import torch

    import paper_1604_04689_amd as nb
    for scale in (1, 8):  # small and large buckets
        meshes = [(0, 5000, hubs(5000, 2000, 30, 800, 100, 1)), (1, 20_000 * scale, concentrated(1, 30_000 * scale, 20_000 * scale, 3, 2, True)),
                  (5, 9000, concentrated(5, 9000 * scale, 9000, 2.5, 3, False)), (3, 100, np.zeros((0, 4), np.int32)),
                  (2, 30_000, concentrated(2, 20_000 * scale, 30_000, 4, 4, False)), (0, 700_000, hubs(700_000, 0, 2, 40_000, 20_000, 5))]
        print(f"[shares] batch x{scale}, {sum(c.size for _, _, c in meshes)} slots", flush=True)
        conn = torch.as_tensor(np.concatenate([c.ravel() for _, _, c in meshes])).to("cuda:0")
        got = []
        for options in (SORTED, None):
            for kind in ("both", "node"):
                b = nb.BatchBuild(kind, [(len(c), et, nv) for et, nv, c in meshes], "cuda:0", options=options)
                b.launch(conn)
                r = b.result()
                got.append([x for rel in (r if kind == "both" else (r,)) for x in rel])
        _equal(got[2], got[0], "both")
        _equal(got[3], got[1], "node")


@pytest.mark.gpu
@pytest.mark.parametrize("n_elem,n_vert,power", [(20_000, 9000, 4), (400_000, 200_000, 3)])
def test_mixed_mesh_with_shared_buckets(n_elem, n_vert, power):
    import torch

    import paper_1604_04689_amd as nb
    rng = np.random.default_rng(n_elem)
    types = rng.integers(0, 6, n_elem).astype(np.uint8)
    off = np.concatenate([[0], np.cumsum(NPE[types])]).astype(np.int32)
    conn = (n_vert * rng.random(off[-1]) ** power).astype(np.int32)
    print(f"[shares] mixed n_elem={n_elem} n_vert={n_vert}", flush=True)
    got = []
    for options in (SORTED, None):
        b = nb.MixedBuild(n_elem, len(conn), int(2 * EDGES[types].sum()), n_vert, "cuda:0", options=options)
        b.launch(*[torch.as_tensor(x).to("cuda:0") for x in (conn, off, types)])
        r = b.result()
        got.append([*r[0], *r[1]])
    _equal(got[1], got[0], "mixed")


def _stretch(m, times):
    """A mesh over `times` as many vertices as its elements use, those first."""
    return m.conn, m.etype, times * m.n_vert


@pytest.mark.gpu
@pytest.mark.parametrize("mesh", [
    # records of a used bucket, for what its block holds: both relations, and the element relation alone
    lambda mg: _stretch(mg.kuhn_tet_grid(50, 2), 3),        # 8800 for 5952, 17,600 for 14,848
    lambda mg: _stretch(mg.tri_grid(700, "coin", 3), 10),   # 8200 for 7680
    lambda mg: _stretch(mg.tri_grid(120, "main", 4), 9),    # small buckets: 3800 for 3072
    lambda mg: _stretch(mg.pyramid_grid(20, 5), 6),
    lambda mg: _stretch(mg.hex_grid(60, 6), 8),
], ids=["tets", "triangles", "few_triangles", "pyramids", "hexahedra"])
def test_elements_on_the_first_vertices_only(mesh):
    """The corners of a quadratic mesh numbered first, or a part of a mesh in
    the numbering of the whole: the used buckets hold more than was planned."""
    from paper_1604_04689_amd import meshgen as mg
    conn, etype, n_vert = mesh(mg)
    _check(conn, etype, n_vert, "first vertices")


@pytest.mark.gpu
@pytest.mark.parametrize("n", [501, 20001])
def test_overlapping_elements_touch_nothing_outside(n):
    """Offsets that go back and forth ask for more (vertex, element) pairs than
    there are ids: reported, and the words around the outputs and behind the
    workspace stay as they were."""
    import torch

    import paper_1604_04689_amd as nb
    off = np.where(np.arange(n + 1) % 2 == 0, 0, 8).astype(np.int32)
    conn = (np.arange(n * 2) % 9000).astype(np.int32)
    b = nb.MixedBuild(n, len(conn), 24 * n, 9000, "cuda:0")
    guard, outs = 1024, {}
    for k in ("row_ptr", "cols", "elem_row_ptr", "elem_cols"):
        t = getattr(b, k)
        outs[k] = torch.full((t.numel() + 2 * guard,), 7, dtype=torch.int32, device="cuda:0")
        setattr(b, k, outs[k][guard:-guard])
    raw = torch.full((b.ws_bytes + 8192,), 90, dtype=torch.uint8, device="cuda:0")
    pad = (-raw.data_ptr()) % 256
    b.workspace = raw[pad:pad + b.ws_bytes]
    print(f"[shares] overlapping n_elem={n}", flush=True)
    b.launch(*[torch.as_tensor(x).to("cuda:0") for x in (conn, off, np.full(n, 2, np.uint8))])
    with pytest.raises(nb.MeshError) as e:
        b.result()
    assert e.value.status == nb.Status.INDEX_RANGE
    for k, t in outs.items():
        assert (t[:guard] == 7).all() and (t[-guard:] == 7).all(), k
    assert (raw[:pad] == 90).all() and (raw[pad + b.ws_bytes:] == 90).all()


@pytest.mark.gpu
def test_graph_replays_and_two_streams():
    """Replays of a captured build over an even mesh, an uneven one and the even
    one again (shares come and go), with an eager build of an uneven mesh on
    another stream beside each."""
    import torch

    import paper_1604_04689_amd as nb
    n_vert, size = 150_000, 40_000
    uneven = torch.as_tensor(hubs(n_vert, 0, 30, 3000, 2 * size, 1)[:3 * size]).to("cuda:0")
    rng = np.random.default_rng(2)
    even = np.stack([rng.permutation(n_vert)[:3 * size] for _ in range(3)], 1)
    even = even[(even[:, 0] != even[:, 1]) & (even[:, 0] != even[:, 2]) & (even[:, 1] != even[:, 2])]
    n = min(len(even), len(uneven))
    inputs = [torch.as_tensor(even[:n].astype(np.int32)).to("cuda:0"), uneven[:n].contiguous()]
    want = []
    for c in inputs:
        node, elem = nb.neighbors(c, 0, n_vert, options=SORTED)
        want.append([*node, *elem])
    conn = inputs[0].clone()
    captured, eager = (nb.NeighborBuild("both", n, 0, n_vert, "cuda:0") for _ in range(2))
    graph = captured.capture(conn)
    side = torch.cuda.Stream()
    for k in (0, 1, 0, 1, 1, 0):
        print(f"[shares] replay over input {k}", flush=True)
        conn.copy_(inputs[k])
        torch.cuda.synchronize()
        graph.launch()
        eager.launch(inputs[1], side)
        node, elem = captured.result()
        _equal([*node, *elem], want[k], ("replay", k))
        node, elem = eager.result(side)
        torch.cuda.synchronize()
        _equal([*node, *elem], want[1], "beside")
        captured.row_ptr.zero_(), captured.cols.zero_(), captured.elem_cols.zero_()
    graph.destroy()
