"""The vertex-bucket pipeline (the library's choice for a mesh of one element
type) at the sizes where it can go wrong: tile and bucket edges, rows of every
class (each network width, rows beyond the networks, rows beyond the LDS),
repeated ids, unused vertices, both bucket sizes.  Exact integer work with one
answer: bit equality, with the oracle or, for the large meshes, with the
sort-based pipeline that the oracle tests cover."""
import numpy as np
import pytest

from paper_1604_04689_amd import binding
from paper_1604_04689_amd import meshgen as mg

ETYPES = list(range(6))
SORTED = {"node_sort": 3}  # the element-rows pipeline, asked for by name


@pytest.mark.parametrize("etype", ETYPES)
def test_choice_does_not_change_sizes(etype):
    """Which pipeline a call takes shows in its time only: workspace and
    capacities are those of the sort-based pipeline at every size and shape
    of mesh (few vertices, many, more than the buckets take)."""
    for n in (0, 1, 255, 4096, 100_000, 1_500_000, 20_000_000):
        for v in (0, 1, 2, n // 40 + 1, n // 6 + 1, 2 * n + 1, 2**29 + 5):
            assert binding.query("both", n, etype, v) == binding.query("both", n, etype, v, SORTED)
            assert binding.query_node(n, etype, v) == binding.query_node(n, etype, v, SORTED)
            assert binding.query_elem(n, etype, v) == binding.query_elem(n, etype, v, SORTED)


def _gpu(conn, etype, n_vert, options=None):
    import torch

    import paper_1604_04689_amd as nb
    c = torch.as_tensor(np.ascontiguousarray(conn)).to("cuda:0")
    (nr, nc), (er, ec) = nb.neighbors(c, etype, n_vert, options=options)
    n1, e1 = nb.node_neighbors(c, etype, n_vert, options=options), nb.elem_neighbors(c, etype, n_vert, options=options)
    return [x.cpu().numpy() for x in (nr, nc, er, ec, *n1, *e1)]


def _check(got, node, elem, what):
    want = [*node, *elem, *node, *elem]
    for g, w, k in zip(got, want, ("node row_ptr", "node cols", "elem row_ptr", "elem cols") * 2):
        assert g.shape == w.shape and np.array_equal(g, w), f"{what}: {k} differs"


def _vs_oracle(oracle_mod, conn, etype, n_vert, what):
    print(f"[buckets] {what} n_elem={len(conn)} n_vert={n_vert}", flush=True)
    _check(_gpu(conn, etype, n_vert), oracle_mod.node_neighbors(conn, etype, n_vert),
           oracle_mod.elem_neighbors(conn, etype, n_vert), what)


def fan(m, at, hub):
    """m triangles around vertex `hub`, rim vertices at .. at + m - 1."""
    i = np.arange(m)
    return np.stack([np.full(m, hub), at + i, at + (i + 1) % m], 1)


@pytest.fixture(scope="module")
def oracle_mod():
    import oracle
    return oracle


@pytest.mark.gpu
@pytest.mark.parametrize("etype", ETYPES)
def test_tile_edges_vs_oracle(oracle_mod, etype):
    """Element counts around the small tile (256) and a bucket's least
    records; random ids, so elements repeat vertices and vertices go unused."""
    for n in (1, 2, 255, 256, 257, 1023, 2049):
        for per in (1, 4):
            m = mg.random_mesh(n, max(2, mg.NODES_PER_ELEM[etype] * n // per), etype, 100 * n + per)
            _vs_oracle(oracle_mod, m.conn, etype, m.n_vert, f"random {per}")


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [(3, 4, 5, 8, 9), (12, 13, 16, 17, 24), (31, 32, 33, 64, 65), (200, 600, 1500),
                                  (3071, 3073), (9000,)])
def test_row_classes_vs_oracle(oracle_mod, rows):
    """Fans of every row class on top of a grid, with and without a repeated
    id in the mesh."""
    m = mg.tri_grid(90, "coin", 7)
    parts, at = [m.conn], m.n_vert
    for k in rows:
        parts.append(fan(k, at + 1, at))
        at += k + 1
    conn = np.concatenate(parts).astype(np.int32)
    rng = np.random.default_rng(3)
    label = rng.permutation(at).astype(np.int32)
    conn = label[conn][rng.permutation(len(conn))]
    _vs_oracle(oracle_mod, conn, 0, at, f"fans {rows}")
    conn[5, 2] = conn[5, 0]
    conn[900, 1] = conn[900, 0] = conn[900, 2]
    _vs_oracle(oracle_mod, conn, 0, at, f"fans {rows}, repeated ids")


@pytest.mark.gpu
@pytest.mark.parametrize("etype,mesh", [(0, lambda: mg.tri_grid(1100, "coin", 1)), (1, lambda: mg.kuhn_tet_grid(50, 2)),
                                        (2, lambda: mg.hex_grid(75, 3)), (3, lambda: mg.quad_grid(1000, 4)),
                                        (4, lambda: mg.wedge_grid(100, 50, 5)), (5, lambda: mg.pyramid_grid(48, 6))])
def test_large_buckets_vs_sort(etype, mesh):
    """Meshes of large buckets and tiles, as generated, in lattice order (each
    tile in few buckets), and with a few elements that repeat an id."""
    m = mesh()
    inv = np.argsort(m.perm).astype(np.int32)
    lattice = inv[m.conn[np.argsort(m.elem_order)]]
    odd = m.conn.copy()
    odd[::5000, 1] = odd[::5000, 0]
    for what, conn in (("shuffled", m.conn), ("lattice order", lattice), ("repeated ids", odd)):
        print(f"[buckets] {m.name} {what}", flush=True)
        w = _gpu(conn, etype, m.n_vert, SORTED)
        _check(_gpu(conn, etype, m.n_vert), w[0:2], w[2:4], f"{m.name} {what}")


@pytest.mark.gpu
def test_uneven_vertices_vs_sort():
    """All elements in the first tenth of the vertices: every used bucket
    holds ten times what was planned."""
    m = mg.tri_grid(500, "coin", 9)
    w = _gpu(m.conn, 0, 10 * m.n_vert, SORTED)
    _check(_gpu(m.conn, 0, 10 * m.n_vert), w[0:2], w[2:4], "uneven")


@pytest.mark.gpu
@pytest.mark.parametrize("etype,mesh", [(0, lambda: mg.tri_grid(60, "coin", 1)), (1, lambda: mg.kuhn_tet_grid(9, 2))])
def test_errors_and_clean_call_after(oracle_mod, etype, mesh):
    """Ids out of range, a capacity too small by one, then a clean call on the
    same workspace; unaligned connectivity."""
    import torch

    import paper_1604_04689_amd as nb
    m = mesh()
    good = torch.as_tensor(m.conn).to("cuda:0")
    for bad_id in (m.n_vert, -1, 2**31 - 1):
        bad = good.clone()
        bad[7, 1] = bad_id
        b = nb.NeighborBuild("both", m.n_elem, etype, m.n_vert, "cuda:0")
        b.launch(bad)
        with pytest.raises(nb.MeshError) as e:
            b.result()
        assert e.value.status == nb.Status.INDEX_RANGE
        b.launch(good)
        b.result()
    want = oracle_mod.node_neighbors(m.conn, etype, m.n_vert)
    small = nb.NeighborBuild("node", m.n_elem, etype, m.n_vert, "cuda:0", cols_capacity=len(want[1]) - 1)
    small.launch(good)
    with pytest.raises(nb.MeshError) as e:
        small.result()
    assert e.value.status == nb.Status.CAPACITY
    odd = torch.empty(good.numel() + 1, dtype=torch.int32, device="cuda:0")[1:]
    odd.copy_(good.reshape(-1))
    r, c = nb.node_neighbors(odd, etype, m.n_vert)
    assert np.array_equal(r.cpu().numpy(), want[0]) and np.array_equal(c.cpu().numpy(), want[1])
