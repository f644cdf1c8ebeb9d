"""The vertex buckets of a mesh of several element types (the library's choice
where no node algorithm, tile shape or digit width is named) where they can go
wrong: tile edges, both bucket sizes, overfull buckets and long rows, repeated
ids, ill-formed elements.  Exact integer work with one answer: bit equality
with the sort-based pipeline, which the oracle tests cover, and the oracle."""
import numpy as np
import pytest

from paper_1604_04689_amd import meshgen as mg

pytestmark = pytest.mark.gpu

SORTED = {"node_sort": 3}  # the element-rows pipeline, asked for by name
NPE = np.array([3, 4, 8, 4, 6, 5])
EDGES = np.array([3, 6, 12, 4, 9, 8])


def _build(conn, off, types, n_vert, options, n_pairs=None):
    import torch

    import paper_1604_04689_amd as nb
    dev = "cuda:0"
    n_pairs = int(2 * EDGES[types].sum()) if n_pairs is None else n_pairs
    b = nb.MixedBuild(len(types), len(conn), n_pairs, n_vert, dev, options=options)
    b.launch(torch.as_tensor(np.ascontiguousarray(conn, np.int32)).to(dev),
             torch.as_tensor(np.ascontiguousarray(off, np.int32)).to(dev),
             torch.as_tensor(np.ascontiguousarray(types, np.uint8)).to(dev))
    return b


def _result(*args):
    (nr, nc), (er, ec) = _build(*args).result()
    return [x.cpu().numpy() for x in (nr, nc, er, ec)]


def _offsets(types):
    return np.concatenate([[0], np.cumsum(NPE[types])])


def _check(conn, types, n_vert, what):
    print(f"[mixed buckets] {what}: {len(types)} elements, {n_vert} vertices", flush=True)
    off = _offsets(types)
    want = _result(conn, off, types, n_vert, SORTED)
    got = _result(conn, off, types, n_vert, None)
    for g, w, k in zip(got, want, ("node row_ptr", "node cols", "elem row_ptr", "elem cols")):
        assert g.shape == w.shape and np.array_equal(g, w), (what, k)
    return got


@pytest.mark.parametrize("n", [1, 319, 320, 321, 2559, 2560, 2561, 30000])
def test_tile_edges(n):
    import oracle
    m = mg.random_mixed(n, max(1, n // 2), seed=n)  # (some elements repeat an id)
    got = _check(np.asarray(m.conn).ravel(), np.asarray(m.etypes), m.n_vert, "random")
    node = oracle.mixed_node_neighbors(m.conn, m.etypes, m.n_vert)
    elem = oracle.mixed_elem_neighbors(m.conn, m.etypes, m.n_vert)
    for g, w in zip(got, [*node, *elem]):
        assert np.array_equal(g, w)


@pytest.mark.parametrize("relabel", [True, False], ids=["shuffled", "kinds_side_by_side"])
def test_large_buckets_and_tiles(relabel):
    m = mg.hybrid_grid(52, seed=4, relabel=relabel)
    _check(np.asarray(m.conn).ravel(), np.asarray(m.etypes), m.n_vert, "hybrid")


def test_uneven():
    """A hub of 20,000 elements, and 30,000 elements on 400 of 60,000 vertices."""
    rng = np.random.default_rng(3)
    types = rng.integers(0, 6, 50000).astype(np.uint8)
    off = _offsets(types)
    conn = rng.integers(0, 400, off[-1])
    hub = rng.integers(400, 60000, off[-1])
    first = np.zeros(off[-1], bool)
    first[off[:-1]] = True
    late = np.repeat(np.arange(50000) >= 30000, NPE[types])
    conn[late] = hub[late]
    conn[late & first] = 59999
    _check(conn, types, 60000, "uneven")


def test_ill_formed_elements_are_left_out():
    """Unknown types and offsets that disagree with the type are reported; the
    other elements' rows are right."""
    import paper_1604_04689_amd as nb
    m = mg.hybrid_grid(9, seed=2)
    types, conn = np.asarray(m.etypes).copy(), np.asarray(m.conn).ravel()
    off = _offsets(types)
    n_pairs = int(2 * EDGES[types].sum())
    ill = np.arange(0, len(types), 7)
    keep = np.setdiff1d(np.arange(len(types)), ill)
    kept = np.concatenate([conn[off[e]:off[e + 1]] for e in keep])
    nr, nc, er, ec = _result(kept, _offsets(types[keep]), types[keep], m.n_vert, SORTED)
    types[ill[::2]] = 99
    types[ill[1::2]] = np.where(types[ill[1::2]] == 0, 1, 0)  # a type of another size
    b = _build(conn, off, types, m.n_vert, None, n_pairs)
    with pytest.raises(nb.MeshError) as e:
        b.result()
    assert e.value.status == nb.Status.INDEX_RANGE
    assert np.array_equal(b.row_ptr.cpu().numpy(), nr) and np.array_equal(b.cols.cpu().numpy()[:nr[-1]], nc)
    assert np.array_equal(b.elem_row_ptr.cpu().numpy(), er)
    assert np.array_equal(b.elem_cols.cpu().numpy()[:er[-1]], keep[ec])


def test_overlapping_elements_stay_in_bounds():
    """Offsets that go back and forth ask for more (vertex, element) pairs than
    there are ids: reported, and nothing outside the buffers is touched (the
    element outputs' guard words)."""
    import torch

    import paper_1604_04689_amd as nb
    n = 20001
    off = np.where(np.arange(n + 1) % 2 == 0, 0, 8)
    types = np.full(n, 2, np.uint8)
    conn = np.arange(n * 2, dtype=np.int32) % 9000
    b = _build(conn, off, types, 9000, None, 24 * n)
    torch.cuda.synchronize()
    with pytest.raises(nb.MeshError) as e:
        b.result()
    assert e.value.status == nb.Status.INDEX_RANGE
