"""Vertex buckets on connectivity that is no lattice: neighbours hardly ever
shared between a vertex's elements, so that rows keep far more distinct values
than a window takes, by the hundred in one bucket of the large size.  Exact
integer work with one answer: bit equality with the oracle, or with the
sort-based pipeline that the oracle tests cover."""
import numpy as np
import pytest

from paper_1604_04689_amd import meshgen as mg

SORTED = {"node_sort": 3}  # the element-rows pipeline, asked for by name
NPE = np.array([3, 4, 8, 4, 6, 5])
EDGES = np.array([3, 6, 12, 4, 9, 8])
KEYS = ("node row_ptr", "node cols", "elem row_ptr", "elem cols")


def spread(etype, n_vert, degree, seed):
    """Every vertex in exactly `degree` elements of shuffled ids."""
    rng = np.random.default_rng(seed)
    ids = np.concatenate([rng.permutation(n_vert) for _ in range(degree)])
    return ids[:ids.size // NPE[etype] * NPE[etype]].reshape(-1, NPE[etype]).astype(np.int32)


def scattered(etype, n_vert, n_elem, seed):
    return mg.random_mesh(n_elem, n_vert, etype, seed).conn


def _single(conn, etype, n_vert, options=None):
    import torch

    import paper_1604_04689_amd as nb
    c = torch.as_tensor(np.ascontiguousarray(conn)).to("cuda:0")
    both = nb.neighbors(c, etype, n_vert, options=options)
    alone = nb.node_neighbors(c, etype, n_vert, options=options), nb.elem_neighbors(c, etype, n_vert, options=options)
    return [[x.cpu().numpy() for r in rel for x in r] for rel in (both, alone)]


def _equal(got, want, what):
    for g, w, k in zip(got, want, KEYS):
        assert g.shape == w.shape and np.array_equal(g, w), (what, k)


@pytest.mark.gpu
@pytest.mark.parametrize("etype,n_vert,conn", [
    (1, 131072, lambda: spread(1, 131072, 20, 1)),             # 256 such rows to a bucket of 256 vertices
    (0, 131072, lambda: spread(0, 131072, 27, 2)),             # the same with records of two neighbours
    (1, 1_000_000, lambda: scattered(1, 1_000_000, 3_000_000, 3)),  # some of a bucket's rows, 256 now and then
], ids=["tets_256_rows", "triangles_256_rows", "tets_some_rows"])
def test_rows_of_many_distinct_values_vs_oracle(oracle_mod, etype, n_vert, conn):
    conn = conn()
    print(f"[irregular] etype={etype} n_elem={len(conn)} n_vert={n_vert}", flush=True)
    want = [*oracle_mod.node_neighbors(conn, etype, n_vert), *oracle_mod.elem_neighbors(conn, etype, n_vert)]
    for got in _single(conn, etype, n_vert):
        _equal(got, want, (etype, n_vert))


@pytest.mark.gpu
@pytest.mark.parametrize("etype,n_vert,n_elem", [(0, 200_000, 1_200_000), (1, 131_072, 655_360), (1, 400_000, 900_000),
                                                 (2, 200_000, 300_000), (3, 300_000, 1_200_000), (4, 250_000, 500_000),
                                                 (5, 200_000, 500_000)])
def test_scattered_connectivity_vs_sort(etype, n_vert, n_elem):
    conn = scattered(etype, n_vert, n_elem, n_elem)
    print(f"[irregular] scattered etype={etype} n_elem={n_elem} n_vert={n_vert}", flush=True)
    for got, want in zip(_single(conn, etype, n_vert), _single(conn, etype, n_vert, SORTED)):
        _equal(got, want, (etype, n_elem))


@pytest.mark.gpu
def test_batch_of_scattered_meshes_vs_sort():
    """Meshes of 512 vertices in 21 tetrahedra each (two buckets of 256 such
    rows), and larger scattered ones of the other types."""
    import torch

    import paper_1604_04689_amd as nb
    meshes = [(1, 512, spread(1, 512, 21, i)) for i in range(240)]
    meshes += [(et, 30_000, scattered(et, 30_000, 10 * 30_000 // int(NPE[et]), et)) for et in range(6)]
    print(f"[irregular] batch of {len(meshes)}, {sum(c.size for _, _, c in meshes)} slots", flush=True)
    conn = torch.as_tensor(np.concatenate([c.ravel() for _, _, c in meshes])).to("cuda:0")
    got = {}
    for options in (None, SORTED):
        for kind in ("both", "node"):
            b = nb.BatchBuild(kind, [(len(c), et, nv) for et, nv, c in meshes], "cuda:0", options=options)
            b.launch(conn)
            r = b.result()
            got[options is None, kind] = [x.cpu().numpy() for rel in (r if kind == "both" else (r,)) for x in rel]
    for kind in ("both", "node"):
        _equal(got[True, kind], got[False, kind], kind)


def _mixed(conn, types, n_vert, options):
    import torch

    import paper_1604_04689_amd as nb
    off = np.concatenate([[0], np.cumsum(NPE[types])]).astype(np.int32)
    b = nb.MixedBuild(len(types), len(conn), int(2 * EDGES[types].sum()), n_vert, "cuda:0", options=options)
    b.launch(*[torch.as_tensor(x).to("cuda:0") for x in (conn, off, types)])
    return [x.cpu().numpy() for rel in b.result() for x in rel]


@pytest.mark.gpu
@pytest.mark.parametrize("n_vert,n_elem", [(131_072, 350_000), (400_000, 900_000)])
def test_scattered_mixed_mesh_vs_sort(n_vert, n_elem):
    m = mg.random_mixed(n_elem, n_vert, seed=n_elem)
    conn, types = np.asarray(m.conn).ravel(), np.asarray(m.etypes)
    print(f"[irregular] mixed n_elem={n_elem} n_vert={n_vert}", flush=True)
    _equal(_mixed(conn, types, n_vert, None), _mixed(conn, types, n_vert, SORTED), n_elem)


@pytest.mark.gpu
@pytest.mark.parametrize("n,buckets", [(170, True), (180, True), (200, False)], ids=["large_tiles", "small_tiles", "sorts"])
def test_too_many_buckets_for_small_tiles_are_left_to_the_sorts(n, buckets):
    """Wedges of an n x n x n / 2 lattice's counts: which pipeline they take
    shows in the names of its launches (the ids do not matter to the choice)."""
    import torch

    import paper_1604_04689_amd as nb
    from paper_1604_04689_amd import binding
    n_elem, n_vert = 2 * (n - 1) ** 2 * (n // 2), n * n * (n // 2 + 1)
    print(f"[irregular] wedges n_elem={n_elem} n_vert={n_vert}", flush=True)
    first = torch.arange(n_elem, dtype=torch.int32, device="cuda:0") % (n_vert // 6) * 6
    conn = first[:, None] + torch.arange(6, dtype=torch.int32, device="cuda:0")
    b = nb.NeighborBuild("both", n_elem, 4, n_vert, "cuda:0")
    binding.timing_read()
    binding.timing_enable(True)
    try:
        b.launch(conn)
        torch.cuda.synchronize()
    finally:
        binding.timing_enable(False)
    names = set(binding.timing_read())
    (rp, cols), (erp, ecols) = b.result()
    assert ("bucket_rows" in names) == buckets, names
    used = n_vert // 6 * 6
    assert cols.numel() == 3 * used and ecols.numel() == 6 * n_elem and int(erp[used]) == 6 * n_elem
