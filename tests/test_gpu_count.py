"""The counting search (histograms without the distance matrix: qc_potential
on a handle whose distances were never asked for, and the batch) against the
oracle's breadth-first search: every launch shape at the edges of its range
(one node below and above the most a shape holds), hub rows and their units,
leaves, isolated edges and nodes, rows beyond 8 entries that are no hub's,
directed graphs, the longest distances and one too many; and the same search writing the
distance rows (qc_distances from the second search on), whose leaves and
unconnected nodes get theirs in a pass of their own. Histograms and distances
are whole numbers: equal, no tolerance."""
import numpy as np
import pytest

import oracle
from paper_2305_14641_amd import graphgen as gg

pytestmark = pytest.mark.gpu


def ring_with_chords(n: int, seed: int):
    """A ring plus a random perfect matching: every node has 2 or 3 edges, so
    every node is searched and holds a position."""
    rng = np.random.default_rng(seed)
    p = rng.permutation(n)
    i = np.arange(n)
    u = np.concatenate([i, p[0:n - n % 2:2]])
    v = np.concatenate([(i + 1) % n, p[1:n:2][:n // 2]])
    rp, c = gg.csr_from_edges(n, u, v)
    return gg.Graph(n, rp, c, np.zeros(n, np.int32), name=f"ring+chords({n})")


def counted(g, directed=False):
    """Histograms of g from the counting search, at their row length."""
    import torch
    from paper_2305_14641_amd import qc
    print(f"[gpu] counting search {g.name} n={g.n} nnz={g.nnz}", flush=True)
    G = qc.Graph.from_graph(g, directed=directed)
    G.potential([1.0])
    first = G.histograms().cpu().numpy()
    dmax = G.info()["dmax"]
    b = qc.Batch([G], [1.0, 2.0], hipgraph=False)   # a second search, sources re-sorted
    out = b.outputs()
    b.run(*out)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(G.histograms().cpu().numpy(), first)
    b.close()
    G.close()
    return first, dmax


def check(g, directed=False, sample=None):
    hist, dmax = counted(g, directed)
    if sample is None:
        rows = np.arange(g.n, dtype=np.int32)
    else:
        rows = np.unique(np.concatenate([np.random.default_rng(g.n).choice(g.n, sample, replace=False),
                                         [0, g.n - 1]])).astype(np.int32)
    dist, far = oracle.bfs_rows(g.n, g.row_ptr, g.col, rows)
    want = np.zeros((len(rows), hist.shape[1]), np.int64)
    for r in range(len(rows)):
        d = dist[r]
        c = np.bincount(d[d >= 0], minlength=hist.shape[1])
        assert len(c) == hist.shape[1]
        want[r] = c
    np.testing.assert_array_equal(hist[rows], want)
    assert dmax == far if sample is None else dmax >= far
    assert hist.shape[1] == (32 if dmax < 32 else 64 if dmax < 64 else 128)


SMALL = [gg.path_graph(1), gg.path_graph(2), gg.empty_graph(70), gg.star_graph(1), gg.star_graph(2),
         gg.star_graph(5000), gg.twin_leaves(60, 40), gg.complete_graph(40), gg.complete_graph(300),
         gg.barbell_graph(33), gg.path_graph(34), gg.path_graph(127),
         gg.disjoint_union(gg.path_graph(2), gg.star_graph(70), gg.empty_graph(3), gg.complete_graph(12),
                           gg.path_graph(3), gg.path_graph(66)),
         gg.random_graph(1500, 0.02, 3), gg.config1(), gg.dcsbm(3000, [0.5, 0.3, 0.2], 9.0, seed=4)]


@pytest.mark.parametrize("g", SMALL, ids=lambda g: g.name)
def test_counts_small(g):
    check(g)


@pytest.mark.parametrize("n", [33, 4095, 4096, 8191, 8192, 10239, 12287, 14336, 16384, 18431, 18432, 20479,
                               24576, 28672, 32768, 36863, 36864, 40960, 45056, 49152, 57344, 65535, 65536])
def test_counts_at_shape_edges(n):
    check(ring_with_chords(n, n), sample=20)


@pytest.mark.parametrize("n,deg,seed", [(17000, 7.5, 3), (43000, 8.0, 4)])
def test_counts_hubs_and_leaves(n, deg, seed):
    check(gg.dcsbm(n, [0.5, 0.3, 0.2], deg, seed=seed), sample=40)


@pytest.mark.parametrize("g", [gg.dcsbm_directed(3000, [0.6, 0.4], 2.0, seed=5), gg.random_digraph(400, 0.03, 6)],
                         ids=lambda g: g.name)
def test_counts_directed(g):
    check(g, directed=True)


@pytest.mark.parametrize("directed", [False, True])
def test_counts_distance_limit(directed):
    """A path of 127 nodes reaches distance 126; one of 128 is refused."""
    from paper_2305_14641_amd import qc
    for n, ok in ((127, True), (128, False)):
        i = np.arange(n - 1)
        rp, c = (gg.csr_from_arcs if directed else gg.csr_from_edges)(n, i, i + 1)
        G = qc.Graph(n, rp, c, directed=directed)
        if ok:
            G.potential([1.0])
            h = G.histograms().cpu().numpy()
            assert G.info()["dmax"] == 126 and h[0, 126] == 1 and h.shape[1] == 128
        else:
            with pytest.raises(qc.QCError) as e:
                G.potential([1.0])
            assert e.value.status == qc.QC_E_OVERFLOW
        G.close()


def circulant(n: int, step: int):
    """A ring with chords of one length: every node alike, largest distance
    about step / 2 + n / (2 step)."""
    i = np.arange(n)
    rp, c = gg.csr_from_edges(n, np.concatenate([i, i]), np.concatenate([(i + 1) % n, (i + step) % n]))
    return gg.Graph(n, rp, c, np.zeros(n, np.int32), name=f"circulant({n},{step})")


def check_rows(g, sample=None, directed=False, weights=None):
    """Distance rows of g (every row, or sampled ones and their columns when
    undirected) and histograms of the same search."""
    import torch
    from paper_2305_14641_amd import qc
    print(f"[gpu] distance rows {g.name} n={g.n} nnz={g.nnz}", flush=True)
    G = qc.Graph.from_graph(g, directed=directed, weights=weights)
    d = torch.full((g.n, g.n), 77, dtype=torch.int8, device="cuda")
    dmax = G.distances(d)
    d.fill_(77)
    assert G.distances(d) == dmax
    rows = np.arange(g.n, dtype=np.int32)
    if sample is not None:
        rows = np.unique(np.concatenate([np.random.default_rng(g.n).choice(g.n, sample, replace=False),
                                         [0, g.n - 1]])).astype(np.int32)
    if weights is None:
        want, _ = oracle.bfs_rows(g.n, g.row_ptr, g.col, rows)
    else:
        want = oracle.weighted_distances(g.n, g.row_ptr, g.col, weights)[0][rows]
    idx = torch.as_tensor(rows.astype(np.int64), device="cuda")
    np.testing.assert_array_equal(d[idx].cpu().numpy(), want)
    if not directed and sample is not None:
        np.testing.assert_array_equal(d[:, idx].cpu().numpy().T, want)
    hist = G.histograms().cpu().numpy()
    for r, w in zip(rows, want):
        np.testing.assert_array_equal(hist[r], np.bincount(w[w >= 0], minlength=hist.shape[1]))
    # rows the library owns have their own stride
    G.distances()
    np.testing.assert_array_equal(G.histograms().cpu().numpy(), hist)
    G.close()


@pytest.mark.parametrize("g", SMALL + [circulant(250, 7), circulant(1001, 30)], ids=lambda g: g.name)
def test_rows_small(g):
    check_rows(g)


@pytest.mark.parametrize("n", [33, 4095, 4096, 8191, 8192, 12287, 12288, 16383, 16384, 20479, 20480, 24575, 24577,
                               28672, 32767, 32768])
def test_rows_at_shape_edges(n):
    check_rows(ring_with_chords(n, n), sample=16)


@pytest.mark.parametrize("n,step", [(4095, 90), (8191, 100), (8192, 100), (9000, 100)])
def test_rows_many_levels(n, step):
    """7 planes, up to two quads of positions per thread (above: the matrix
    search)."""
    check_rows(circulant(n, step), sample=16)


@pytest.mark.parametrize("n,deg,seed", [(12500, 4.0, 5), (19999, 4.5, 6), (19001, 8.0, 7), (27000, 5.0, 8)])
def test_rows_hubs_and_leaves(n, deg, seed):
    check_rows(gg.dcsbm(n, [0.5, 0.3, 0.2], deg, seed=seed), sample=24)


@pytest.mark.parametrize("n,deg", [(700, 2.0), (9973, 3.0)])
def test_rows_directed(n, deg):
    check_rows(gg.dcsbm_directed(n, [0.6, 0.4], deg, seed=9), sample=40, directed=True)


@pytest.mark.parametrize("n,most,directed", [(300, 5, False), (1500, 4, False), (1500, 3, True)])
def test_rows_weighted(n, most, directed):
    g = (gg.dcsbm_directed if directed else gg.dcsbm)(n, [0.6, 0.4], 3.0, seed=11)
    check_rows(g, directed=directed, weights=gg.edge_weights(g, most, seed=3, directed=directed))
