"""The counting search (histograms without the distance matrix: qc_potential
on a handle whose distances were never asked for, and the batch) against the
oracle's breadth-first search: every launch shape at the edges of its range
(one node below and above the most a shape holds), hub rows and their units,
leaves, isolated edges and nodes, rows beyond 8 entries that are no hub's,
directed graphs, the longest distances and one too many. Histograms are whole
numbers: equal, no tolerance."""
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
