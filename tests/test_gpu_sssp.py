"""Shortest paths under real weights at the edges of every launch shape of the
search, against the oracle's binary32 Dijkstra bit for bit: node counts at and
one above the most a shape holds (and that leave sources over in the last
workgroup), in-lists around the length that is cut into parts, nodes without
in-edges, directed graphs, searches that stay in either kind of round, and a
padded row stride. Lengths are sums in a fixed order: equal, no tolerance."""
import numpy as np
import pytest

import oracle
from paper_2305_14641_amd import graphgen as gg

pytestmark = pytest.mark.gpu


def grid(k):
    i = np.arange(k * k)
    r, c = i // k, i % k
    rp, col = gg.csr_from_edges(k * k, np.concatenate([i[c < k - 1], i[r < k - 1]]),
                                np.concatenate([i[c < k - 1] + 1, i[r < k - 1] + k]))
    return gg.Graph(k * k, rp, col, np.zeros(k * k, np.int32), name=f"grid{k}")


def stars(sizes):
    """Disjoint stars: in-lists of exactly these lengths."""
    return gg.disjoint_union(*[gg.star_graph(k) for k in sizes])


GRAPHS = ([(gg.dcsbm(n, [0.5, 0.3, 0.2], 4.0, seed=n), False)
           for n in (63, 64, 65, 1023, 1024, 1025, 2432, 2433, 4928, 4929, 9920, 9921, 19840, 19841, 32767)]
          + [(gg.dcsbm_directed(n, [0.6, 0.4], 3.0, seed=n), True) for n in (1024, 2431, 4925, 9919, 19839, 32768)]
          + [(stars([1, 31, 32, 33, 34, 63, 64, 65, 66, 96, 97, 1500]), False), (gg.complete_graph(33), False),
             (gg.complete_graph(34), False), (gg.complete_graph(700), False), (gg.path_graph(1500), False),
             (gg.empty_graph(130), False), (grid(50), False), (grid(120), False)])


@pytest.mark.parametrize("g,directed", GRAPHS, ids=lambda x: f"{x.name}" if hasattr(x, "name") else str(x))
def test_lengths(g, directed):
    import torch
    from paper_2305_14641_amd import qc
    print(f"[gpu] lengths {g.name} n={g.n} nnz={g.nnz}", flush=True)
    w = gg.real_edge_weights(g, seed=g.n, directed=directed)
    ld = g.n + g.n % 3
    out = torch.full((g.n, ld), -1.0, dtype=torch.float32, device="cuda")
    d = qc.distances_real(g.n, g.row_ptr, g.col, w, directed=directed, out=out)
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([np.random.default_rng(g.n).choice(g.n, min(g.n, 12), replace=False),
                                     [0, g.n - 1]])).astype(np.int32)
    idx = torch.as_tensor(rows.astype(np.int64), device="cuda")
    np.testing.assert_array_equal(d[idx, :g.n].cpu().numpy(), oracle.real_rows(g.n, g.row_ptr, g.col, w, rows))
    assert bool((d[:, :g.n].diagonal() == 0).all())
    if ld > g.n:
        assert bool((out[:, g.n:] == -1.0).all())
