"""Integer edge weights where the search takes narrower batches of sources to
occupy more of the chip, on both sides of the rule: the sizes at which the
batches of 16 and of 8 sources just fit one per CU and one node more, against
the oracle. Distances and histograms are whole numbers: equal, no tolerance."""
import numpy as np
import pytest

import oracle
from paper_2305_14641_amd import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("directed", [False, True])
@pytest.mark.parametrize("n,deg,most", [(700, 3.0, 5), (1500, 2.5, 5), (2048, 3.0, 4), (2049, 3.0, 4), (3000, 3.0, 4),
                                        (4096, 4.5, 4), (4097, 4.5, 4)])
def test_rows(n, deg, most, directed):
    import torch
    from paper_2305_14641_amd import qc
    g = gg.dcsbm_directed(n, [0.6, 0.4], deg / 2, seed=n) if directed else gg.dcsbm(n, [0.6, 0.4], deg, seed=n)
    w = gg.edge_weights(g, most, seed=3, directed=directed)
    G = qc.Graph.from_graph(g, weights=w, directed=directed)
    d = torch.full((n, n), 77, dtype=torch.int8, device="cuda")
    for _ in range(2):   # the first search, and one with the plan for the largest distance
        G.distances(d.fill_(77))
    print(f"[gpu] weighted widths n={n} directed={directed} plan={G.bfs_plan()}", flush=True)
    rows = np.unique(np.concatenate([np.random.default_rng(n).choice(n, 40, replace=False), [0, n - 1]])).astype(np.int32)
    want = oracle.weighted_rows(n, g.row_ptr, g.col, w, rows)[0]
    np.testing.assert_array_equal(d[torch.as_tensor(rows.astype(np.int64), device="cuda")].cpu().numpy(), want)
    hist = G.histograms().cpu().numpy()
    for r, x in zip(rows, want):
        np.testing.assert_array_equal(hist[r], np.bincount(x[x >= 0], minlength=hist.shape[1]))
    G.close()
