"""The one-call form without a matrix on graphs with nodes that the counting
search leaves out (leaves, isolated edges and nodes, nothing but them) and with
largest distances at the edges of the histogram row lengths (a leaf's may be
the one that no longer fits), against the step calls, byte for byte, and the
oracle's refusal of distances beyond the limit."""
import numpy as np
import pytest

from paper_2305_14641_amd import graphgen as gg

pytestmark = pytest.mark.gpu

SIGMAS = [0.4, 1.0, 2.0, 3.5, 6.0]
GRAPHS = [gg.path_graph(1), gg.path_graph(2), gg.path_graph(3), gg.empty_graph(300), gg.star_graph(1),
          gg.star_graph(2), gg.star_graph(700), gg.twin_leaves(20, 30), gg.complete_graph(70), gg.barbell_graph(30),
          gg.disjoint_union(gg.path_graph(2), gg.star_graph(70), gg.empty_graph(3), gg.complete_graph(12),
                            gg.path_graph(3), gg.path_graph(2)),
          gg.dcsbm(257, [0.5, 0.5], 3.0, seed=1), gg.dcsbm(5000, [0.5, 0.5], 3.0, seed=2)] + \
         [gg.path_graph(n) for n in (31, 32, 33, 34, 63, 64, 65, 66, 126, 127)]


@pytest.mark.parametrize("form", ["cluster", "cluster_noalloc"])
@pytest.mark.parametrize("g", GRAPHS, ids=lambda g: f"{g.name}-{g.n}")
def test_equals_the_step_calls(g, form):
    import torch
    from paper_2305_14641_amd import qc
    print(f"[gpu] one call {form} {g.name} n={g.n}", flush=True)
    S = len(SIGMAS)
    psi = torch.full((S, g.n), -1.0, dtype=torch.float32, device="cuda")
    v = torch.full_like(psi, -1.0)
    labels = torch.full((S, g.n), -1, dtype=torch.int32, device="cuda")
    getattr(qc, form)(g.n, g.row_ptr, g.col, SIGMAS, psi=psi, v=v, labels=labels)
    G = qc.Graph.from_graph(g)
    p, w = torch.empty_like(psi), torch.empty_like(psi)
    G.potential(SIGMAS, psi=p, v=w)
    np.testing.assert_array_equal(psi.cpu().numpy(), p.cpu().numpy())
    np.testing.assert_array_equal(v.cpu().numpy(), w.cpu().numpy())
    for k in range(S):
        np.testing.assert_array_equal(labels[k].cpu().numpy(), G.labels(k).cpu().numpy())
    G.close()


@pytest.mark.parametrize("n", [128, 129, 200])
def test_too_long_is_refused(n):
    import torch
    from paper_2305_14641_amd import qc
    g = gg.path_graph(n)   # largest distance n - 1
    labels = torch.empty((1, n), dtype=torch.int32, device="cuda")
    with pytest.raises(Exception):
        qc.cluster(g.n, g.row_ptr, g.col, [1.0], labels=labels)
