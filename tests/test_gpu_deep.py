"""Distances of small graphs on both sides of the rule that sends those of many
levels to the matrix search, before and after their potentials, against the
oracle; histograms and potentials of both routes agree byte for byte."""
import numpy as np
import pytest

import oracle
from paper_2305_14641_amd import graphgen as gg

pytestmark = pytest.mark.gpu


def grid(w, h):
    i = np.arange(w * h).reshape(h, w)
    rp, c = gg.csr_from_edges(w * h, np.concatenate([i[:, :-1].ravel(), i[:-1].ravel()]),
                              np.concatenate([i[:, 1:].ravel(), i[1:].ravel()]))
    return gg.Graph(w * h, rp, c, np.zeros(w * h, np.int32), name=f"grid{w}x{h}")


GRAPHS = [gg.path_graph(n) for n in (1, 2, 24, 25, 26, 27, 33, 64, 65, 127)] + \
         [grid(2, 60), grid(8, 64), grid(9, 57), grid(6, 80), grid(4, 64), grid(10, 10), grid(13, 13), grid(20, 20), gg.twin_leaves(12, 30),
          gg.disjoint_union(gg.path_graph(40), gg.star_graph(9), gg.empty_graph(2), gg.path_graph(2)),
          gg.dcsbm(512, [0.5, 0.5], 3.0, seed=1), gg.dcsbm(513, [0.5, 0.5], 3.0, seed=2),
          # leaves' rows searched like the others' (up to 2,048 nodes, most of them no leaves), or derived
          gg.dcsbm(2048, [0.5, 0.5], 3.0, seed=3), gg.dcsbm(2049, [0.5, 0.5], 3.0, seed=4), gg.star_graph(60),
          gg.disjoint_union(gg.complete_graph(9), gg.empty_graph(3), gg.path_graph(2), gg.star_graph(4))]


@pytest.mark.parametrize("first", ["distances", "potential"])
@pytest.mark.parametrize("g", GRAPHS, ids=lambda g: f"{g.name}-{g.n}")
def test_distances_of_deep_graphs(g, first):
    import torch
    from paper_2305_14641_amd import qc
    print(f"[gpu] deep {g.name} n={g.n} {first}", flush=True)
    want, dmax = oracle.distances(g.n, g.row_ptr, g.col)
    G = qc.Graph.from_graph(g)
    if first == "potential":
        psi, v = G.potential([0.8, 2.0])
        h = G.histograms()
    for _ in range(2):
        d = torch.full((g.n, g.n), 99, dtype=torch.int8, device="cuda")
        assert G.distances(d) == dmax
        np.testing.assert_array_equal(d.cpu().numpy(), want)
    if first == "distances":
        psi, v = G.potential([0.8, 2.0])
        h = G.histograms()
    np.testing.assert_array_equal(G.histograms().cpu().numpy()[:, :dmax + 1], oracle.hist_rows(want, dmax + 1))
    assert torch.equal(G.histograms(), h)
    p2, v2 = G.potential([0.8, 2.0])
    assert torch.equal(p2, psi) and torch.equal(v2, v)
    G.close()


@pytest.mark.parametrize("mixed", [False, True], ids=["deep", "mixed"])
def test_a_batch_of_deep_graphs(mixed):
    """Nothing but small deep graphs (the matrix search), and beside others."""
    import torch
    from paper_2305_14641_amd import qc
    graphs = [gg.path_graph(127), gg.path_graph(40), grid(2, 60), gg.path_graph(128 - 1)]
    if mixed:
        graphs += [gg.path_graph(9), gg.dcsbm(700, [0.5, 0.5], 4.0, seed=3)]
    sigmas = [0.6, 1.9]
    print(f"[gpu] deep batch mixed={mixed}", flush=True)
    handles = [qc.Graph.from_graph(g) for g in graphs]
    handles[1].potential([1.0])      # (one has searched before)
    b = qc.Batch(handles, sigmas)
    outs = b.outputs()
    for _ in range(2):
        b.run(*outs)
    torch.cuda.synchronize()
    for i, (g, h) in enumerate(zip(graphs, handles)):
        dist, dmax = oracle.distances(g.n, g.row_ptr, g.col)
        hist = oracle.hist_rows(dist, dmax + 1)
        at = slice(int(b.offsets[i]), int(b.offsets[i + 1]))
        for k, s in enumerate(sigmas):
            psi, v = oracle.potential_canonical(hist, s)
            np.testing.assert_allclose(outs[0][k, at].cpu().numpy(), psi, rtol=1e-6, atol=0)
            np.testing.assert_allclose(outs[1][k, at].cpu().numpy(), v, rtol=1e-6, atol=0)
            want = oracle.find_centers(oracle.ggd_parent(g.n, g.row_ptr, g.col, v, 0))
            np.testing.assert_array_equal(outs[2][k, at].cpu().numpy(), want)
        d = torch.full((g.n, g.n), 99, dtype=torch.int8, device="cuda")
        assert h.distances(d) == dmax
        np.testing.assert_array_equal(d.cpu().numpy(), dist)
    b.close()
    for h in handles:
        h.close()
