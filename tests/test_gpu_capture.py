"""A handle's calls recorded into a HIP graph: a replay does what the recorded
call did, whatever the handle was used for in between."""
import numpy as np
import pytest

import oracle
from paper_2305_14641_amd import graphgen as gg

pytestmark = pytest.mark.gpu

GRAPHS = {"undirected": (gg.dcsbm(700, [0.5, 0.5], 4.0, seed=3), {}),
          "directed": (gg.dcsbm_directed(700, [0.5, 0.5], 4.0, seed=3), {"directed": True}),
          "weighted": (gg.dcsbm(300, [0.5, 0.5], 4.0, seed=4), {"weights": 3})}


def handle(name, qc):
    g, kw = GRAPHS[name]
    if "weights" in kw:
        kw = {"weights": gg.edge_weights(g, kw["weights"], seed=1)}
    return g, qc.Graph(g.n, g.row_ptr, g.col, **kw)


@pytest.mark.parametrize("name", list(GRAPHS))
def test_replayed_distances_go_where_they_were_recorded(name):
    import torch
    from paper_2305_14641_amd import qc
    g, G = handle(name, qc)
    print(f"[gpu] capture {name} n={g.n}", flush=True)
    a = torch.full((g.n, g.n), 99, dtype=torch.int8, device="cuda")
    b = torch.full_like(a, 99)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        G.distances(a)
        G.distances(a)              # (the device's descriptor is this call's already)
        s.synchronize()
        want = a.cpu().numpy().copy()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            G.distances(a)
        for k in range(3):
            a.fill_(99)
            b.fill_(99)
            G.distances(b)
            s.synchronize()
            np.testing.assert_array_equal(b.cpu().numpy(), want)
            b.fill_(98)
            graph.replay()
            s.synchronize()
            np.testing.assert_array_equal(a.cpu().numpy(), want)
            assert bool((b == 98).all())
    G.close()
    if name == "undirected":
        np.testing.assert_array_equal(want, oracle.distances(g.n, g.row_ptr, g.col)[0])


FIRST = {"potential": lambda qc, G: G.potential([1.0]), "batch": lambda qc, G: qc.Batch([G], [1.0])}


@pytest.mark.parametrize("resident", [False, True], ids=["into", "resident"])
@pytest.mark.parametrize("first", list(FIRST))
@pytest.mark.parametrize("name", ["undirected", "directed", "long"])
def test_distances_recorded_before_they_ever_ran(name, first, resident):
    """A potential (or a batch) alone has learnt the largest distance: the
    distances can be recorded, and the recorded call outlives ordinary ones."""
    import torch
    from paper_2305_14641_amd import qc
    if name == "long":      # no shape of the row-writing search holds it
        i = np.arange(12600)
        rp, col = gg.csr_from_edges(12600, np.concatenate([i, i]),
                                    np.concatenate([(i + 1) % 12600, (i + 120) % 12600]))
        G = qc.Graph(12600, rp, col)
        n = 12600
    else:
        g, G = handle(name, qc)
        n = g.n
    print(f"[gpu] capture first {name} n={n} {first} resident={resident}", flush=True)
    a = torch.full((n, n), 99, dtype=torch.int8, device="cuda")
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        kept = FIRST[first](qc, G)   # noqa: F841
        h0 = G.histograms()
        s.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            G.distances(None if resident else a)
        graph.replay()
        s.synchronize()
        assert torch.equal(G.histograms(), h0)
        b = torch.full_like(a, 98)
        for k in range(2):
            G.distances(b)           # (tables and plans of its own)
            a.fill_(99)
            graph.replay()
            s.synchronize()
            if not resident:
                assert torch.equal(a, b)
            assert torch.equal(G.histograms(), h0)
        counts = torch.stack([(b[:64] == k).sum(1) for k in range(h0.shape[1])], 1).int()
        assert torch.equal(counts, h0[:64])
        s.synchronize()
    if hasattr(kept, "close"):
        kept.close()
    G.close()
