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
