"""Server requests that return potentials, on graphs whose largest distance lies
at the edges of the histogram row lengths (31 | 32, 63 | 64, the limit 126):
labels, psi, V and dmax against the step calls, byte for byte."""
import numpy as np
import pytest

from paper_2305_14641_amd import graphgen as gg

pytestmark = pytest.mark.gpu


def request_graph(dmax, others):
    """A path of largest distance `dmax`, alone or beside denser components."""
    path = gg.path_graph(dmax + 1)
    if not others:
        return path
    return gg.disjoint_union(gg.dcsbm(others, [0.5, 0.5], 5.0, seed=others), path, gg.star_graph(9))


@pytest.mark.parametrize("sigmas", [[1.3], [0.4, 1.0, 2.0, 3.5, 6.0]], ids=["S1", "S5"])
@pytest.mark.parametrize("others", [0, 900])
@pytest.mark.parametrize("dmax", [31, 32, 63, 64, 126])
def test_potentials_of_long_graphs(dmax, others, sigmas):
    import torch
    from paper_2305_14641_amd import qc
    g = request_graph(dmax, others)
    print(f"[gpu] server n={g.n} dmax={dmax} S={len(sigmas)}", flush=True)
    srv = qc.Server(max_slots=2, hbm_budget_bytes=1 << 30, want_potentials=True)
    ids = [srv.submit(g.n, g.row_ptr, g.col, sigmas) for _ in range(3)]
    got = [srv.wait(i) for i in ids]
    srv.close()
    G = qc.Graph.from_graph(g)
    psi, v = G.potential(sigmas)
    labels = torch.stack([G.labels(k) for k in range(len(sigmas))]).cpu().numpy()
    for lab, p, w, info in got:
        assert info["status"] == 0 and info["dmax"] == dmax
        np.testing.assert_array_equal(p, psi.cpu().numpy())
        np.testing.assert_array_equal(w, v.cpu().numpy())
        np.testing.assert_array_equal(lab, labels)
    G.close()
