"""The one-call forms on graphs with distances beyond the limit of 126: the
status is QC_E_OVERFLOW and the outputs are as they were, where only two leaves
are that far apart, where nodes of any kind are, and above the size that one
workgroup descends."""
import numpy as np
import pytest

from paper_2305_14641_amd import graphgen as gg

pytestmark = pytest.mark.gpu


def cycle(n):
    i = np.arange(n)
    return gg.csr_from_edges(n, i, (i + 1) % n)


def csr(g):
    return (g.n, g.row_ptr, g.col) if hasattr(g, "row_ptr") else (len(g[0]) - 1, *g)


CASES = [("path128", gg.path_graph(128), ("cluster", "cluster_noalloc")),     # the two ends, 127 apart
         ("path129", gg.path_graph(129), ("cluster", "cluster_noalloc")),
         ("path200", gg.path_graph(200), ("cluster", "cluster_noalloc")),
         ("cycle254", cycle(254), ("cluster", "cluster_noalloc")),            # no leaves
         ("twins", gg.disjoint_union(gg.star_graph(40), gg.path_graph(128), gg.complete_graph(9)),
          ("cluster", "cluster_noalloc")),
         ("large", gg.disjoint_union(gg.dcsbm(27000, [0.5, 0.5], 4.0, seed=7), gg.path_graph(128)), ("cluster",))]


@pytest.mark.parametrize("name,g,forms", CASES, ids=[c[0] for c in CASES])
def test_an_overflow_leaves_the_outputs_alone(name, g, forms):
    import torch
    from paper_2305_14641_amd import qc
    n, rp, col = csr(g)
    sigmas = [0.7, 2.0]
    for form in forms:
        print(f"[gpu] overflow {form} {name} n={n}", flush=True)
        psi = torch.full((2, n), -1.0, dtype=torch.float32, device="cuda")
        v = torch.full_like(psi, -1.0)
        labels = torch.full((2, n), -7, dtype=torch.int32, device="cuda")
        with pytest.raises(qc.QCError) as e:
            getattr(qc, form)(n, rp, col, sigmas, psi=psi, v=v, labels=labels)
        assert e.value.status == qc.QC_E_OVERFLOW
        assert bool((psi == -1.0).all()) and bool((v == -1.0).all()) and bool((labels == -7).all())


def test_the_server_reports_it():
    from paper_2305_14641_amd import qc
    srv = qc.Server(max_slots=1, hbm_budget_bytes=1 << 30, want_potentials=True)
    for g in (gg.path_graph(128), gg.path_graph(127)):
        rid = srv.submit(g.n, g.row_ptr, g.col, [1.0])
        if g.n == 127:
            assert srv.wait(rid)[3]["dmax"] == 126
        else:
            with pytest.raises(qc.QCError) as e:
                srv.wait(rid)
            assert e.value.status == qc.QC_E_OVERFLOW
    srv.close()
