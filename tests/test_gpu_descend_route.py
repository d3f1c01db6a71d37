"""Descent in one workgroup's LDS or through global memory: graphs on both sides
of the rule (dense, regular and large ones go through global memory, few pairs
or many), in label calls, one-call forms and batches, against the oracle's
centres of the oracle's potentials. Labels are whole numbers: no tolerance."""
import numpy as np
import pytest

import oracle
from paper_2305_14641_amd import graphgen as gg

pytestmark = pytest.mark.gpu


def graph(n, u, v, name):
    rp, c = gg.csr_from_edges(n, u, v)
    return gg.Graph(n, rp, c, np.zeros(n, np.int32), name=name)


def random_ring(n, extra, seed):
    """A ring in a random order and `extra` random chords per node."""
    r = np.random.default_rng(seed)
    p = r.permutation(n)
    u, v = r.integers(0, n, extra * n), r.integers(0, n, extra * n)
    keep = u != v
    return graph(n, np.concatenate([p, u[keep]]), np.concatenate([np.roll(p, 1), v[keep]]), f"ring+{extra}")


def circulant(n, half):
    i = np.repeat(np.arange(n), half)
    k = np.tile(np.arange(1, half + 1), n)
    return graph(n, i, (i + k) % n, f"circulant{half}")


def centres(g, sigmas):
    hist, dmax = oracle.hist_all(g.n, g.row_ptr, g.col, 128)
    hist = np.ascontiguousarray(hist[:, :dmax + 1])
    return np.stack([oracle.find_centers(oracle.ggd_parent(g.n, g.row_ptr, g.col,
                                                           oracle.potential_canonical(hist, s)[1], 0))
                     for s in sigmas])


GRAPHS = [gg.complete_graph(500), gg.complete_graph(700), random_ring(3000, 1, 1), random_ring(7000, 1, 2),
          random_ring(1500, 5, 3), random_ring(6000, 5, 4), gg.dcsbm(20000, [0.5, 0.5], 8.0, seed=5),
          gg.dcsbm(26560, [0.5, 0.5], 8.0, seed=6)]


@pytest.mark.parametrize("g", GRAPHS, ids=lambda g: f"{g.name}-{g.n}")
def test_labels_on_both_sides_of_the_rule(g):
    import torch
    from paper_2305_14641_amd import qc
    print(f"[gpu] route {g.name} n={g.n} nnz={g.nnz}", flush=True)
    sigmas = [0.3, 0.8, 1.7, 2.5, 6.0]
    want = centres(g, sigmas)
    G = qc.Graph.from_graph(g)
    G.potential(sigmas)
    for k in range(len(sigmas)):
        np.testing.assert_array_equal(G.labels(k).cpu().numpy(), want[k])
    for S in (1, 5):
        labels = torch.full((S, g.n), -1, dtype=torch.int32, device="cuda")
        qc.cluster(g.n, g.row_ptr, g.col, sigmas[:S], labels=labels)
        np.testing.assert_array_equal(labels.cpu().numpy(), want[:S])
        b = qc.Batch([G], sigmas[:S])
        outs = b.outputs()
        for _ in range(2):
            b.run(*outs)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(outs[2].cpu().numpy().reshape(S, -1), want[:S])
        b.close()
    G.close()


def test_many_pairs_of_dense_ties_descend_in_lds():
    """Enough pairs that they take turns on the chip, each with more near ties
    among many neighbours than LDS queues."""
    import torch
    from paper_2305_14641_amd import qc
    g = circulant(4096, 20)
    sigmas = list(np.geomspace(0.4, 6.0, 32))
    print(f"[gpu] route {g.name} n={g.n} x 16 x 32", flush=True)
    want = centres(g, sigmas)
    handles = [qc.Graph.from_graph(g) for _ in range(16)]
    b = qc.Batch(handles, sigmas)
    outs = b.outputs()
    b.run(*outs)
    torch.cuda.synchronize()
    got = outs[2].cpu().numpy().reshape(32, 16, g.n)
    for i in range(16):
        np.testing.assert_array_equal(got[:, i], want)
    b.close()
    for h in handles:
        h.close()
