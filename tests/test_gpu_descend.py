"""The descent and its centres in one workgroup's LDS (qc_ggd_labels, the
batch, the one-call paths) against the oracle's parents and centres of the
oracle's potentials: node counts at the edges of a slice, of a window of the
thread order and of both LDS sizes (and one node more, where the descent goes
through global memory), lists around the length that a thread scans alone,
more near ties of either kind than LDS queues, and both tie rules and
precisions. Labels are whole numbers: equal, no tolerance."""
import numpy as np
import pytest

import oracle
from paper_2305_14641_amd import graphgen as gg

pytestmark = pytest.mark.gpu

SIGMAS = [0.2, 0.8, 2.5]


def circulant(n, half):
    """Every node joined to the half next and previous ones: all V equal."""
    i = np.repeat(np.arange(n), half)
    k = np.tile(np.arange(1, half + 1), n)
    rp, c = gg.csr_from_edges(n, i, (i + k) % n)
    return gg.Graph(n, rp, c, np.zeros(n, np.int32), name=f"circulant({n},{half})")


def ring_with_chords(n, seed):
    """A ring plus a random perfect matching: degrees 2 and 3, V nearly equal at small sigmas."""
    p = np.random.default_rng(seed).permutation(n)
    i = np.arange(n)
    rp, c = gg.csr_from_edges(n, np.concatenate([i, p[0:n - n % 2:2]]),
                              np.concatenate([(i + 1) % n, p[1:n:2][:n // 2]]))
    return gg.Graph(n, rp, c, np.zeros(n, np.int32), name=f"ring+chords({n})")


def fans(leaves):
    """Hubs in a path with fans of the given sizes, each hub's degree 1 or 2 more."""
    hubs = len(leaves)
    n = hubs + sum(leaves)
    u = list(range(hubs - 1)) + [h for h, k in enumerate(leaves) for _ in range(k)]
    v = list(range(1, hubs)) + list(range(hubs, n))
    rp, c = gg.csr_from_edges(n, np.array(u), np.array(v))
    return gg.Graph(n, rp, c, np.zeros(n, np.int32), name=f"fans({leaves})")


GRAPHS = [gg.path_graph(1), gg.path_graph(2), gg.empty_graph(65), gg.path_graph(63), gg.path_graph(64),
          gg.path_graph(65), gg.complete_graph(32), gg.complete_graph(33), gg.complete_graph(34),
          gg.complete_graph(300), fans([6, 7, 8, 9, 29, 30, 31, 32, 33, 63, 64, 130]), gg.twin_leaves(60, 40),
          circulant(4095, 700), circulant(4096, 20), ring_with_chords(5000, 1), gg.dcsbm(4097, [0.6, 0.4], 6.0, seed=2),
          gg.dcsbm(12864, [0.5, 0.5], 5.0, seed=3), gg.dcsbm(12865, [0.5, 0.5], 5.0, seed=4),
          gg.dcsbm(26560, [0.4, 0.6], 5.0, seed=5), gg.dcsbm(26561, [0.4, 0.6], 5.0, seed=6),
          gg.dcsbm(40705, [0.4, 0.6], 5.0, seed=7), gg.dcsbm(65533, [0.4, 0.6], 4.0, seed=8),
          gg.dcsbm(65536, [0.4, 0.6], 4.0, seed=9)]


@pytest.mark.parametrize("g", GRAPHS, ids=lambda g: f"{g.name}-{g.n}")
def test_labels(g):
    import torch
    from paper_2305_14641_amd import qc
    print(f"[gpu] descent {g.name} n={g.n} nnz={g.nnz}", flush=True)
    G = qc.Graph.from_graph(g)
    want = {}
    for precision in (qc.PREC_FP64ACC, qc.PREC_FP32C):
        G.potential(SIGMAS, precision=precision)
        hist = G.histograms().cpu().numpy()
        for k, sigma in enumerate(SIGMAS):
            for mode in (0, 1):
                if (k, mode) not in want:
                    v = oracle.potential_canonical(hist, sigma)[1]
                    want[k, mode] = oracle.find_centers(oracle.ggd_parent(g.n, g.row_ptr, g.col, v, tie_mode=mode))
                np.testing.assert_array_equal(G.labels(k, tie_mode=mode).cpu().numpy(), want[k, mode])
    for mode in (0, 1):
        b = qc.Batch([G], SIGMAS, tie_mode=mode, hipgraph=False)
        psi, v, labels = b.outputs()
        b.run(psi, v, labels)
        torch.cuda.synchronize()
        for k in range(len(SIGMAS)):
            np.testing.assert_array_equal(labels.cpu().numpy().reshape(len(SIGMAS), -1)[k], want[k, mode])
        b.close()
    G.close()


def test_mixed_sizes_in_a_batch():
    """Graphs of every size class in one batch, each as by itself."""
    import torch
    from paper_2305_14641_amd import qc
    graphs = [gg.path_graph(1), gg.dcsbm(26561, [0.4, 0.6], 4.0, seed=1), circulant(2000, 9),
              gg.dcsbm(13000, [0.4, 0.6], 6.0, seed=2), gg.star_graph(200), gg.dcsbm(900, [0.5, 0.5], 5.0, seed=3)]
    handles = [qc.Graph.from_graph(g) for g in graphs]
    b = qc.Batch(handles, SIGMAS, hipgraph=True)
    outs = b.outputs()
    for _ in range(3):
        b.run(*outs)
        torch.cuda.synchronize()
    labels = outs[2].cpu().numpy().reshape(len(SIGMAS), -1)
    at = 0
    for g, h in zip(graphs, handles):
        hist = h.histograms().cpu().numpy()
        for k, sigma in enumerate(SIGMAS):
            v = oracle.potential_canonical(hist, sigma)[1]
            want = oracle.find_centers(oracle.ggd_parent(g.n, g.row_ptr, g.col, v, tie_mode=0))
            np.testing.assert_array_equal(labels[k, at:at + g.n], want)
        at += g.n
    b.close()
    for h in handles:
        h.close()


@pytest.mark.parametrize("sigmas", [[0.3], [0.3, 1.0]])
def test_recheck_counts_add_up(sigmas):
    """Near ties of a batch are those of its graphs, also where each launch
    holds one (graph, sigma) only; a graph's own count is its last call's."""
    import torch
    from paper_2305_14641_amd import qc
    handles = [qc.Graph.from_graph(gg.dcsbm(n, [0.4, 0.6], 5.0, seed=n)) for n in (27000, 13000, 900)]
    want = 0
    for h in handles:
        h.potential(sigmas)
        counts = []
        for k in range(len(sigmas)):
            h.labels(k)
            counts.append(h.recheck_count())
            h.labels(k)
            assert h.recheck_count() == counts[-1]
        assert counts[0] > 0
        want += sum(counts)
    b = qc.Batch(handles, sigmas, hipgraph=False)
    outs = b.outputs()
    for _ in range(2):
        b.run(*outs)
        torch.cuda.synchronize()
        assert b.recheck_count() == want
    b.close()
    for h in handles:
        h.close()
