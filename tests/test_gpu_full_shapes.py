"""Distance rows of graphs that fill a launch shape to the last position (no
leaves, no spare one), with and without hubs, with 4, 5 and 7 bit-planes, and of
sizes on both sides of the rules that choose between the two searches, against
the oracle."""
import numpy as np
import pytest

import oracle
from paper_2305_14641_amd import graphgen as gg

pytestmark = pytest.mark.gpu


def ring(n, chords, seed, hubs=0):
    """A ring in a random order, `chords` random chords, and `hubs` nodes joined
    to 300 others each: no leaves."""
    r = np.random.default_rng(seed)
    p = r.permutation(n)
    u, v = r.integers(0, n, chords), r.integers(0, n, chords)
    hu = np.repeat(r.choice(n, hubs, replace=False), 300) if hubs else np.zeros(0, np.int64)
    u = np.concatenate([p, u, hu])
    v = np.concatenate([np.roll(p, 1), v, r.integers(0, n, len(hu))])
    keep = u != v
    return gg.csr_from_edges(n, u[keep], v[keep])


CASES = [(n, c * n // 10, h) for n in (4095, 4096, 4097, 8192, 12288) for c, h in ((15, 0), (15, 7), (4, 0), (2, 3))] + \
        [(4096, 300, 0), (8192, 700, 0), (8192, 4096, 40), (16383, 24576, 0), (16384, 24576, 5), (16384, 6000, 0), (16385, 6000, 0),
         (18200, 7000, 0), (18201, 7000, 0)]


@pytest.mark.parametrize("n,chords,hubs", CASES)
def test_rows_of_full_shapes(n, chords, hubs):
    import torch
    from paper_2305_14641_amd import qc
    rp, col = ring(n, chords, seed=n + chords + hubs, hubs=hubs)
    want, dmax = oracle.distances(n, rp, col)
    print(f"[gpu] full shape n={n} chords={chords} hubs={hubs} dmax={dmax}", flush=True)
    assert dmax <= 126
    G = qc.Graph(n, rp, col)
    d = torch.full((n, n), 99, dtype=torch.int8, device="cuda")
    for _ in range(2):
        assert G.distances(d) == dmax
    np.testing.assert_array_equal(d.cpu().numpy(), want)
    h = G.histograms()
    np.testing.assert_array_equal(h.cpu().numpy()[:256, :dmax + 1], oracle.hist_rows(want[:256], dmax + 1))
    assert int(h.sum()) == int((want >= 0).sum())
    G.close()
