"""Algorithm 1 on dense matrices whose rows start at every offset from a
16-byte boundary, with few columns and around a whole round of loads, and with
entries on both sides of where a weight's exponent gets its own handling (and
entries that name no path), against the same sums in FP64. Weights carry the
rounding of one FP32 exponential (below 1.2e-7 relative); psi and V are sums
and ratios of sums of them: 3e-7 relative."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = 3e-7


def reference(d, sigma):
    a = 2.0 * sigma * sigma
    d = d.astype(np.float64)
    ok = np.isfinite(d) & (d >= 0)
    d2 = np.where(ok, d * d, 0.0)
    e = np.where(ok, np.exp(-d2 / a), 0.0)
    psi = e.sum(1)
    return psi, (d2 * e).sum(1) / a / psi


def check(d, n_cols, sigmas):
    import torch
    from paper_2305_14641_amd import qc
    psi, v = qc.potential_dense(d, sigmas, n_cols=n_cols)
    torch.cuda.synchronize()
    host = d.cpu().numpy()[:, :n_cols]
    for s, sigma in enumerate(sigmas):
        p, w = reference(host, sigma)
        np.testing.assert_allclose(psi[s].cpu().numpy(), p, rtol=TOL, atol=0)
        np.testing.assert_allclose(v[s].cpu().numpy(), w, rtol=TOL, atol=1e-300)


@pytest.mark.parametrize("n_sig", [1, 2, 4, 8])
@pytest.mark.parametrize("n_cols,ld", [(1, 1), (2, 3), (3, 5), (4, 7), (5, 5), (63, 65), (1023, 1023), (1024, 1025),
                                       (1026, 1027), (1031, 1031), (4097, 4099)])
def test_offsets(n_cols, ld, n_sig):
    import torch
    print(f"[gpu] dense rows n_cols={n_cols} ld={ld} n_sig={n_sig}", flush=True)
    g = torch.Generator().manual_seed(n_cols)
    d = (torch.rand((9, ld), generator=g) * 6.0).cuda()
    d[:, 0] = 0.0
    check(d, n_cols, [0.7 + 0.4 * k for k in range(n_sig)])


@pytest.mark.parametrize("sigmas", [[1.0], [0.05, 3.0], [0.3, 1e-3, 1e30, 7.0, 2.0]])
def test_range_of_the_exponent(sigmas):
    import torch
    print(f"[gpu] dense exponents {sigmas}", flush=True)
    g = torch.Generator().manual_seed(len(sigmas))
    d = (torch.rand((40, 2051), generator=g) * 5.0)
    edge = min(sigmas) * np.sqrt(2000.0 * np.log(2.0))     # where d^2 / (2 sigma^2) = 1000 ln 2
    d[3] = float(edge)
    d[4:8, ::7] = torch.nextafter(torch.tensor(float(edge)), torch.tensor(0.0))
    d[8:12, ::5] = float(edge) * 1.0001
    d[12, 5] = float("inf")
    d[13, 900] = float("nan")
    d[14, 1500] = -1.0
    d[15, ::2] = 3.0e38
    d[16, ::3] = -0.0
    d[:, 0] = 0.0
    check(d.cuda(), 2051, sigmas)
