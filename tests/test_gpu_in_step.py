"""The pairwise pass of a step on dense rows beyond 1 GiB: the eight waves of a workgroup in step, with rounds in which some or
all but the first have no slab, and the way out for sums that are not finite."""
import numpy as np
import pytest
import torch

from parity_checks import TOL_H, TOL_K

pytestmark = pytest.mark.gpu


def _reference(X, chunk=1 << 18):
    """h and K in 64 bits, a stretch of columns at a time."""
    n, D = X.shape
    d2 = torch.zeros(n, n, dtype=torch.float64, device=X.device)
    for s in range(0, D, chunk):
        Y = X[:, s:s + chunk].double()
        Y -= Y.mean(0, keepdim=True)
        S = Y @ Y.t().contiguous()
        q = S.diagonal()
        d2 += q[:, None] + q[None, :] - 2.0 * S
    d2.clamp_(min=0.0).fill_diagonal_(0.0)
    v = d2.flatten().sort().values
    h = float(0.5 * (v[(n * n - 1) // 2] + v[n * n // 2])) / float(np.log(n + 1.0))
    return h, torch.exp(-d2 / h).cpu().numpy()


@pytest.mark.parametrize("n,D", [(64, 4_194_367), (64, 4_194_497), (60, 4_500_001), (48, 5_592_407), (45, 5_965_235), (44, 6_100_807)])
def test_h_of_a_step(n, D):
    """h and K against 64 bits, and bit for bit as svgd_bandwidth finds them (whose waves take the same slabs one after the other,
    but do not wait for each other).  The first and last slab of every range and the columns after the last slab are scaled until
    they are two thirds of all distances: one of the 1,024 ranges' is some 3e-4 of them, a column of the rest at least a few
    thousandths.  Then one value whose products overflow sends the waves that meet it the fp32 way: that particle is infinitely
    far from all others."""
    from paper_2306_06528_amd import svgd
    assert 4 * n * D > 1 << 30 and torch.cuda.get_device_properties(0).multi_processor_count == 256
    g = torch.Generator(device="cuda").manual_seed(n)
    X = torch.randn(n, D, device="cuda", generator=g)
    G = torch.zeros(n, D, device="cuda")
    nfull, rest = D // 64, D % 64
    per = -(-nfull // 1024)
    slabs = X[:, :64 * nfull].view(n, nfull, 64)
    slabs[:, 0::per] *= (per / 2) ** 0.5
    slabs[:, per - 1::per] *= (per / 2) ** 0.5
    X[:, 64 * nfull:] *= (D / rest) ** 0.5
    with svgd.Svgd(n, D) as eng, svgd.Svgd(n, D) as other:
        h_ref, K_ref = _reference(X)
        for far in (False, True):
            if far:
                X[3, D // 2] = 1e30
            h = other.bandwidth(X)
            _, K = other.get_last(n)
            eng.step(X, G, 0.0)
            h2, K2 = eng.get_last(n)
            assert h2 == h and np.array_equal(K2, K)
            if far:
                assert np.all(K[3, np.arange(n) != 3] == 0.0) and np.all(np.isfinite(K))
            else:
                assert abs(h - h_ref) <= TOL_H * h_ref and float(np.abs(K - K_ref).max()) <= TOL_K
