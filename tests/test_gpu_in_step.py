"""The pairwise pass of a step on dense rows beyond 1 GiB: the eight waves of a workgroup in step, with rounds in which some or
all but the first have no slab, and the way out for sums that are not finite."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,D", [(64, 4_194_367), (64, 4_194_497), (60, 4_500_001), (48, 5_592_407), (45, 5_965_235)])
def test_h_of_a_step(n, D):
    """h and K as svgd_bandwidth finds them (another order of the waves, the same sums up to rounding); a column of values
    whose products overflow sends the waves that meet it the fp32 way."""
    from paper_2306_06528_amd import svgd
    assert 4 * n * D > 1 << 30
    g = torch.Generator(device="cuda").manual_seed(n)
    X = torch.randn(n, D, device="cuda", generator=g)
    G = torch.zeros(n, D, device="cuda")
    with svgd.Svgd(n, D) as eng, svgd.Svgd(n, D) as other:
        for big in (False, True):
            if big:
                X[:, D // 2] *= 2.0 ** 70
            h = other.bandwidth(X)
            _, K = other.get_last(n)
            eng.step(X, G, 0.0)
            h2, K2 = eng.get_last(n)
            # two fp32 sums of the same products in other orders: a few 2^-24; with squares of 2^140 not finite, or what
            # is made of that, either way
            assert h2 == h or abs(h2 - h) <= 1e-6 * h
            assert np.allclose(K2, K, rtol=0.0, atol=1e-6, equal_nan=True)
