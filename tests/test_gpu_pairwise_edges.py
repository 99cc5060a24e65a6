"""The pairwise pass where a wave has one slab of 64 columns: rows of fewer than four columns, partial slabs of every
kind of end, particle counts that fill their last block of 16 rows or not.  What lies beside the rows is NaN."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [1, 2, 3, 4, 5, 7, 61, 63, 64, 66, 255, 256, 257, 1022, 65_534])
@pytest.mark.parametrize("n", [13, 16, 17, 31, 33, 47, 48, 49, 63, 64])
def test_last_columns_and_last_rows(n, D):
    from paper_2306_06528_amd import svgd
    g = torch.Generator(device="cuda").manual_seed(1000 * n + D)
    buf = torch.full((n + 1, D + 9), float("nan"), device="cuda")
    X = buf[:n, 3:D + 3]
    X.copy_(torch.randn(n, D, device="cuda", generator=g))
    Y = X.double() - X.double().mean(0, keepdim=True)
    d2 = (Y[:, None, :] - Y[None, :, :]).square().sum(2) if n * n * D < 2 ** 24 else torch.cdist(Y, Y, compute_mode="donot_use_mm_for_euclid_dist").square()
    v = d2.flatten().sort().values
    h_ref = float(0.5 * (v[(n * n - 1) // 2] + v[(n * n) // 2])) / float(torch.log(torch.tensor(n + 1.0, dtype=torch.float64)))
    with svgd.Svgd(n, D + 9) as eng:
        h = eng.bandwidth(X)
        _, K = eng.get_last(n)
    # d2 of a pair is off by a few 2^-24 of the squares it is made of, at most some ten times the median's share here
    assert abs(h - h_ref) <= 1e-5 * h_ref
    assert float((torch.from_numpy(K).double() - torch.exp(-d2 / h_ref).cpu()).abs().max()) <= 1e-5
