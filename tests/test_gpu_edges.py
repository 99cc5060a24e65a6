"""Sizes at which the split of the work leaves remainders: the columns after the last full tile of the
matrix-core update (one workgroup, 4 x 4 tiles of rows and columns, pairs of row groups for the
carried sums) and the last, partly filled round of the streaming moments kernel."""
import pytest
import torch

from parity_checks import check_carried_chain

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("padded", [True, False])
@pytest.mark.parametrize("D", [33, 63, 65, 127, 259])
@pytest.mark.parametrize("n", [13, 16, 20, 31, 36, 52, 61, 64])
def test_columns_after_the_last_tile(n, D, padded):
    """Two steps on carried sums (the second reads the tail's pair sums) against the oracle.  (Not at a D
    of one or two: a squared difference of two single numbers, taken from sums of their squares,
    keeps 2^-24 of the squares, so that h from carried and from recomputed sums differ by more
    than the one-ulp comparison of the update allows.)"""
    from paper_2306_06528_amd import svgd
    g = torch.Generator().manual_seed(1000 * n + D)
    X = (0.3 * torch.randn(n, D, generator=g)).cuda()
    G = torch.randn(n, D, generator=g).cuda()
    check_carried_chain(svgd, X, G, 0.05, padded=padded, steps=2)


@pytest.mark.parametrize("total", [1, 5, 1024 * 2048 + 3, 13_981_013, 13_981_014, 4 * 256 * 256 * 4 * 13 + 1029])
def test_moments_at_the_edges(total):
    """Totals around one round of all threads, around the size at which the kernel changes, odd ends.
    One update of fp32 running means: m + (x - m)/(c + 1), rounded a handful of times."""
    from paper_2306_06528_amd import svgd
    g = torch.Generator().manual_seed(total)
    mean, sq, X = (torch.randn(1, total, generator=g) for _ in range(3))
    sq = sq.abs()
    md, sd, Xd = mean.cuda(), sq.cuda(), X.cuda()
    svgd.swag_update_moments(md, sd, Xd, 3)
    m, s, x = mean.double(), sq.double(), X.double()
    ref_m, ref_s = m + (x - m) / 4.0, s + (x * x - s) / 4.0
    # three roundings of numbers no larger than |m| + |x|, or s + x^2
    tol = 2.0 ** -22
    assert bool(((md.cpu().double() - ref_m).abs() <= tol * (m.abs() + x.abs())).all())
    assert bool(((sd.cpu().double() - ref_s).abs() <= tol * (s + x * x)).all())
