"""The vector-ALU path (up to 12 particles) at its remainders: rows of fewer than four columns and last column
groups of one to three, on every kind of call; lists of partial sums around the rounds in which the update reads
them; and distances with ties, whose ranks are found by counting."""
import numpy as np
import pytest
import torch

from parity_checks import TOL_H, TOL_K, TOL_PHI, assert_x_new, check_carried_chain
from oracle import svgd_oracle as orc

pytestmark = pytest.mark.gpu


def _inputs(n, D, seed):
    g = torch.Generator().manual_seed(seed)
    return (0.3 * torch.randn(n, D, generator=g)).cuda(), torch.randn(n, D, generator=g).cuda()


@pytest.mark.parametrize("D", [1, 2, 3, 5, 1021, 2049, 16387])
@pytest.mark.parametrize("n", [1, 2, 3, 7, 8, 9, 12])
def test_last_column_group(n, D):
    """Columns behind the rows hold NaN: a value read beyond D and not replaced would show."""
    from paper_2306_06528_amd import svgd
    X, G = _inputs(n, D, 100 * n + D)
    ref = orc.step(X.cpu().numpy(), G.cpu().numpy(), 0.05)
    ld = D + 5
    bx, bg, bp = (torch.full((n + 1, ld), float("nan"), device="cuda") for _ in range(3))
    Xp, Gp, PHI = bx[:n, :D], bg[:n, :D], bp[:n, :D]
    Xp.copy_(X)
    Gp.copy_(G)
    with svgd.Svgd(n, D) as eng:
        eng.phi(Xp, Gp, PHI)
        scale = max(float(np.abs(ref["phi"]).max()), 1e-30)
        assert float(np.abs(PHI.cpu().numpy() - ref["phi"]).max()) <= TOL_PHI * scale
        rows, grows = [X[i].clone() for i in range(n)], [G[i].clone() for i in range(n)]
        eng.step_rows(rows, grows, 0.05)
        assert_x_new(torch.stack(rows).cpu().numpy(), ref, 0.05, "rows")
        h = eng.bandwidth(Xp)
        assert abs(h - ref["h"]) <= TOL_H * ref["h"]
        eng.step(Xp, Gp, 0.05)
        assert_x_new(Xp.cpu().numpy(), ref, 0.05, "step")
    for b in (bx, bg, bp):  # nothing is written behind the rows
        assert bool(torch.isnan(b[:, D:]).all()) and bool(torch.isnan(b[n]).all())


# (the list has one partial per 1024 columns, up to two per CU: the update reads it in rounds of 16, 8 or 4 loads of
# 4 R partials, R = 16, 8, 7, 3)
@pytest.mark.parametrize("n,D", [(2, 4 * 16 * 4 * 1024), (4, 8 * 16 * 4 * 1024 + 4), (6, 8 * 8 * 4 * 1024 + 1), (8, 4 * 7 * 4 * 1024),
                                 (8, 4 * 7 * 4 * 1024 + 3), (8, 16 * 7 * 4 * 1024 + 1), (12, 8 * 3 * 4 * 1024 + 2), (12, 16 * 3 * 4 * 1024 + 1)])
def test_lists_around_a_round_of_loads(n, D):
    from paper_2306_06528_amd import svgd
    X, G = _inputs(n, D, n + D)
    check_carried_chain(svgd, X, G, 0.05, padded=False, steps=3)


@pytest.mark.parametrize("D", [40, 8195])
@pytest.mark.parametrize("n", range(2, 13))
def test_equal_distances(n, D):
    """Particles in two places: all distances are 0 or one value (exactly, both sides of the rank), and with
    n // 3 in the second place the median is one or the other."""
    from paper_2306_06528_amd import svgd
    a, b = _inputs(2, D, D)[0]
    for second in {1, n // 3, n // 2}:
        X = torch.stack([b if i < second else a for i in range(n)])
        G = torch.ones_like(X)
        ref = orc.step(X.cpu().numpy(), G.cpu().numpy(), 0.05)
        with svgd.Svgd(n, D) as eng:
            eng.step(X, G, 0.05)
            h, K = eng.get_last(n)
        assert abs(h - ref["h"]) <= TOL_H * ref["h"], second
        assert float(np.abs(K - ref["K"]).max()) <= TOL_K
        assert_x_new(X.cpu().numpy(), ref, 0.05, f"second {second}")


@pytest.mark.parametrize("kind", ["line", "line_reversed", "two_places", "half_equal", "one_far", "random"])
@pytest.mark.parametrize("n", [13, 14, 15, 16])
def test_selection_by_a_wave(n, kind):
    """13 to 16 particles, whose distances the waves rank in shares, each picking the middle ones for itself: orders
    in the data, ties on either side of the wanted ranks, all sizes of what is left above them."""
    from paper_2306_06528_amd import svgd
    D = 600
    base = _inputs(n, D, n)[0]
    at = {"line": torch.arange(n), "line_reversed": torch.arange(n).flip(0), "two_places": torch.arange(n) % 2,
          "half_equal": torch.clamp(torch.arange(n) - n // 2, min=0), "one_far": (torch.arange(n) == 3) * 50,
          "random": torch.zeros(n)}[kind].float().cuda()
    X = base if kind == "random" else at[:, None] * base[0][None, :] / 8 + base[1][None, :]
    X = X.contiguous()
    G = torch.ones_like(X)
    ref = orc.step(X.cpu().numpy(), G.cpu().numpy(), 0.05)
    with svgd.Svgd(n, D) as eng:
        eng.step(X, G, 0.05)
        h, K = eng.get_last(n)
    # sums of squares in fp32 around the mean: a distance is good to some 2^-22 of the largest square
    assert abs(h - ref["h"]) <= TOL_H * ref["h"]
    assert float(np.abs(K - ref["K"]).max()) <= TOL_K
