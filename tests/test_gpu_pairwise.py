"""The pairwise pass on the matrix cores where products are taken from values split into three bf16 parts: where every
wave has several slabs (D >= 65,536 on 256 CUs), and from 33 particles on at every D."""
import math

import numpy as np
import pytest
import torch

from oracle import svgd_oracle as orc
from parity_checks import TOL_H, TOL_K, TOL_PHI, assert_x_new, padded_copy

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [65_535, 65_536, 200_003])
@pytest.mark.parametrize("n,m", [(17, 14), (24, 20), (32, 28), (33, 30), (48, 40), (64, 56), (64, 60)])
def test_equal_particles_across_blocks(n, m, D):
    """m of n particles are equal and lie in all blocks of 16: their distances are exactly 0 (K exactly
    1), and with more than half of all distances 0 the median is 0 and h = 1, by every entry point."""
    from paper_2306_06528_amd import svgd
    for seed in (1, 2):
        g = torch.Generator().manual_seed(100 * n + seed)
        Xh = torch.randn(n, D, generator=g)
        same = torch.randperm(n, generator=g)[:m].sort().values
        Xh[same] = Xh[same[0]].clone()
        Gh = torch.randn(n, D, generator=g)
        ref = orc.step(Xh.numpy(), Gh.numpy(), 0.01)
        assert ref["h"] == 1.0
        inside = np.ix_(same.numpy(), same.numpy())

        def check(eng, what):
            h, K = eng.get_last(n)
            assert abs(h - ref["h"]) <= TOL_H * ref["h"], f"{what}: h = {h}"
            assert np.all(K[inside] == 1.0), f"{what}: K down to {K[inside].min()} between equal particles"
            assert np.abs(K - ref["K"]).max() <= TOL_K, what

        X, G = Xh.cuda(), Gh.cuda()
        Xp, Gp = padded_copy(svgd, X), padded_copy(svgd, G)
        with svgd.Svgd(n, D) as eng:
            for what, x, gr in (("dense", X, G), ("padded", Xp, Gp)):
                PHI = torch.empty_strided(x.shape, x.stride(), device="cuda")
                eng.bandwidth(x)
                check(eng, what + " bandwidth")
                eng.phi(x, gr, PHI)
                check(eng, what + " phi")
                assert np.abs(PHI.cpu().numpy() - ref["phi"]).max() <= TOL_PHI * np.abs(ref["phi"]).max(), what
            rows = [X[i].clone() for i in range(n)]
            eng.step_rows(rows, [G[i].clone() for i in range(n)], 0.01)
            check(eng, "rows")
            assert_x_new(torch.stack(rows).cpu().numpy(), ref, 0.01, "rows")
            Xs = X.clone()
            svgd.step_static(Xs, G, 0.01)
            assert_x_new(Xs.cpu().numpy(), ref, 0.01, "static")
            eng.step(X, G, 0.01)
            check(eng, "step")
            assert_x_new(X.cpu().numpy(), ref, 0.01, "step")
        with svgd.Svgd(n, D, flags=svgd.FLAG_CARRY_GRAM) as eng:
            eng.step(Xp, Gp, 0.01)
            check(eng, "first step of a chain")


@pytest.mark.parametrize("padded", [False, True])
@pytest.mark.parametrize("n,m,D", [(10, 8, 5001), (16, 12, 5001), (24, 20, 20_001), (32, 28, 20_001), (48, 40, 130), (64, 56, 20_035)])
def test_equal_particles_stay_equal_on_carried_sums(n, m, D, padded):
    """Particles that are equal and have equal scores stay equal, and a chain of steps on carried pair sums,
    the columns after the last full tile among them, keeps their distances at exactly 0."""
    from paper_2306_06528_amd import svgd
    g = torch.Generator().manual_seed(n)
    Xh, Gh = torch.randn(n, D, generator=g), torch.randn(n, D, generator=g)
    same = torch.randperm(n, generator=g)[:m].sort().values
    Xh[same], Gh[same] = Xh[same[0]].clone(), Gh[same[0]].clone()
    X, G = Xh.cuda(), Gh.cuda()
    if padded:
        X, G = padded_copy(svgd, X), padded_copy(svgd, G)
    inside = np.ix_(same.numpy(), same.numpy())
    with svgd.Svgd(n, D, flags=svgd.FLAG_CARRY_GRAM) as eng:
        for step in range(5):
            eng.step(X, G, 0.01)
            h, K = eng.get_last(n)
            assert h == 1.0, f"step {step}: h = {h}"
            assert np.all(K[inside] == 1.0), f"step {step}: K down to {K[inside].min()} between equal particles"
    Xh = X.cpu()
    assert all(torch.equal(Xh[i], Xh[same[0]]) for i in same)


def _pairs(svgd, X, layout, h_fixed):
    """h and K of the rows of X (h_fixed = 0: the median's)."""
    n, D = X.shape
    with svgd.Svgd(n, D) as eng:
        eng.set_bandwidth(h_fixed)
        if layout == "rows":
            eng.step_rows([X[i].clone() for i in range(n)], [torch.zeros(D, device="cuda") for _ in range(n)], 0.0)
        else:
            eng.bandwidth(padded_copy(svgd, X) if layout == "padded" else X)
        return eng.get_last(n)


# d2 read back from K = exp(-d2 / h) at a fixed h = d2 / 16 or so: K is rounded to 2^-24 of itself, d2 by
# 2^-24 / 16 = 4e-9.  The pass itself is off by up to 1.2e-8 (measured, n = 13..64, D = 65,536..3 M), h by
# 5e-9 (n = 33..64, D = 20,001: 1.4e-8 and 4e-9): four times that.  With few slabs fewer roundings cancel: D = 1,001,
# n = 33..64, 4.8e-8 and 1.7e-8 (from fp32 products twice that).
TOL_D2, TOL_H_FINE = 5.2e-8, 2e-8
TOL_D2_SMALL, TOL_H_SMALL = 2e-7, 6.6e-8


@pytest.mark.parametrize("layout", ["dense", "padded", "rows"])
@pytest.mark.parametrize("n,D", [(13, 70_001), (16, 300_007), (20, 131_100), (33, 70_001), (48, 300_007), (64, 131_100),
                                 (33, 1_001), (48, 1_001), (64, 1_001), (33, 20_001), (48, 20_001), (64, 20_001)])
def test_distances_to_seven_digits(n, D, layout):
    from paper_2306_06528_amd import svgd
    tol_d2, tol_h = (TOL_D2, TOL_H_FINE) if D > 20_000 else (TOL_D2_SMALL, TOL_H_SMALL)
    Xh = torch.randn(n, D, generator=torch.Generator().manual_seed(7 * n + D))
    d2 = orc.pairwise_d2(Xh.numpy())
    h_ref = orc.bandwidth(d2)
    h, _ = _pairs(svgd, Xh.cuda(), layout, 0.0)
    assert abs(h - h_ref) <= tol_h * h_ref
    iu = np.triu_indices(n, 1)
    hf = float(np.median(d2[iu])) / 16.0
    _, K = _pairs(svgd, Xh.cuda(), layout, hf)
    got = -hf * np.log(K[iu].astype(np.float64))
    assert np.abs(got / d2[iu] - 1.0).max() <= tol_d2


@pytest.mark.parametrize("layout", ["dense", "padded", "rows"])
@pytest.mark.parametrize("n,D", [(14, 70_001), (16, 70_001), (20, 131_100), (34, 70_001), (48, 70_001), (64, 131_100),
                                 (34, 1_001), (48, 1_001), (64, 1_001), (34, 20_001), (48, 20_001), (64, 20_001)])
def test_every_product_of_the_parts_is_there(n, D, layout):
    """All values are a or -a, in every column as many of the one as of the other (so that centring changes
    nothing), with a = 1 + 2^-8 - 2^-17 to the last bits: its parts are 1, 2^-8 and -2^-17, and d2 = 4 a^2
    times the number of columns in which two particles differ.  A missing product of the parts shifts
    d2 by 1.5e-5 (h l or m m) or 8e-3 (h m).  The products of m and l are left out by design, 2^-24 in
    all; as every column contributes the same, roundings at 2^-24 of a 64-column sum add up as well."""
    from paper_2306_06528_amd import svgd
    a = 1.0 + 2.0 ** -8 - 2.0 ** -17 + 3 * 2.0 ** -23
    g = torch.Generator().manual_seed(n)
    order = torch.rand(n, D, generator=g).argsort(0)
    sign = 2.0 * (order < n // 2).float() - 1.0
    diff = (sign[:, None] != sign[None]).sum(-1).numpy() if n <= 20 else \
        np.stack([(sign[i] != sign).sum(-1).numpy() for i in range(n)])
    d2 = 4.0 * a * a * diff
    iu = np.triu_indices(n, 1)
    hf = float(np.median(d2[iu])) / 16.0
    _, K = _pairs(svgd, (a * sign).cuda(), layout, hf)
    got = -hf * np.log(K[iu].astype(np.float64))
    assert np.abs(got / d2[iu] - 1.0).max() <= 4 * 2.0 ** -24
    h, _ = _pairs(svgd, (a * sign).cuda(), layout, 0.0)
    h_ref = float(np.median(d2)) / math.log(n + 1.0)
    assert abs(h - h_ref) <= 4 * 2.0 ** -24 * h_ref


@pytest.mark.parametrize("n,D", [(13, 2_001), (16, 200_001), (33, 200_001), (64, 100_001), (33, 1_001), (48, 20_001), (64, 20_001)])
def test_distances_beside_overflowing_ones(n, D):
    """Two particles lie so far off in one column, on opposite sides, that their squares overflow (their
    mean is that of the others): the distances, kernel values and updates of all other particles are
    what they are without the column's overflow."""
    from paper_2306_06528_amd import svgd
    g = torch.Generator().manual_seed(n)
    Xh, Gh = torch.randn(n, D, generator=g), torch.randn(n, D, generator=g)
    off = np.array([i for i in range(n) if i not in (3, 7)])
    inside = np.ix_(off, off)
    for big in (2.5e19, 1e30):
        Xb = Xh.clone()
        Xb[3, D // 2], Xb[7, D // 2] = big, -big
        d2 = orc.pairwise_d2(Xb.numpy())
        h = float(2 * D)
        X, G = Xb.cuda(), Gh.cuda()
        with svgd.Svgd(n, D) as eng:
            eng.set_bandwidth(h)
            eng.step(X, G, 0.01)
            _, K = eng.get_last(n)
        assert np.abs(K[inside] - np.exp(-d2[inside] / h)).max() <= TOL_K
        assert np.all(K[3, off] == 0.0) and np.all(K[7, off] == 0.0) and K[3, 7] == 0.0
        Kr = np.exp(-d2 / h)
        Kr[[3, 7]] = 0.0
        Kr[:, [3, 7]] = 0.0
        Kr[3, 3] = Kr[7, 7] = 1.0
        x, gr = Xb.double().numpy()[off], Gh.double().numpy()[off]
        Ko = Kr[inside]
        phi = (Ko @ (gr - 2.0 / h * x) + 2.0 / h * Ko.sum(1, keepdims=True) * x) / n
        want = x + float(np.float32(0.01)) * phi
        err = np.abs(X.cpu().double().numpy()[off] - want)
        assert err.max() <= TOL_PHI * 0.01 * np.abs(phi).max() + np.spacing(np.float32(np.abs(x).max()))
