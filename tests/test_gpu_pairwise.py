"""The pairwise pass on the matrix cores where every wave has several slabs (D >= 65,536 on 256 CUs) and the
products are taken from values split into three bf16 parts."""
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
