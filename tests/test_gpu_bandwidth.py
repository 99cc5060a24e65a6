"""Pass 2 (bandwidth and kernel matrix) where its rule can go wrong: the median of sets that are all
equal, that crowd into one bucket of the selection, or that hold infinities, at the particle counts
where the way it is computed changes - by the kernel of its own (svgd_bandwidth) and as the prologue
of the update (svgd_step, which up to 48 particles derives h and K in every workgroup, from the list of partial sums or,
from 21 on where that is long, from what a launch in between has made of it)."""
import numpy as np
import pytest
import torch

from oracle import svgd_oracle as orc
from parity_checks import TOL_H, TOL_K

pytestmark = pytest.mark.gpu


def _particles(kind, n, D):
    g = torch.Generator().manual_seed(97 * n + D)
    X = torch.zeros(n, D)
    if kind == "equal":            # every distance the same
        X[torch.arange(n), torch.arange(n)] = 1.5
    elif kind == "crowded":        # two far outliers; all other distances within 1/256 of the range
        X[torch.arange(n), torch.arange(n)] = 1.0 + 1e-3 * torch.rand(n, generator=g)
        X[0, 0], X[n - 1, n - 1] = 40.0, 25.0
    elif kind == "infinite":       # one particle so far off that its squared distances overflow
        X = torch.randn(n, D, generator=g)
        X[n // 2] = 1e30
    else:
        X = torch.randn(n, D, generator=g)
    return X


@pytest.mark.parametrize("kind", ["equal", "crowded", "random"])
@pytest.mark.parametrize("n", [2, 8, 9, 11, 12, 13, 16, 17, 32, 33, 64])
def test_median_of_awkward_sets(n, kind):
    _check(n, 3001, kind)


@pytest.mark.parametrize("kind", ["equal", "crowded", "random"])
@pytest.mark.parametrize("n,D", [(24, 52_003), (32, 16_387), (33, 8_001), (36, 8_001), (44, 6_001), (48, 6_001)])
def test_median_of_awkward_sets_on_sums(n, D, kind):
    """256 threads and up to five pairs each: the refining levels of the selection, and a fixed bandwidth."""
    _check(n, D, kind, launches=[1, 1, 0, 1])
    _check(n, D, kind, launches=[1, 1, 0, 1], fixed=2.0 * D if kind == "random" else 2.5)


@pytest.mark.parametrize("n,D", [(4, 100), (8, 3001)])   # direct differences: infinite d2, not inf - inf
def test_median_with_infinite_distances(n, D):
    _check(n, D, "infinite")


@pytest.mark.parametrize("n,D", [(13, 2001), (16, 200_001), (33, 200_001), (64, 100_001), (33, 1001), (48, 20_001), (64, 20_001)])
def test_pair_sums_that_overflow(n, D):
    """One particle is far enough off in one column for its squares to overflow fp32 sums, at both ends of
    the range where products of its parts overflow to different signs.  The pair sums then have to be
    those of the fp32 products: infinite distances to that particle (K exactly 0), never NaN."""
    from paper_2306_06528_amd import svgd
    for big in (2.5e19, 1e30):
        X = torch.randn(n, D, generator=torch.Generator().manual_seed(n)).cuda()
        X[3, D // 2] = big
        G = torch.randn(n, D, device="cuda")
        with svgd.Svgd(n, D) as eng:
            eng.set_bandwidth(float(2 * D))
            eng.bandwidth(X)
            h, K = eng.get_last(n)
            assert np.isfinite(K).all() and np.all(np.diag(K) == 1.0) and np.array_equal(K, K.T)
            off = np.arange(n) != 3
            assert np.all(K[3, off] == 0.0)
            eng.step(X, G, 1e-3)
            assert bool(torch.isfinite(X[torch.tensor(off)]).all())


@pytest.mark.parametrize("n,D", [(4, 100), (8, 3001), (16, 3001), (33, 3001)])
def test_equal_particles_under_a_tiny_fixed_bandwidth(n, D):
    """K = exp(-d2 / h) of equal particles is 1 at every h, also where 1 / h overflows; of others it is 0."""
    from paper_2306_06528_amd import svgd
    X = torch.randn(n, D, generator=torch.Generator().manual_seed(n))
    X[1] = X[n - 1]
    want = np.eye(n, dtype=np.float32)
    want[1, n - 1] = want[n - 1, 1] = 1.0
    with svgd.Svgd(n, D) as eng:
        for h in (1e-300, 1e-310, 5e-324):
            eng.set_bandwidth(h)
            eng.bandwidth(X.cuda())
            got_h, K = eng.get_last(n)
            assert got_h == h and np.array_equal(K, want), h



# The list of partial sums (one per 1,024 columns up to 12 particles, one per 256 above) is summed in shares of KL
# partials, four at a time.  svgd_bandwidth: KL = 32 up to 12 particles, 30 at 16, 13 at 24; the update: 11 at
# 13, 7 at 16, 4 at 20, 3 at 24.
@pytest.mark.parametrize("n,nparts", [(n, k) for n, KL in ((2, 32), (8, 32), (13, 11), (16, 7), (16, 30), (20, 4), (24, 3), (24, 13))
                                      for k in sorted({4 * KL, 4 * KL + 1, 8 * KL, 8 * KL + 1, 12 * KL + 1, 16 * KL, 16 * KL + 1})
                                      if k <= (768 if n <= 12 else 256)])
def test_lists_around_a_share_of_the_partials(n, nparts):
    per = 1024 if n <= 12 else 256
    _check(n, per * nparts - 3, "random")


def _check(n, D, kind, launches=None, fixed=0.0):
    from paper_2306_06528_amd import svgd
    Xh = _particles(kind, n, D)
    if fixed:
        d2 = orc.pairwise_d2(Xh.numpy())
        K_ref, _ = orc.kernel(d2, fixed)
        ref = {"h": fixed, "K": K_ref}
    else:
        ref = orc.step(Xh.numpy(), np.zeros((n, D), np.float32), 0.0, want_phi=False, want_xnew=False)
    X, G = Xh.cuda(), torch.zeros(n, D, device="cuda")
    with svgd.Svgd(n, D) as eng:
        eng.set_bandwidth(fixed)
        eng.bandwidth(X)
        got = [eng.get_last(n)]
        if launches:
            eng.profile_begin()
        eng.step(X, G, 0.0)
        if launches:
            prof = eng.profile_end()
            assert [prof[k][1] for k in svgd.KERNEL_KINDS] == launches
        got.append(eng.get_last(n))
    for h, K in got:
        assert abs(h - ref["h"]) <= TOL_H * ref["h"]
        assert np.abs(K - ref["K"]).max() <= TOL_K
        assert np.array_equal(K, K.T) and np.all(np.diag(K) == 1.0)
