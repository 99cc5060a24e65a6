"""Sizes at which the split of the work leaves remainders: the columns after the last full tile of the
matrix-core update (one workgroup, four columns of every sixteenth row per thread, 4 x 4 tiles of pairs for
the carried sums), the last, partly filled round of the streaming moments kernel, and the sizes at which a
rule takes another way: pass 2 inside the update, direct and re-aligned stores, shared ranges."""
import pytest
import torch

from parity_checks import check_carried_chain, ulp_diff_device

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


def _counts(svgd, eng, calls):
    """Launches per kernel kind (gram, reduce, bandwidth, update) that `calls` make."""
    eng.profile_begin()
    calls()
    prof = eng.profile_end()
    return [prof[k][1] for k in svgd.KERNEL_KINDS]


@pytest.mark.parametrize("flags", ["carry", "carry_and_fuse"])
@pytest.mark.parametrize("n,D,fused", [
    (8, 100_003, True), (12, 300_007, True),          # vector ALU: always
    (13, 5_001, True), (16, 8_577, True), (24, 40_003, True), (24, 50_001, "on sums"),
    (32, 12_289, True), (32, 20_001, "on sums"), (33, 5_001, False),
    (16, 300_007, True),                              # 255 workers and the tail's workgroup fill the chip
    (16, 131_100, True), (15, 131_100, True),         # 255 workers with a third tile per wave; 257 workgroups, two a CU
    (20, 131_072, True), (16, 131_072, True),         # no columns after the last tile, no workgroup for them
])
def test_where_pass_2_is_part_of_the_update(n, D, fused, flags):
    """The launches of a plain step, phi, separate rows and a carried step on both sides of the rule that
    makes pass 2 part of the update, on the list or on its sums (a device of 256 CUs), and their results on either side: phi
    and a chain of steps against the oracle.  SVGD_FLAG_FUSE_MFMA changes nothing."""
    from paper_2306_06528_amd import svgd
    assert torch.cuda.get_device_properties(0).multi_processor_count == 256
    g = torch.Generator().manual_seed(n + D)
    X, G = (0.3 * torch.randn(n, D, generator=g)).cuda(), torch.randn(n, D, generator=g).cuda()
    PHI = torch.empty_like(X)
    one = lambda gram: [gram, 0, 0, 1]
    def expect(got, gram):
        if fused == "on sums":
            assert got == [gram, 1, 0, 1]
        elif fused:
            assert got == one(gram)
        else:
            assert got[0] == gram and got[2:] == [1, 1]
    with svgd.Svgd(n, D) as eng:
        expect(_counts(svgd, eng, lambda: eng.phi(X, G, PHI)), 1)
        expect(_counts(svgd, eng, lambda: eng.step(X.clone(), G, 0.05)), 1)
        rows, grows = [X[i].clone() for i in range(n)], [G[i].clone() for i in range(n)]
        expect(_counts(svgd, eng, lambda: eng.step_rows(rows, grows, 0.05)), 1)
    f = svgd.FLAG_CARRY_GRAM | (svgd.FLAG_FUSE_MFMA if flags == "carry_and_fuse" else 0)
    with svgd.Svgd(n, D, flags=f) as eng:
        Xc = X.clone()
        expect(_counts(svgd, eng, lambda: eng.step(Xc, G, 0.05)), 1)
        expect(_counts(svgd, eng, lambda: eng.step(Xc, G, 0.05)), 0)
    if flags == "carry":
        for padded in (False, True):
            check_carried_chain(svgd, X, G, 0.05, padded=padded, steps=3)


# MiB of X up to which rows off the 128-byte boundaries are stored directly, re-aligned above (n <= 16, 32, 48, 64): phi 24,
# 24, 40, 76; a plain step 100 (n = 16: 120), 56, 56, 144; carried sums 92, 92, 92, 256.  Every form of the kernel - padded
# and full blocks of rows, one to four rows on top of them - stores both ways in all three here.
@pytest.mark.parametrize("n,mib", [(13, 24), (14, 100), (14, 184), (15, 92), (16, 120), (16, 184), (16, 92), (18, 92), (20, 24), (24, 56), (26, 92), (32, 92),
                                   (33, 40), (35, 92), (44, 92), (48, 56), (48, 92), (51, 76), (51, 256), (60, 144), (60, 256), (64, 76), (64, 256)])
def test_direct_and_staged_stores(n, mib):
    """One column less and one more than the size at which the stores change, and odd row starts: what both leave
    is the oracle's (through phi of the same sizes), nothing between the rows is touched.  Three carried steps: forwards,
    backwards on the sums of that, forwards on the sums of the walk backwards."""
    from paper_2306_06528_amd import svgd
    D0 = (mib << 20) // (4 * n)
    for D in (D0 - 1, D0 + 1):
        g = torch.Generator(device="cuda").manual_seed(D)
        buf, G = torch.full((n, D + 3), 7.0, device="cuda"), torch.randn(n, D + 3, device="cuda", generator=g)
        X = buf[:, 1:D + 1]
        X.copy_(0.3 * torch.randn(n, D, device="cuda", generator=g))
        old, Gv = X.clone(), G[:, 1:D + 1]
        pbuf = torch.full((n, D + 3), 7.0, device="cuda")
        PHI = pbuf[:, 1:D + 1]
        with svgd.Svgd(n, D) as eng:
            eng.phi(X, Gv, PHI)
            h, K = eng.get_last(n)
            Kd = torch.from_numpy(K).cuda().double()
            ref = Kd @ (Gv.double() - (2.0 / h) * old.double()) / n + (2.0 / h) * Kd.sum(1, keepdim=True) / n * old.double()
            assert float((PHI.double() - ref).abs().max()) <= 1e-5 * float(ref.abs().max())
            eng.step(X, Gv, 0.05)
        assert ulp_diff_device(X, old, PHI, 0.05) <= 1.0
        with svgd.Svgd(n, D, flags=svgd.FLAG_CARRY_GRAM) as eng:
            X.copy_(old)
            eng.step(X, Gv, 0.05)
            assert ulp_diff_device(X, old, PHI, 0.05) <= 1.0
            for _ in range(2):
                now = X.clone()
                with svgd.Svgd(n, D) as plain:
                    plain.phi(X, Gv, PHI)
                eng.step(X, Gv, 0.05)
                assert ulp_diff_device(X, now, PHI, 0.05) <= 1.0
        for b in (buf, pbuf):
            assert bool((b[:, 0] == 7.0).all()) and bool((b[:, D + 1:] == 7.0).all())
        del buf, G, X, Gv, PHI, pbuf, old, now, ref


@pytest.mark.parametrize("D", [65_590, 65_600, 71_700, 71_750, 80_003, 81_660, 81_700, 97_980, 98_000, 98_300, 98_400, 131_100, 135_003, 147_500, 147_600, 196_150])
@pytest.mark.parametrize("n", [49, 52, 53, 64])
def test_direct_stores_in_adjacent_tiles_or_ranges(n, D):
    """More than 48 particles on dense rows at the sizes where the waves of a workgroup stop and start to share a range
    of 64-column tiles (a range of 5, in a plain step 6 tiles for each of 255 workers: not; a device of 256 CUs), or where one worker
    less would give them a tile more: phi, a plain step and carried steps in
    both directions."""
    from paper_2306_06528_amd import svgd
    g = torch.Generator(device="cuda").manual_seed(n + D)
    X, G = 0.3 * torch.randn(n, D, device="cuda", generator=g), torch.randn(n, D, device="cuda", generator=g)
    check_carried_chain(svgd, X, G, 0.05, padded=False, steps=3)
    old, PHI = X.clone(), torch.empty_like(X)
    with svgd.Svgd(n, D) as eng:
        eng.phi(X, G, PHI)
        eng.step(X, G, 0.05)
    assert ulp_diff_device(X, old, PHI, 0.05) <= 1.0
