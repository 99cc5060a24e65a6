"""21 to 48 particles and a list of partial sums too long for every workgroup to read: a launch sums it, the update does
pass 2 on the sums.  Sizes at the rule's edges: the shortest such lists and one partial less, columns after the last tile or none,
full and padded blocks of rows, rows on top of them."""
import pytest
import torch

from parity_checks import check_carried_chain, ulp_diff_device

pytestmark = pytest.mark.gpu


def _launches(svgd, eng, call):
    eng.profile_begin()
    call()
    prof = eng.profile_end()
    return [prof[k][1] for k in svgd.KERNEL_KINDS]


# launches of a step: the list read by the update, summed for it, or pass 2 apart (with the list read there or summed before)
ON_LIST, ON_SUMS, APART, APART_ON_SUMS = [1, 0, 0, 1], [1, 1, 0, 1], [1, 0, 1, 1], [1, 1, 1, 1]


@pytest.mark.parametrize("n,D,launches", [
    (22, 70_001, ON_LIST), (23, 49_152, ON_LIST), (23, 49_153, ON_SUMS), (24, 49_150, ON_LIST), (24, 51_203, ON_SUMS), (28, 32_768, ON_LIST), (28, 32_769, ON_SUMS),
    (32, 16_384, ON_LIST), (32, 16_385, ON_SUMS), (32, 52_003, ON_SUMS), (32, 65_536, ON_SUMS),
    (33, 7_500, ON_SUMS), (33, 7_400, APART), (36, 131_072, ON_SUMS), (37, 6_000, ON_SUMS), (44, 70_001, ON_SUMS), (48, 3_400, ON_SUMS),
    (48, 3_300, APART), (48, 65_600, ON_SUMS), (49, 3_400, APART_ON_SUMS)])
def test_pass_2_on_sums(n, D, launches):
    from paper_2306_06528_amd import svgd
    assert torch.cuda.get_device_properties(0).multi_processor_count == 256
    g = torch.Generator().manual_seed(n + D)
    X, G = (0.3 * torch.randn(n, D, generator=g)).cuda(), torch.randn(n, D, generator=g).cuda()
    for padded in (False, True):
        check_carried_chain(svgd, X, G, 0.05, padded=padded, steps=3)
    old, PHI = X.clone(), torch.empty_like(X)
    rows, grows = [X[i].clone() for i in range(n)], [G[i].clone() for i in range(n)]
    with svgd.Svgd(n, D) as eng:
        for call in (lambda: eng.phi(X, G, PHI), lambda: eng.step(X, G, 0.05), lambda: eng.step_rows(rows, grows, 0.05)):
            assert _launches(svgd, eng, call) == launches
            h, K = eng.get_last(n)  # workgroup 0 of the update leaves them, where pass 2 is done there
            assert abs(h - svgd_h(old)) <= 1e-5 * h and float(K[0, 0]) == 1.0
    assert ulp_diff_device(X, old, PHI, 0.05) <= 1.0
    assert ulp_diff_device(torch.stack(rows), old, PHI, 0.05) <= 1.0


@pytest.mark.parametrize("n,D,launches", [(33, 65_407, APART_ON_SUMS), (44, 65_407, APART_ON_SUMS), (44, 65_563, ON_SUMS), (33, 131_070, APART_ON_SUMS), (33, 196_100, ON_SUMS),
                                          (48, 196_100, ON_SUMS), (52, 65_407, APART_ON_SUMS), (64, 131_070, APART_ON_SUMS)])
def test_where_a_worker_less_costs_a_tile(n, D, launches):
    """Just below a multiple of 1,024 tiles of 64 columns (a device of 256 CUs): 256 workers and the tail's workgroup for most plain
    steps with two or three tiles per wave; 255, and pass 2 on the sums, for phi and on carried sums up to 48 particles (dense rows)."""
    from paper_2306_06528_amd import svgd
    g = torch.Generator(device="cuda").manual_seed(n + D)
    X, G = 0.3 * torch.randn(n, D, device="cuda", generator=g), torch.randn(n, D, device="cuda", generator=g)
    old, PHI = X.clone(), torch.empty_like(X)
    inside = ON_SUMS if n <= 48 else APART_ON_SUMS
    with svgd.Svgd(n, D) as eng:
        assert _launches(svgd, eng, lambda: eng.phi(X, G, PHI)) == inside
        assert _launches(svgd, eng, lambda: eng.step(X, G, 0.05)) == launches
        h, K = eng.get_last(n)
        assert abs(h - svgd_h(old)) <= 1e-5 * h
    assert ulp_diff_device(X, old, PHI, 0.05) <= 1.0
    with svgd.Svgd(n, D, flags=svgd.FLAG_CARRY_GRAM) as eng:
        Y = old.clone()
        assert _launches(svgd, eng, lambda: eng.step(Y, G, 0.05)) == inside
        assert _launches(svgd, eng, lambda: eng.step(Y, G, 0.05)) == [0] + inside[1:]
        h, K = eng.get_last(n)
        assert abs(h - svgd_h(X)) <= 1e-5 * h


def svgd_h(X):
    """The median bandwidth in 64 bits."""
    Y = X.double() - X.double().mean(0, keepdim=True)
    S = Y @ Y.t().contiguous()
    s = S.diagonal()
    v = (s[:, None] + s[None, :] - 2.0 * S).clamp_(min=0.0).fill_diagonal_(0.0).flatten().sort().values
    m = v.numel()
    return float(0.5 * (v[(m - 1) // 2] + v[m // 2])) / float(torch.log(torch.tensor(X.shape[0] + 1.0, dtype=torch.float64)))
