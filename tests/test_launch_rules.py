"""How the matrix-core update's work is split, as far as numbers decide it: compiled for the host and asked."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CUS = 256

PROGRAM = r"""
#include <cstdio>
#include "launch_rules.hpp"
int main()
{
    long long n, D;
    int aligned, emit, carry;
    while (std::scanf("%lld %lld %d %d %d", &n, &D, &aligned, &emit, &carry) == 5) {
        const bool room = svgd::leaves_room_for_tail((int)n, D, 256, aligned, emit, carry);
        const long long workers = 256 - room, per = (D / 64 + workers - 1) / workers;
        // workers of an update that reads a long list, with direct stores and without; and those that the pairwise pass
        // before it reckons with (which knows nothing of the two)
        const bool beyond = 4 * n * D > (320ll << 20);
        std::printf("%d %lld %d %d %d %d\n", room, (long long)svgd::tiles_per_wave(D / 64, workers), svgd::own_ranges(per, emit, carry),
                    svgd::long_list_workers((int)n, D, 256, 2048, beyond, aligned, true, emit, carry),
                    svgd::long_list_workers((int)n, D, 256, 2048, beyond, aligned, false, emit, carry),
                    svgd::long_list_workers((int)n, D, 256, 2048, beyond, aligned, false, false, carry));
    }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not installed")
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(PROGRAM)
    csrc = os.path.join(HERE, "..", "paper_2306_06528_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-I", csrc, "-o", str(d / "rules"), str(d / "rules.cpp")], check=True, timeout=120)

    def ask(cases):
        text = "".join("%d %d %d %d %d\n" % c for c in cases)
        out = subprocess.run([str(d / "rules")], input=text, capture_output=True, text=True, check=True, timeout=120).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return ask


# (rows on 128-byte boundaries, phi written out, carried sums)
STEP, PHI, CARRY, STEP_PADDED, PHI_PADDED, CARRY_PADDED = KINDS = [(a, e, c) for a in (0, 1) for e, c in ((0, 0), (1, 0), (0, 1))]


def test_a_worker_less_gives_no_wave_a_tile_more_unless_measured_to_be_faster(rules):
    cases = [(n, 64 * t + 1, *k) for n in range(13, 65) for t in [*range(1, 4200, 5), *range(1000, 16500, 61), *(1024 * k + d for k in range(1, 16) for d in range(-17, 2))]
             for k in KINDS]
    whole = lambda n: n > 32 or n % 16 == 0 or (n > 16 and 1 <= n % 16 <= 4)
    seen = 0
    for (n, D, a, e, c), (room, tiles, *_) in zip(cases, rules(cases)):
        t = D // 64
        before, after = -(-t // (4 * CUS)), -(-t // (4 * (CUS - 1)))
        assert tiles == (after if room else before)
        per = -(-t // CUS)
        if not whole(n) or t > 16 * 4 * CUS or (n > 48 and (a or c) and 8 * -(-t // per) <= 7 * CUS):
            assert not room
        elif before == after:
            assert room
        elif room:
            seen += 1
            assert c or n <= 48  # carried sums, or a launch less
            assert after <= (16 if n <= 36 else 5)
    assert seen


@pytest.mark.parametrize("n,tiles,kind,room", [
    # measured to be slower with a tile more, or with nothing to make room for, by 2 to 13 %
    (33, 1021, STEP_PADDED, False), (48, 1022, STEP_PADDED, False), (48, 1022, PHI_PADDED, False), (44, 1023, STEP, False), (44, 2048, STEP_PADDED, False),
    (48, 1024, STEP_PADDED, False), (44, 2046, PHI, False), (40, 6130, PHI_PADDED, False), (33, 12_270, CARRY_PADDED, False), (40, 8180, CARRY_PADDED, False), (50, 2046, STEP, False), (52, 1021, STEP, False),
    (50, 1093, STEP_PADDED, False), (64, 1120, STEP_PADDED, False), (52, 2048, PHI_PADDED, False), (52, 4092, CARRY, False), (64, 1022, STEP_PADDED, False), (64, 3064, PHI, False),
    # and faster all the same
    (32, 1021, CARRY, True), (33, 1022, PHI, True), (44, 1022, PHI_PADDED, True), (33, 3068, STEP, True), (48, 3068, STEP, True), (48, 2046, STEP, True),
    (50, 1150, STEP_PADDED, True), (64, 1121, CARRY_PADDED, True), (48, 4090, STEP, True), (48, 2046, CARRY, True), (64, 1024, CARRY, True), (64, 2046, CARRY_PADDED, True), (33, 8180, STEP_PADDED, True), (44, 1024, STEP, True)])
def test_where_a_worker_less_costs_a_tile(rules, n, tiles, kind, room):
    assert rules([(n, 64 * tiles + 27, *kind)])[0][0] == room


def test_nothing_is_left_out_without_a_tail(rules):
    assert all(not room for room, *_ in rules([(n, 64 * t, *k) for n in (16, 33, 64) for t in (1019, 1024, 3000) for k in KINDS]))


@pytest.mark.parametrize("tiles,tail,step,phi", [
    (1024, 27, False, False),  # four per workgroup, 256 workers
    (1025, 27, True, True), (1275, 27, True, True), (1276, 27, True, False), (1281, 27, True, False), (1530, 27, True, False), (1531, 27, False, False), (1535, 27, False, False),
    (2048, 27, False, False), (2049, 27, False, False), (2295, 27, False, False),
    (1280, 0, True, True), (1281, 0, True, False), (1536, 0, True, False), (1537, 0, False, False), (2049, 0, False, False)])
def test_ranges_of_their_own_by_the_workers_that_are_launched(rules, tiles, tail, step, phi):
    """Above 48 particles: five tiles per workgroup, in a plain step six; never on carried sums."""
    D = 64 * tiles + tail
    assert [bool(own) for _, _, own, *_ in rules([(n, D, *k) for n in (49, 56, 64) for k in (STEP, PHI, CARRY)])] == 3 * [step, phi, False]


def test_the_pairwise_pass_reckons_with_the_workers_of_the_update(rules):
    """An X larger than twice the memory-side cache: the pass visits the first tiles of the update's ranges last.  (Stores off the
    line boundaries are re-aligned at these sizes.)"""
    cases = [(n, D, *k) for n in range(13, 65) for D in ((1 << 27) // n + 1, 5_000_003, 9_000_003, 11_173_962, 11_173_888) for k in KINDS if n * D > 1 << 27]
    for (n, D, *_), (*_, launched, reckoned) in zip(cases, rules(cases)):
        assert launched == reckoned, (n, D)


def test_pass_2_inside_the_update_only_with_all_workgroups_resident(rules):
    cases = [(n, D, *k) for n in range(13, 49) for D in (70_001, 131_071, 300_007, 5_000_003) for k in KINDS if n <= 20 or k in (STEP_PADDED, PHI_PADDED)]
    for (n, D, *_), (*_, launched, _) in zip(cases, rules(cases)):
        inside = n <= 20 or launched != 256
        whole = n > 32 or n % 16 == 0 or (n > 16 and 1 <= n % 16 <= 4)
        if inside:
            assert launched + 1 <= CUS * (1 if whole else 2), (n, D)
