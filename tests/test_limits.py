"""The limits of a work plan (cvo_limits.hpp), on the host: totals are compared
in 64 bits, so a plan whose slots pass 2^32 is refused and not taken for its
remainder."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "cvo_limits.hpp"
int main(int argc, char **argv)
{
    if (argc == 2) {  // costs on standard input, their buckets on standard output
        unsigned long long cost;
        while (scanf("%llu", &cost) == 1) printf("%d\n", cvo::cost_bucket(cost));
        return 0;
    }
    const unsigned long long pieces = strtoull(argv[1], nullptr, 10), slots = strtoull(argv[2], nullptr, 10);
    // a place among the points of both sides, counted up as the sort's passes do
    cvo::SortPlace place = (cvo::SortPlace)(cvo::kMaxSidePoints - 1);
    place += (cvo::SortPlace)(cvo::kMaxSidePoints - 1);
    printf("%d %d %llu\n", (int)cvo::plan_fits(pieces, slots), (int)cvo::joint_fits(slots, strtoull(argv[3], nullptr, 10)),
           (unsigned long long)place);
}
"""


@pytest.fixture(scope="module")
def fits(tmp_path_factory):
    d = tmp_path_factory.mktemp("limits")
    (d / "limits.cpp").write_text(PROGRAM)
    exe = str(d / "limits")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2012_03683_amd", "csrc"),
                    str(d / "limits.cpp"), "-o", exe], check=True)

    def call(pieces, slots=0, bytes_per_slot=60):
        if isinstance(pieces, list):
            out = subprocess.run([exe, "buckets"], input=" ".join(map(str, pieces)), check=True, capture_output=True,
                                 text=True).stdout
            return [int(b) for b in out.split()]
        out = subprocess.run([exe, str(pieces), str(slots), str(bytes_per_slot)], check=True, capture_output=True,
                             text=True).stdout.split()
        return out[0] == "1", out[1] == "1", int(out[2])
    return call


def _plan(n_ref, n_query, cluster=16, least=512, most=4096):
    """Pieces and slots of a plan without a cutoff: every cluster has every reference point."""
    clusters = -(-n_query // cluster)
    pieces = min(-(-n_ref // least), most)
    return clusters * pieces, n_query * pieces


@pytest.mark.parametrize("n,ok", [(1000, True), (1_000_000, True), (1_048_000, True), (1_049_000, False),
                                  (1_500_000, False), (4_000_000, False)])
def test_plan_without_cutoff(fits, n, ok):
    pieces, slots = _plan(n, n)
    assert (slots < 2 ** 31) == ok
    assert fits(pieces, slots)[0] == ok


def test_totals_are_not_taken_modulo(fits):
    pieces, slots = _plan(1_500_000, 1_500_000)
    assert slots == 4_395_000_000 and slots % 2 ** 32 < 2 ** 31  # (32 bits of it would pass)
    assert not fits(pieces, slots)[0]
    # three plans that fit one by one, and whose sum passes 2^32
    one = _plan(860_000, 860_000)
    assert fits(*one)[0] and not fits(3 * one[0], 3 * one[1])[0]


@pytest.mark.parametrize("slots,bytes_per_slot,ok", [(0, 60, True), (2 ** 26, 64, True), (2 ** 26 + 1, 64, False),
                                                     (2 ** 31 - 1, 2, True), (2 ** 31, 1, False),
                                                     (2 ** 62 + 1, 4, False)])
def test_joint_plan(fits, slots, bytes_per_slot, ok):
    assert fits(0, slots, bytes_per_slot)[1] == ok


def test_places_of_both_sides(fits):
    """The last place of a call with as many points as each side may have."""
    assert fits(0, 0)[2] == 2 * (2 ** 31 - 1)


def test_cost_buckets(fits):
    """Non-decreasing and within the table; steps of 96 for every piece of the default
    plan; above, costs a quarter apart are told apart up to the largest there is."""
    top = 64 * (2 ** 30 + 64)
    costs = sorted(set(list(range(0, 40_000, 7)) + [36_864, 36_865] + [int(36_864 * 1.1 ** k) for k in range(150)] + [top]))
    costs = [c for c in costs if c <= top]
    b = fits(costs)
    assert all(x <= y for x, y in zip(b, b[1:])) and b[0] == 0 and b[-1] < 512
    assert all(x == c // 96 for c, x in zip(costs, b) if c <= 36_864)
    above = [36_865 * 5 ** k // 4 ** k for k in range(64) if 36_865 * 5 ** k // 4 ** k <= top]
    u = fits(above)
    assert len(above) > 60 and all(x < y for x, y in zip(u, u[1:]))
