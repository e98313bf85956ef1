"""When assignments go by groups of centroids: the rule of csrc/group_cost.hpp, compiled for the host, at what was measured on both sides.  A
group's members are read for every vector by itself, so groups of many members are dearer than comparing with every centroid."""
import ctypes
import pathlib
import shutil
import subprocess

import pytest

CSRC = pathlib.Path(__file__).resolve().parent.parent / "paper_2210_15748_amd" / "csrc"
SOURCE = """
#include "group_cost.hpp"
extern "C" int pays(uint32_t groups, uint32_t easy, uint32_t members, uint32_t K) {
    dessert::GroupCtl c{};
    c.groups = groups;
    c.easy = easy;
    c.members = members;
    return dessert::groups_pay(c, K);
}
extern "C" int hopeless(uint32_t led, uint32_t alone) { return dessert::groups_hopeless(led, alone); }
extern "C" uint32_t largest(uint32_t K) { return dessert::groups_largest(K); }
extern "C" uint32_t room(uint32_t K) { return dessert::groups_room(K); }
"""
TRIAL = 4096


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    d = tmp_path_factory.mktemp("groups")
    (d / "rule.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-O1", "-shared", "-fPIC", "-I", str(CSRC), str(d / "rule.cpp"), "-o", str(d / "rule.so")],
                   check=True)
    return ctypes.CDLL(str(d / "rule.so"))


# centres of the mixture, share of the vectors that need one group; time by groups / by all centroids
@pytest.mark.parametrize("K,groups,easy,pays", [
    (16384, 64, 1.0, False),       # 1.24: 256 members to a vector
    (8192, 64, 1.0, False),        # 1.38: 128
    (16384, 128, 1.0, True),       # 0.60
    (16384, 1024, 0.98, True),     # 0.36
    (16384, 4096, 0.95, True),     # 0.57
    (8192, 4096, 0.95, False),     # more groups than are made
    (16384, 1024, 0.02, False),    # nearly every vector left over
    (16384, 1, 1.0, False),        # one group of everything
    (1 << 20, 1000, 1.0, True),    # the largest: nothing overflows
    (1 << 20, 50, 1.0, False),
    (1 << 20, 300_000, 1.0, True),
])
def test_where_groups_pay(rule, K, groups, easy, pays):
    count = int(easy * TRIAL)
    assert bool(rule.pays(groups, count, count * (K // groups), K)) == pays


@pytest.mark.parametrize("K", [4096, 16384, 1 << 20])
def test_a_group_never_costs_a_vector_more_than_every_centroid(rule, K):
    m = rule.largest(K)
    assert 56 * m <= 80 * m <= 1.1 * K
    assert TRIAL * m < 1 << 32
    assert not rule.pays(0, TRIAL, 0, K) and not rule.pays(rule.room(K) + 1, TRIAL, TRIAL, K)


def test_when_leaders_are_not_looked_for(rule):
    assert not rule.hopeless(0, 0)                                            # nothing known: fewer centroids than GROUP_MANY
    assert rule.hopeless(8192, 8192) and rule.hopeless(4096, 4096 * 2 // 5)   # 1.24 of the time, see group_cost.hpp
    assert not rule.hopeless(8192, 8192 // 4)
