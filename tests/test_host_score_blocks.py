"""How many documents a workgroup of the mask-table kernels takes: the rule of csrc/score_blocks.hpp, compiled for the host.  Whole rounds
over the chip only where they were measured to pay: not for tables that are small against the rows they are read with, nor for query sets
of unequal numbers of chunks, nor for documents of one length unless the tables are a good part of the work."""
import ctypes
import pathlib
import shutil
import subprocess

import pytest

CSRC = pathlib.Path(__file__).resolve().parent.parent / "paper_2210_15748_amd" / "csrc"
SOURCE = """
#include "score_blocks.hpp"
extern "C" uint32_t docs(uint64_t n, uint64_t gy, uint64_t slots, uint64_t most, uint32_t least) { return dessert::whole_round_docs(n, gy, slots, most, least); }
extern "C" int pays(uint64_t table, uint64_t code, int equal_docs, int equal_sets, int any) { return dessert::whole_rounds_pay(table, code, equal_docs, equal_sets, any); }
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    d = tmp_path_factory.mktemp("blocks")
    (d / "rule.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-O1", "-shared", "-fPIC", "-I", str(CSRC), str(d / "rule.cpp"), "-o", str(d / "rule.so")],
                   check=True)
    lib = ctypes.CDLL(str(d / "rule.so"))
    lib.docs.argtypes = [ctypes.c_uint64] * 4 + [ctypes.c_uint32]
    lib.docs.restype = ctypes.c_uint32
    lib.pays.argtypes = [ctypes.c_uint64] * 2 + [ctypes.c_int] * 3
    return lib


def table(L, C, sets=1):
    return (L << C) * 4 * sets


# (L, C, sets per workgroup, documents of a halved block, their mean length, bytes of a code, one length, sets of equal chunks, the kernel for
# any number of tables): measured with whole rounds / without
@pytest.mark.parametrize("L,C,sets,block,length,width,equal_docs,equal_sets,any_tables,pays", [
    (64, 9, 1, 128, 137, 2, True, True, True, False),      # 1.50
    (48, 4, 1, 64, 70, 1, False, True, True, False),       # 1.35
    (40, 6, 1, 32, 298, 1, True, False, True, False),      # 1.28
    (40, 5, 1, 64, 70, 1, True, True, True, False),        # 1.26
    (24, 6, 1, 64, 70, 1, False, True, True, False),       # 1.13
    (64, 6, 2, 64, 70, 1, True, True, False, False),       # 1.19
    (16, 6, 2, 128, 70, 1, False, False, False, False),    # 1.12
    (32, 7, 1, 64, 70, 1, False, True, True, True),        # 0.82
    (32, 7, 2, 64, 70, 1, False, True, False, True),       # 0.82
    (128, 6, 1, 64, 8, 1, True, True, False, True),        # 0.7
])
def test_where_whole_rounds_pay(rule, L, C, sets, block, length, width, equal_docs, equal_sets, any_tables, pays):
    assert bool(rule.pays(table(L, C, sets), block * length * L * width, equal_docs, equal_sets, any_tables)) == pays


@pytest.mark.parametrize("most,least", [(256, 64), (512, 128), (256, 128)])
@pytest.mark.parametrize("n", [64, 1000, 20_000, 123_457, 10_000_000])
@pytest.mark.parametrize("gy", [1, 3, 37, 300, 65_535])
@pytest.mark.parametrize("slots", [32, 160, 224])
def test_blocks_make_whole_rounds(rule, n, gy, slots, most, least):
    d = rule.docs(n, gy, slots, most, least)
    assert least <= d <= most
    # an XCD takes every 8th block, and all gy groups of it
    workgroups = lambda d: (-(-n // d) + 7) // 8 * gy
    rounds = -(-workgroups(d) // slots)
    if d > least:                                    # no smaller block fits the same rounds
        assert -(-workgroups(d - 1) // slots) > rounds
