"""How a decode handle divides sequences (csrc/rl_split_rule.h, compiled here with
g++): CPU checks of the rule over every length."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "rl_split_rule.h"
using namespace rl_da;
extern "C" {
int splits_of(int p, int mn, int w, int most, int n) { return SplitRule{p, mn, w, most}.splits_of(n); }
int pages_of(int p, int mn, int w, int most, int n) { return SplitRule{p, mn, w, most}.pages_of(n); }
}
"""

# pages, min_pages, whole, most; pages of the handle's table
RULES = [
    (256, 32, 47, 16, 4096),       # 128 pairs
    (128, 32, 47, 32, 4096),       # 8 pairs: a default split of 2048 tokens
    (256, 32, 47, 16, 8192),       # a table of 131072 tokens
    (256, 256, 0, 16, 4096),       # not by length
]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("rule")
    src, so = str(d / "rule.cpp"), str(d / "rule.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC",
                    "-I", os.path.join(ROOT, "paper_2512_22492_amd", "csrc"), src, "-o", so],
                   check=True)
    return ctypes.CDLL(so)


@pytest.mark.parametrize("rule", RULES)
def test_every_length_is_divided_within_the_partials_of_its_rows(lib, rule):
    """The splits cover the sequence, none is longer than the handle's split
    size, there are no more than a table of that length may have (which sizes a
    launch's partials) and than the handle's rows have; even cuts leave no
    sliver: the last split is shorter by less than a page a split."""
    pages, min_pages, whole, most, table = rule
    slots = (table + pages - 1) // pages
    before = 0
    for n in range(table + 1):
        sp, limit = lib.pages_of(*rule[:4], n), lib.splits_of(*rule[:4], n)
        splits = (n + sp - 1) // sp
        assert 1 <= sp <= pages and splits <= limit <= slots
        assert before <= limit
        before = limit
        if n > whole and min_pages != pages:
            last = n - (splits - 1) * sp
            assert last > sp - splits, n
            assert splits >= 2 and sp >= 2 * min_pages // 3
        else:
            assert sp == pages
