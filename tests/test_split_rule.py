"""How a decode handle divides sequences and in which order a launch takes the
units (csrc/rl_split_rule.h, compiled here with g++): CPU checks of the rule and
of the plan's entries over every length."""
import ctypes
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "rl_split_rule.h"
using namespace rl_da;
extern "C" {
int splits_of(int p, int mn, int w, int most, int n) { return SplitRule{p, mn, w, most}.splits_of(n); }
int pages_of(int p, int mn, int w, int most, int n) { return SplitRule{p, mn, w, most}.pages_of(n); }
void shape(int p, int mn, int w, int most, int n, int* out)
{
    const PlanShape s(SplitRule{p, mn, w, most}, n);
    out[0] = s.pages; out[1] = s.full; out[2] = s.full_cls; out[3] = s.last_cls;
}
int pack(int b, int pages, int split) { return pack_entry(b, pages, split); }
void unpack(int e, int* out) { unpack_entry(e, out[0], out[1], out[2]); }
int classes() { return kLengthClasses; }
int batch_limit() { return kPlanBatchByLength; }
int split_limit() { return kPlanSplitsByLength; }
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


def shape(lib, rule, n):
    out = (ctypes.c_int * 4)()
    lib.shape(*rule[:4], n, out)
    return list(out)


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


@pytest.mark.parametrize("rule", RULES[:3])
@pytest.mark.parametrize("seed", range(6))
def test_units_go_longest_first(lib, rule, seed):
    """A plan by length takes its entries by class: no unit is longer than one
    taken before it by more than a class (an eighth of the handle's split), full
    splits of shorter sequences and whole sequences in between included, and
    every split of every sequence is taken once."""
    rng = random.Random(seed)
    table = rule[4]
    lengths = [rng.choice([0, 1, rng.randint(1, table), rng.randint(1, table // 8),
                           int(table ** rng.random())]) for _ in range(rng.choice([3, 40, 300]))]
    entries = []
    for b, n in enumerate(lengths):
        sp, full, full_cls, last_cls = shape(lib, rule, n)
        assert sp == lib.pages_of(*rule[:4], n)
        assert 0 <= full_cls < lib.classes() and 0 <= last_cls < lib.classes()
        if full:
            entries.append((full_cls, b, sp, 0, full))
        entries.append((last_cls, b, sp, full, 1))
    units = []
    for cls, b, sp, first, count in sorted(entries, key=lambda e: e[0]):  # stable
        for s in range(first, first + count):
            units.append((b, s, min(sp, lengths[b] - s * sp)))
    taken = {(b, s) for b, s, _ in units}
    assert len(taken) == len(units)
    assert taken == {(b, s) for b, n in enumerate(lengths)
                     for s in range(max(1, -(-n // lib.pages_of(*rule[:4], n))))}
    shortest = rule[0]
    for b, s, size in units:
        assert size <= shortest + (rule[0] + 1) / lib.classes() + 1, (b, s)
        shortest = min(shortest, size)


def test_entries_round_trip(lib):
    out = (ctypes.c_int * 3)()
    for b in (0, 1, 255, lib.batch_limit() - 1):
        for pages in (1, 2, 33, 255, 256):
            for split in (0, 1, 15, lib.split_limit() - 1):
                lib.unpack(lib.pack(b, pages, split), out)
                assert list(out) == [b, pages, split]
