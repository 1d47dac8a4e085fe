"""The rule that cuts a context's rows into the ranges of the range kernel, compiled by itself: what the kernel needs of a range, over
the contexts that it admits, and where its lines lie."""
import os
import shutil
import subprocess

import pytest

from paper_2506_15704_amd import build

MAIN = r"""
#include <cstdio>
#include "range_rule.h"
int main() {
  long long groups; int rows, heads, tables;
  while (scanf("%lld %d %d %d", &groups, &rows, &heads, &tables) == 4)
    printf("%d\n", lfps::range_rows_for(groups, rows, heads, tables != 0));
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    where = tmp_path_factory.mktemp("rule")
    (where / "main.cpp").write_text(MAIN)
    compiler = shutil.which("g++") or build.hipcc()
    subprocess.run([compiler, "-std=c++17", "-O1", "-I", build.CSRC, str(where / "main.cpp"), "-o", str(where / "rule")], check=True)

    def ask(cases):
        text = "\n".join(" ".join(str(int(x)) for x in c) for c in cases)
        res = subprocess.run([str(where / "rule")], input=text, capture_output=True, text=True, check=True)
        return [int(x) for x in res.stdout.split()]
    return ask


def test_ranges_are_what_the_kernel_can_take(rule):
    rows = sorted({x + d for e in range(21) for x in (1 << e, 3 << e) for d in (-65, -1, 0, 1, 63) if 0 < x + d <= 88 * 1024 * 8})
    cases = [(g, n, h, t) for g in list(range(1, 70)) + [127, 128, 200, 341, 342, 512, 513, 700, 1023, 1024, 1025, 4096, 16383]
             for n in rows for h in (1, 2, 4) for t in (0, 1)]
    for (groups, n, heads, tables), r in zip(cases, rule(cases)):
        admitted = groups * n <= (4 << 20 if tables else 1 << 20)
        assert admitted or r == 0, (groups, n, heads, tables)
        if r == 0:
            assert not admitted or n > 256 * 8192, (groups, n, heads, tables)
            continue
        assert r % 64 == 0 and 64 <= r <= 8192, (groups, n, heads, tables, r)
        assert -(-n // r) <= 256, (groups, n, heads, tables, r)             # four pieces each, 1024 per head


def test_one_range_per_group_where_it_is_the_faster_form(rule):
    # table form: (groups, rows, heads per group, ranges of a group)
    cases = [(520, 8009, 4, 3), (704, 5909, 4, 3), (600, 6909, 4, 3), (600, 5009, 4, 2), (1000, 4159, 4, 2), (800, 3659, 4, 1),
             (600, 6909, 1, 1), (520, 8009, 2, 1), (360, 11509, 4, 2), (64, 65509, 4, 16), (64, 32777, 4, 16), (64, 30000, 4, 15),
             (1024, 4009, 4, 1)]
    got = rule([(g, n, h, 1) for g, n, h, _ in cases])
    assert [-(-n // r) for (_, n, _, _), r in zip(cases, got)] == [c[3] for c in cases]
    # from the Top-k
    cases = [(200, 5195, 4, 5), (72, 14505, 4, 14), (600, 1395, 4, 1), (64, 16384, 4, 16), (8, 32773, 4, 33)]
    got = rule([(g, n, h, 0) for g, n, h, _ in cases])
    assert [-(-n // r) for (_, n, _, _), r in zip(cases, got)] == [c[3] for c in cases]


def test_the_contexts_of_the_gpu_tests_take_the_ranges_they_are_for(rule):
    # tests/test_gpu_ranges.py, test_ranges_that_are_no_power_of_two and test_one_range_per_group: (groups, max_seq_len, heads per
    # group, tables)
    cases = [(25 * 8, 5200, 1, 0), (43 * 8, 4108, 1, 1), (65 * 8, 5008, 1, 1), (65 * 8, 5008, 4, 1)]
    assert rule(cases) == [1088, 2112, 5056, 2560]
