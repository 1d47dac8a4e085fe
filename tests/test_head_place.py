"""Which workgroup makes which part of which head's output row, compiled by itself."""
import shutil
import subprocess

import numpy as np
import pytest

from paper_2506_15704_amd import build

MAIN = r"""
#include <cstdio>
#include "head_place.h"
using namespace lfps;
template <int kParts>
void all(int requests, int kv_heads, int heads) {
  const int blocks = attend_blocks_for(requests * kv_heads, heads, kParts);
  for (int i = 0; i < blocks; ++i) {
    const HeadPlace p = place_of_block_for<kParts>(requests, kv_heads, heads, (uint32_t)i);
    if (!p.none) printf("%d %d %d %d %d %d %d\n", i, p.bg, p.b, p.g, p.bh, p.in_group, p.part);
  }
}
int main(int n, char** v) {
  if (n == 3) {                      // heads, are the values on the device?
    int heads, on;
    sscanf(v[1], "%d", &heads);
    sscanf(v[2], "%d", &on);
    printf("%d\n", attend_parts_for(heads, on));
    return 0;
  }
  int x[4];
  for (int i = 0; i < 4; ++i) sscanf(v[i + 1], "%d", x + i);
  if (x[3] == 4) all<4>(x[0], x[1], x[2]);
  else all<1>(x[0], x[1], x[2]);
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    where = tmp_path_factory.mktemp("place")
    (where / "main.cpp").write_text(MAIN)
    compiler = shutil.which("g++") or build.hipcc()
    subprocess.run([compiler, "-std=c++17", "-O1", "-I", build.CSRC, str(where / "main.cpp"), "-o", str(where / "place")], check=True)
    return str(where / "place")


@pytest.mark.parametrize("B,Hkv,G,parts", [(1, 8, 4, 4), (1, 4, 4, 4), (1, 12, 4, 4), (1, 1, 1, 4), (3, 3, 2, 4), (3, 8, 2, 4), (15, 1, 4, 4),
                                           (7, 8, 1, 4), (1, 2, 4, 4), (16, 8, 4, 1), (5, 3, 4, 1), (9, 8, 2, 1), (3, 5, 1, 1)])
def test_every_part_once_and_a_groups_parts_on_one_xcd(program, B, Hkv, G, parts):
    res = subprocess.run([program] + [str(x) for x in (B, Hkv, G, parts)], capture_output=True, text=True, check=True)
    got = np.array([[int(x) for x in line.split()] for line in res.stdout.splitlines()])
    block, bg, b, g, bh, in_group, part = got.T
    assert sorted(zip(bh, part)) == [(h, p) for h in range(B * Hkv * G) for p in range(parts)]
    assert (bg == bh // G).all() and (b == bg // Hkv).all() and (g == bg % Hkv).all() and (in_group == bh % G).all()
    if parts > 1 or B * Hkv % 8 == 0:
        for x in range(B * Hkv):
            assert len(set(block[bg == x] % 8)) == 1, x            # (workgroup i runs on XCD i % 8)
        per_xcd = np.bincount(block % 8, minlength=8)
        assert parts == 1 or per_xcd.max() <= 32                       # a CU for each


def test_values_in_host_memory_have_one_workgroup_a_head(program):
    def parts(heads, on_device):
        return int(subprocess.run([program, str(heads), str(int(on_device))], capture_output=True, text=True, check=True).stdout)
    assert [parts(h, True) for h in (1, 64, 65, 4096)] == [4, 4, 1, 1]
    assert [parts(h, False) for h in (1, 64, 65)] == [1, 1, 1]
