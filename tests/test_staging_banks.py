"""Distances of staged score rows in LDS (csrc/laq_staging.h) against a model of the banks (no GPU needed)."""
import os
import subprocess

import pytest

MAIN = r"""
#include <cstdio>
#include "laq_staging.h"
using namespace laq;
int main() {
  for (int d = 4; d <= 256; d += 4)
    for (int planes = 1; planes <= 3; planes += 2)
      printf("%d %d %d %d %d %d\n", d, planes, plane_bytes(d), staged_row(d, planes), plane16_bytes(d), staged_row16(d, planes));
  return 0;
}
"""
# lanes of half a wave whose 16-byte reads are worked off together
FIRST = [0, 1, 2, 3, 12, 13, 14, 15, 20, 21, 22, 23, 24, 25, 26, 27]
TOGETHER = [[h + l for l in p] for h in (0, 32) for p in (FIRST, [l for l in range(32) if l not in FIRST])]


def extra_cycles(address):
    """Cycles that a read of 16 bytes per lane, lane l at address(l), takes beyond those of different banks."""
    extra = 0
    for lanes in TOGETHER:
        words = {a for l in lanes for a in range(address(l) // 4, address(l) // 4 + 4)}
        extra += max(sum(w % 64 == b for w in words) for b in range(64)) - 1
    return extra


@pytest.fixture(scope="module")
def rows(repo_root, tmp_path_factory):
    d = tmp_path_factory.mktemp("staging")
    src, exe = d / "staging.cpp", d / "staging"
    src.write_text(MAIN)
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-O1", "-Wall", "-I",
                    os.path.join(repo_root, "paper_2505_20334_amd", "csrc"), "-o", str(exe), str(src)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60, check=True).stdout
    return [tuple(map(int, line.split())) for line in out.splitlines()]


def test_reads_of_staged_rows_are_free_of_bank_conflicts(rows):
    for d, planes, plane, stride, plane16, stride16 in rows:
        assert plane >= 2 * d and plane % 32 == 0 and plane16 >= 2 * d and plane16 % 64 == 0
        assert stride >= planes * plane and stride16 >= planes * plane16 and stride % 16 == 0 and stride16 % 16 == 0
        assert extra_cycles(lambda l: l % 32 * stride + l // 32 * 16) == 0, (d, planes, stride)
        assert extra_cycles(lambda l: l % 16 * stride16 + l // 16 * 16) == 0, (d, planes, stride16)


def test_the_model_finds_conflicts():
    """16 x 16 tiles at an odd number of 16 bytes; every row in the same banks."""
    assert extra_cycles(lambda l: l % 16 * 272 + l // 16 * 16) == 4 and extra_cycles(lambda l: l % 32 * 144 + l // 32 * 16) == 0
    assert extra_cycles(lambda l: l % 16 * 256 + l // 16 * 16) == 4 * 7
