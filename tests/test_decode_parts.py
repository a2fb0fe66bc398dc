"""How decode attention cuts the caches of a call into parts (csrc/laq_parts.h), against a search one step at a time (no GPU needed)."""
import os
import random
import subprocess

import pytest

MAIN = r"""
#include <cstdio>
#include <vector>
#include "laq_parts.h"
using namespace laq;
int main() {                                            // n, L, columns, budgets -> limit, workgroups, rows of the longest part, most parts of a cache
  int n, L;
  long long columns;
  while (scanf("%d %d %lld", &n, &L, &columns) == 3) {
    std::vector<int32_t> b(n);
    for (int32_t& x : b)
      if (scanf("%d", &x) != 1) return 1;
    const int limit = limit_of_parts(n, L, columns, b.data());
    long long parts = 0;
    int longest = 0, most = 0;
    for (int32_t x : b) {
      const int bk = x < L ? x : L, p = parts_of(bk, limit), each = p == 1 ? bk : even_rows(bk, p);
      if (p > (bk + limit - 1) / limit || (p - 1) * each >= bk) return 2;      // evening out adds no part and leaves none empty
      parts += p;
      if (each > longest) longest = each;
      if (p > most) most = p;
    }
    printf("%d %lld %d %d\n", limit, parts * columns, longest, most);
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def cut(repo_root, tmp_path_factory):
    d = tmp_path_factory.mktemp("parts")
    src, exe = d / "parts.cpp", d / "parts"
    src.write_text(MAIN)
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-O1", "-Wall", "-I",
                    os.path.join(repo_root, "paper_2505_20334_amd", "csrc"), "-o", str(exe), str(src)], check=True)

    def run(calls):
        text = "\n".join("%d %d %d %s" % (len(b), L, c, " ".join(map(str, b))) for b, L, c in calls)
        r = subprocess.run([str(exe)], input=text, capture_output=True, text=True, timeout=60)
        assert r.returncode == 0
        out = [tuple(map(int, line.split())) for line in r.stdout.splitlines()]
        assert len(out) == len(calls)
        return out
    return run


def up(x, step=64):
    return -(-x // step) * step


def even_of(b, columns):
    return max((sum(b) * columns // 768 // 64 + 1) * 64, -(-max(b) // 128))


@pytest.mark.parametrize("b,columns", [([32768] + [64] * 94, 8), ([32768] + [64] * 99, 8), ([8192] + [256] * 94, 8), ([16384] * 4 + [512] * 96, 8),
                                       ([8192] * 4 + [256] * 80, 8), ([2048] + [512] * 95, 8), ([16384] + [128] * 190, 4), ([9000] + [70] * 22, 32)])
def test_a_few_long_caches_among_short_ones_are_cut(cut, b, columns):
    (limit, workgroups, longest, _), = cut([(b, max(b), columns)])
    assert longest <= up(2 * even_of(b, columns)), longest
    assert workgroups < len(b) * columns + 768


@pytest.mark.parametrize("b,columns,limit", [([2048 - 1920 * i // 31 for i in range(32)], 8, 448), ([2048] * 90, 8, 2048), ([200] * 90, 8, 200),
                                             ([2048] * 100, 8, 2048), ([2048 - 1920 * i // 119 for i in range(120)], 8, 2048),
                                             ([64] * 127 + [9000], 8, 9000)])
def test_lengths(cut, b, columns, limit):
    # the pyramid's; caches that are enough workgroups whole, or nearly; from 1024 workgroups on all stay whole
    assert cut([(b, max(b), columns)])[0][0] == limit


def test_against_a_search_step_by_step(cut):
    rng = random.Random(11)
    calls = []
    for _ in range(3000):
        n, columns, top = rng.randint(1, 140), rng.choice([1, 2, 4, 7, 8, 16, 32]), rng.choice([65, 300, 2048, 9000, 40000])
        if n * columns >= 1024:
            n = max(1, 1023 // columns)
        kind = rng.random()
        b = [rng.randint(1, top) if kind < 0.5 else int(top ** rng.random()) for _ in range(n)] if kind < 0.8 else [top] * n
        calls.append((b, max(b), columns))

    def parts_of(bk, limit):
        steps = up(bk) // 64
        return -(-steps // -(-steps // -(-bk // limit)))

    for (b, L, columns), (limit, workgroups, longest, parts) in zip(calls, cut(calls)):
        most, even = max(b), even_of(b, columns)
        if even >= most:
            want = most
        else:
            top = min(2 * even, most)
            lengths = [] if len(b) * columns > 768 else [x for x in range(even, top + 1, 64)
                                                        if sum(parts_of(k, x) for k in b) * columns <= 768]
            want = lengths[0] if lengths else most if top == most else even
        assert limit == want, (b, columns)
        assert parts <= 128 and workgroups <= len(b) * columns + 768 and longest <= max(up(2 * even), 64)
