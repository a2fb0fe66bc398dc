"""The rule that keeps the waits of the single-read kernel safe next to other launches (csrc/laq_team.h), against a model of a
device that is filled in the worst order (no GPU needed)."""
import os
import subprocess

import pytest

MODEL = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>
#include "laq_team.h"
using namespace laq;

// A launch: its workgroups that have not started, per counter; members of the counter's present team that are on the device.
struct Launch { int T, left[2], part[2]; };

// Places are handed out one at a time, always to a workgroup that completes no team if there is one; a complete team ends at once.
// Returns whether all launches end; *held: the most places that parts of teams held.
static bool all_end(std::vector<Launch> ls, int places, int* held) {
  *held = 0;
  for (;;) {
    int in_parts = 0, left = 0;
    for (const Launch& l : ls) in_parts += l.part[0] + l.part[1], left += l.left[0] + l.left[1];
    if (in_parts > *held) *held = in_parts;
    if (left == 0) return true;
    if (in_parts == places) return false;
    Launch* take = nullptr;
    int counter = 0;
    for (int completes = 0; completes < 2 && !take; ++completes)
      for (Launch& l : ls)
        for (int c = 0; c < 2 && !take; ++c)
          if (l.left[c] > 0 && (l.part[c] + 1 == l.T) == (completes == 1)) take = &l, counter = c;
    --take->left[counter];
    if (++take->part[counter] == take->T) take->part[counter] = 0;
  }
}

static Launch launch(int T, int places, int heads = 1 << 20) {
  TeamPlan p;
  if (!plan_teams(heads, T, places, &p)) { printf("no plan for %d of %d\n", T, places); exit(1); }
  if (p.n_teams * T > places || p.early % T != 0 || p.early < 0 || p.early > p.n_teams * T) { printf("bad plan %d\n", T); exit(1); }
  return Launch{T, {p.early, p.n_teams * T - p.early}, {0, 0}};
}

int main(int argc, char** argv) {
  if (!strcmp(argv[1], "line")) {                       // T, places -> ordinary, counters
    const int T = atoi(argv[2]), places = atoi(argv[3]);
    printf("%d %d\n", ordinary_team(T, places) ? 1 : 0, counters_of(T, places));
    return 0;
  }
  if (!strcmp(argv[1], "stream")) {                     // compute units, priority, words of the mask
    uint32_t mask[32] = {};
    for (int i = 4; i < argc; ++i) mask[i - 4] = (uint32_t)strtoul(argv[i], nullptr, 16);
    printf("%d\n", stream_counted(mask, atoi(argv[2]), atoi(argv[3])) ? 1 : 0);
    return 0;
  }
  const int places = atoi(argv[2]);
  int held, most = 0;
  if (!strcmp(argv[1], "given")) {                      // launches of these lengths
    std::vector<Launch> ls;
    for (int i = 3; i < argc; ++i) ls.push_back(launch(atoi(argv[i]), places));
    printf("%s\n", all_end(ls, places, &held) ? "ends" : "stuck");
    return 0;
  }
  srand(5);                                             // "covered": any HW_QUEUES launches that the rule covers
  int longest = 0;
  while (longest < places && ordinary_team(longest + 1, places)) ++longest;
  for (int round = 0; round < 3000; ++round) {
    std::vector<Launch> ls;
    for (int q = 0; q < HW_QUEUES; ++q) {
      const int T = round < longest ? round + 1 : 1 + rand() % longest;
      if (!ordinary_team(T, places)) { printf("not monotone at %d\n", T); return 1; }
      ls.push_back(launch(T, places, round < longest ? 1 << 20 : 1 + rand() % 600));
    }
    if (!all_end(ls, places, &held)) { printf("stuck\n"); return 1; }
    most = held > most ? held : most;
  }
  printf("ends, longest %d, held %d\n", longest, most);
  return 0;
}
"""


@pytest.fixture(scope="module")
def model(repo_root, tmp_path_factory):
    d = tmp_path_factory.mktemp("team")
    src, exe = d / "model.cpp", d / "model"
    src.write_text(MODEL)
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-O1", "-Wall", "-I",
                    os.path.join(repo_root, "paper_2505_20334_amd", "csrc"), "-o", str(exe), str(src)], check=True)

    def run(*args):
        r = subprocess.run([str(exe)] + [str(a) for a in args], capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, r.stdout
        return r.stdout.strip()
    return run


def test_lines(model):
    for T, want in ((1, "1 2"), (64, "1 2"), (65, "1 1"), (128, "1 1"), (129, "0 2"), (512, "0 2")):
        assert model("line", T, 512) == want, T


def test_streams(model):
    full, rest = ["ffffffff"] * 8, ["ffffffff"] * 7
    assert model("stream", 256, 0, *full) == "1"
    assert model("stream", 250, 0, *rest, "03ffffff") == "1" and model("stream", 250, 0, *rest, "01ffffff") == "0"
    assert model("stream", 256, 0, *rest, "7fffffff") == "0" and model("stream", 256, 0) == "0"      # some compute units, none known
    assert model("stream", 256, -1, *full) == "0" and model("stream", 256, 1, *full) == "0"          # queues of their own


@pytest.mark.parametrize("places,longest", [(512, 128), (256, 64), (608, 152)])
def test_covered_launches_end_in_the_worst_order(model, places, longest):
    out = model("covered", places)
    assert out.startswith("ends, longest %d," % longest), out
    assert int(out.split()[-1]) < places


@pytest.mark.parametrize("lengths", [(64, 500), (64, 512), (64, 64, 64, 64, 64), (64, 64, 64, 64, 128), (128, 128, 128, 128, 100)])
def test_what_the_rule_leaves_out_can_get_stuck(model, lengths):
    # a long team beside a short one, and one launch more than the queues hold: what is not to be on the device together
    assert model("given", 512, *lengths) == "stuck"
