"""The decode's rules on sizes, compiled for the host from the library's own header: how the
workgroups of a split launch fall on the 8 XCDs, and how long the splits of a batch are whose requests
hold less than the bound."""
import os
import subprocess

import pytest

from paper_2608_13263_amd import build

CSRC = build.CSRC
PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include "vtoken_internal.h"
using namespace vtoken;

// `pairs` requests and heads with `work` splits each of `splits`: the busiest XCD's workgroups
static int busiest(int pairs, int work, int splits) {
  const int gs = decode_grid_splits(splits);
  int load[8] = {};
  for (int b = 0; b < pairs * gs; ++b) load[b % 8] += b % gs < work;
  return *std::max_element(load, load + 8);
}

int main() {
  for (int splits = 1; splits <= 600; ++splits) {
    if (decode_grid_splits(splits) < splits) return std::printf("no room for %d splits\n", splits), 1;
    for (int work = 1; work <= std::min(splits, 9); ++work) {
      const int got = busiest(64, work, splits);
      if (got > 8 * work) return std::printf("%d of %d splits: %d\n", work, splits, got), 1;
    }
  }
  std::printf("ok\n");
}
"""


@pytest.fixture(scope="module")
def run_program(tmp_path_factory):
    try:
        hipcc = build.hipcc()
    except RuntimeError:
        pytest.skip("hipcc not available")

    def run(text):
        d = tmp_path_factory.mktemp("split")
        src, exe = d / "rule.hip", d / "rule"
        src.write_text(text)
        subprocess.run([hipcc, "--offload-host-only", "-O1", "-std=c++17", "-w", "-I", CSRC, "-I",
                        os.path.join(build.ROOT, "include"), str(src), "-o", str(exe)],
                       check=True)
        return subprocess.run([str(exe)], capture_output=True, text=True).stdout.strip()
    return run


def test_work_falls_on_all_xcds(run_program):
    """Under a bound far above the requests only their first splits have work: in every launch
    those fall on the 8 XCDs evenly (64 (request, KV head) pairs: 8 on each for every split)."""
    assert run_program(PROGRAM) == "ok"


LENGTHS = r"""
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include "vtoken_internal.h"
using namespace vtoken;

int main() {
  std::srand(1);
  auto pick = [](int64_t lo, int64_t hi) { return lo + (std::rand() * 32768ll + std::rand()) % (hi - lo + 1); };
  int shortened = 0;
  for (int i = 0; i < 200000; ++i) {
    const int D = 32 << pick(0, 3), elem = pick(1, 2), group = 1 << pick(0, 3);
    const int64_t heads = 1 << pick(0, 3), reqs = pick(1, i % 2 ? 8 : 600);
    const int64_t bound = i % 7 == 0 ? 0x7fffffff - pick(0, 3) : pick(0, 1 << pick(4, 20));
    const DecodeSplit s = decode_split_rule(D, elem, reqs, heads, bound);
    const int splits = decode_splits(s, bound);
    const int64_t unit = decode_unit_tokens(D, elem);
    if (splits < 1 || splits > std::max<int64_t>(1, (bound + unit - 1) / unit))
      return std::printf("%d splits, bound %lld\n", splits, (long long)bound), 1;
    // requests of one length, any total a table with room at its ends may show
    const int64_t most = decode_max_count(D, elem, group, bound);
    const int64_t count = std::min<int64_t>(std::max<int64_t>(1, pick(0, most) >> pick(0, 12)), 0x7fffffff);
    const int64_t total = std::min<int64_t>(0x7fffffff, reqs * count);
    const int t = decode_request_tokens(s, count, total);
    const int64_t ns = (count + t - 1) / t;
    if (t % decode_round_tokens(D, elem) || t > s.tokens || t < unit)
      return std::printf("%d tokens a split, %d at most\n", t, s.tokens), 1;
    if (t < s.tokens && ns > splits)
      return std::printf("%lld splits of %d, room for %d\n", (long long)ns, t, splits), 1;
    // long splits only where they fill the chip, or shorter ones have no room
    if (t > unit && reqs * heads * ((count + t - 1) / t) < kDecodeFewGroups &&
        (count + t / 2 - 1) / (t / 2) <= splits)
      return std::printf("%lld requests of %lld under %lld: %d\n", (long long)reqs, (long long)count,
                         (long long)bound, t), 1;
    shortened += t < s.tokens;
    const int any = decode_request_tokens(s, count, static_cast<int>(pick(0, 0x7fffffff)) * (i % 2 ? 1 : -1));
    if (any < s.tokens && (count + any - 1) / any > splits) return std::printf("malformed\n"), 1;
  }
  std::printf(shortened > 1000 ? "ok\n" : "never shorter\n");
}
"""


def test_split_lengths(run_program):
    """Over random sizes: a request's splits are whole rounds, fit the room that the host's length
    leaves (or have the host's length), and a batch far below its bound is spread over the chip."""
    assert run_program(LENGTHS) == "ok"
