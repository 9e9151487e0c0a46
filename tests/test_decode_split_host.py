"""The decode's rules on sizes, compiled for the host from the library's own header: how the
workgroups of a split launch fall on the 8 XCDs."""
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
