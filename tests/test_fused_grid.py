"""The fused stages are asked to run only where HIP can launch them: fewer than 2^32 work items in a grid dimension."""

import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_18239_amd", "csrc")

PROGRAM = """
#include <cstdio>
#include <initializer_list>
#include "fused_grid.hpp"
using namespace lime;
#define CHECK(x) if (!(x)) { std::printf("line %d: %s\\n", __LINE__, #x); return 1; }
int main() {
  // 65 535 users of 8192 items, four heads: the last that fits, with 128 workgroups to spare
  CHECK(history_workgroups(65535, 8192, 4) == 65535 * 32 * 4 && launch_fits(history_workgroups(65535, 8192, 4)));
  CHECK(!launch_fits(history_workgroups(65535, 8193, 4)));
  CHECK(history_workgroups(1, 1, 1) == 1 && history_workgroups(2, 257, 4) == 16);
  for (int64_t total : {int64_t{1}, int64_t{8}, int64_t{9}, (int64_t{1} << 23) - 9, (int64_t{1} << 23) - 8, (int64_t{1} << 23) - 7, (int64_t{1} << 23),
                        (int64_t{1} << 31) - 9}) {
    CHECK(launched_workgroups(total) >= total && launched_workgroups(total) % 8 == 0);
    CHECK(launch_fits(total) == (launched_workgroups(total) * kThreads < int64_t{1} << 32));
  }
  return 0;
}
"""


def test_no_launch_past_the_limit(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_the_rules_ask_it():
    for f in ("fused_history.hip", "fused_rows.hip"):
        text = open(os.path.join(CSRC, f)).read()
        assert "launch_fits(" in text and "dim3(launched_workgroups(a.total))" in text, f
