"""The fused stages' launches: only where HIP can launch them (fewer than 2^32 work items in a grid dimension), and who takes what."""

import os
import subprocess

import pytest

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


# Every tile of every user's every chunk is taken once, by a wave of a workgroup that has all tiles of that chunk, as the kernel counts.
TAILS = """
#include <cstdio>
#include <initializer_list>
#include <vector>
#include "fused_grid.hpp"
using namespace lime;
#define CHECK(x) if (!(x)) { std::printf("B=%d N=%d at_once=%d line %d: %s\\n", B, N, at_once, __LINE__, #x); return 1; }
int main() {
  for (int B : {1, 2, 7, 8, 9, 64, 1000})
    for (int N : {1, 20, 32, 33, 64, 65, 96, 100, 128, 129, 200, 255, 256, 257, 270, 288, 300, 512, 513, 777})
      for (int at_once : {0, 1, 5, 64, 256, 512}) {
        const int h = 4, chunks = (N + kChunkKeys - 1) / kChunkKeys;
        const HistoryTails t = history_tails(B, N, h, at_once);
        CHECK(t.users >= 1 && t.tiles >= 1 && t.users * t.tiles <= kWaves && (at_once > 0 || t.users == 1));
        const int64_t total = tails_workgroups(t, B, h);
        CHECK(total <= history_workgroups(B, N, h));
        std::vector<int> seen(B * chunks * kWaves);
        for (int64_t group = 0; group < total / h; ++group)
          for (int wave = 0; wave < kWaves; ++wave) {
            int chunk = chunks - 1, b0 = (group - t.first) * t.users, users = std::min(t.users, B - b0), tiles = t.tiles, per_tile = t.per_tile;
            if (group < t.first) chunk = group % (chunks - 1), b0 = group / (chunks - 1), users = 1, tiles = kWaves, per_tile = 65536 / kWaves;
            const int slot = wave * per_tile >> 16, tile = wave - slot * tiles;
            CHECK(tile >= 0 && tile < tiles && slot == wave / tiles && users >= 1 && b0 + users <= B);
            if (slot < users) ++seen[((b0 + slot) * chunks + chunk) * kWaves + tile];
          }
        for (int b = 0; b < B; ++b)
          for (int c = 0; c < chunks; ++c)
            for (int tile = 0; tile < kWaves; ++tile) {
              const int times = seen[(b * chunks + c) * kWaves + tile];
              CHECK(c * kChunkKeys + 32 * tile < N ? times == 1 : times <= 1);
            }
      }
  return 0;
}
"""


@pytest.mark.parametrize("program", [PROGRAM, TAILS], ids=["limit", "tails"])
def test_launch(tmp_path, program):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(program)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_the_rules_ask_it():
    for f in ("fused_history.hip", "fused_rows.hip"):
        text = open(os.path.join(CSRC, f)).read()
        assert "launch_fits(" in text and "dim3(launched_workgroups(a.total))" in text, f
