"""A kernel's leave to use more than 64 KiB of LDS is a device's own: it is asked for on every device that runs the kernel."""

import os
import re
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_18239_amd", "csrc")

PROGRAM = """
#include <atomic>
#include <cstdio>
#include <thread>
#include <vector>
#include "per_device.hpp"
#define CHECK(x) if (!(x)) { std::printf("line %d: %s\\n", __LINE__, #x); return 1; }
int main() {
  lime::PerDevice a, b;
  int calls = 0;
  auto make = [&] { ++calls; return 0; };
  CHECK(a.ensure(0, make) == 0 && calls == 1);
  CHECK(a.ensure(0, make) == 0 && calls == 1);   // once per device
  CHECK(a.ensure(1, make) == 0 && calls == 2);   // a second device has its own
  CHECK(a.ensure(63, make) == 0 && a.ensure(63, make) == 0 && calls == 3);
  CHECK(b.ensure(0, make) == 0 && calls == 4);   // and another kernel
  CHECK(a.ensure(5, [&] { ++calls; return 7; }) == 7 && calls == 5);
  CHECK(a.ensure(5, make) == 0 && calls == 6);   // a failure is tried again
  CHECK(a.ensure(5, make) == 0 && calls == 6);
  for (int odd : {64, 1000, -1}) CHECK(a.ensure(odd, make) == 0 && a.ensure(odd, make) == 0);
  CHECK(calls == 12);
  lime::PerDevice c;
  std::atomic<int> made{0}, wrong{0};
  std::vector<std::thread> ts;
  for (int t = 0; t < 8; ++t)
    ts.emplace_back([&] {
      for (int i = 0; i < 1000; ++i)
        if (c.ensure(i % 64, [&] { ++made; return 0; }) != 0 || made < 1) ++wrong;
    });
  for (auto& t : ts) t.join();
  CHECK(wrong == 0 && made >= 64 && made <= 8 * 64);
  return 0;
}
"""


def test_a_setting_is_made_on_each_device(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-pthread", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_every_kernel_asks_through_it():
    for f in sorted(os.listdir(CSRC)):
        if f.endswith((".hip", ".hpp")) and f != "device.hip":
            assert not re.search(r"hipFuncSetAttribute\s*\(", open(os.path.join(CSRC, f)).read()), f
