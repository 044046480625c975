"""Settings a kernel needs before its first launch are made once per device, again after a failure, and before any thread that
needs them goes on; and the launchers leave none of them to a switch of the whole process (CPU only)."""
import glob
import os
import re
import subprocess

from paper_2307_02628_amd import _build

DRIVER = r"""
#include <cstdio>
#include <thread>
#include <vector>
#include "once_per_device.h"
#define EXPECT(c) do { if (!(c)) { printf("FAILED %s:%d: %s\n", __FILE__, __LINE__, #c); return 1; } } while (0)
int main() {
  std::atomic<uint64_t> done{0}, other{0};
  int calls = 0;
  auto good = [&]() { ++calls; return true; };
  EXPECT(skd::once_per_device(done, 0, good) && calls == 1);
  EXPECT(skd::once_per_device(done, 0, good) && calls == 1);
  EXPECT(skd::once_per_device(done, 1, good) && calls == 2);     // a second device has its own settings
  EXPECT(skd::once_per_device(done, 63, good) && skd::once_per_device(done, 63, good) && calls == 3);
  EXPECT(skd::once_per_device(other, 0, good) && calls == 4);    // and so have other kernels
  EXPECT(!skd::once_per_device(done, 2, [&]() { ++calls; return false; }) && calls == 5);
  EXPECT(skd::once_per_device(done, 2, good) && calls == 6);     // a failure is not remembered
  EXPECT(skd::once_per_device(done, 64, good) && skd::once_per_device(done, 64, good) && calls == 8);
  EXPECT(skd::once_per_device(done, -1, good) && calls == 9);
  for (int round = 0; round < 50; ++round) {
    std::atomic<uint64_t> d{0};
    std::atomic<int> set[8] = {};
    std::atomic<int> early{0};
    std::vector<std::thread> t;
    for (int i = 0; i < 8; ++i)
      t.emplace_back([&, i]() {
        for (int dev = 0; dev < 8; ++dev) {
          const int k = (dev + i) % 8;
          skd::once_per_device(d, k, [&]() { set[k].fetch_add(1); return true; });
          if (set[k].load() < 1) early.fetch_add(1);
        }
      });
    for (auto &x : t) x.join();
    EXPECT(early.load() == 0 && d.load() == 0xff);
    for (int k = 0; k < 8; ++k) EXPECT(set[k].load() >= 1 && set[k].load() <= 8);
  }
  printf("all checks passed\n");
  return 0;
}
"""


def test_once_per_device(tmp_path):
    src = tmp_path / "driver.cpp"
    src.write_text(DRIVER)
    exe = str(tmp_path / "driver")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-O1", "-pthread", "-I", _build.CSRC, str(src), "-o", exe], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0 and "all checks passed" in res.stdout, res.stdout + res.stderr


def test_no_process_wide_switch():
    for path in glob.glob(os.path.join(_build.CSRC, "*.h*")):
        text = open(path).read()
        assert not re.search(r"\bstatic\s+bool\s+\w+\s*=", text), path
        for use in re.finditer(r"hipFuncSetAttribute", text):
            assert "once_per_device(done" in text[max(0, use.start() - 300):use.start()], path
