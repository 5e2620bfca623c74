"""The per-device count that the launchers size grids by: each device has its own, and several host threads may ask at
once.  A host program, so it needs neither HIP nor a GPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <thread>
#include <vector>
#include "compute_units.h"
static seka::PerDeviceCount counts;
static std::atomic<int> asked{0}, wrong{0};
int main() {
  auto ask = [](int d) { ++asked; return 100 + d; };
  std::vector<std::thread> threads;
  for (int t = 0; t < 8; ++t)
    threads.emplace_back([&, t] {
      for (int i = 0; i < 20000; ++i) {
        const int d = (i + t) % 5;
        if (counts.of(d, ask) != 100 + d) ++wrong;
      }
    });
  for (auto& t : threads) t.join();
  if (wrong || asked < 5 || asked > 5 * 8) return 1;          // at most once per device and thread
  if (counts.of(1000, ask) != 1100 || counts.of(-1, ask) != 99 || counts.of(3, ask) != 103) return 2;
  return 0;
}
"""


def test_each_device_has_its_own_count(tmp_path):
    src, exe = tmp_path / "counts.cpp", tmp_path / "counts"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-pthread", "-I", os.path.join(ROOT, "paper_2603_01281_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)], timeout=60).returncode == 0
