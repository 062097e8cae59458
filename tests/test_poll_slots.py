"""The slots of host memory that polls copy into (csrc/pollslots.hpp), on the
CPU: more threads than slots take and give them as fast as they can, and no
slot has two holders; all are free again afterwards, and a full set says so."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <thread>
#include <vector>
#include "pollslots.hpp"
using ens::PollSlots;
int main() {
  PollSlots s;
  std::atomic<int> holder[PollSlots::kSlots] = {};
  std::atomic<int> shared{0}, none{0};
  std::vector<std::thread> t;
  for (int k = 0; k < 80; ++k)
    t.emplace_back([&, k] {
      for (int n = 0; n < 2000; ++n) {
        const int i = s.take();
        if (i < 0) {
          ++none;
          continue;
        }
        int nobody = 0;
        if (i >= PollSlots::kSlots || !holder[i].compare_exchange_strong(nobody, k + 1)) ++shared;
        std::this_thread::yield();
        if (holder[i].exchange(0) != k + 1) ++shared;
        s.give(i);
      }
    });
  for (auto& th : t) th.join();
  bool seen[PollSlots::kSlots] = {};
  for (int n = 0; n < PollSlots::kSlots; ++n) {
    const int i = s.take();
    if (i < 0 || i >= PollSlots::kSlots || seen[i]) return 2;
    seen[i] = true;
  }
  if (s.take() != -1) return 3;
  s.give(17);
  if (s.take() != 17) return 4;
  printf("%d shared, %d none\n", shared.load(), none.load());
  return shared.load() ? 1 : 0;
}
"""


def test_no_slot_has_two_holders(tmp_path):
    src, exe = tmp_path / "slots.cpp", tmp_path / "slots"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", os.path.join(ROOT, "paper_1511_03703_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True, timeout=120)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
