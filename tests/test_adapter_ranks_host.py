"""Host-side bookkeeping of the slots' ranks (compiled for the CPU with g++): slots set from several threads while
another asks whether any is below the pool's rank.  Built with the thread sanitizer, which reports a call that looks at
another slot's entry, and without it for the outcome."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r'''
#include <cstdio>
#include <thread>
#include "adapter_ranks.h"
int main() {
  const int32_t first[6] = {16, 8, 16, 1, 16, 16};
  lora::AdapterRanks r;
  r.init(16, 6, nullptr);
  if (r.any_lower()) return 2;
  r.init(16, 6, first);
  if (!r.any_lower() || r[1] != 8 || r[3] != 1 || r[5] != 16) return 3;
  std::vector<std::thread> threads;
  for (int a = 0; a < 4; ++a)
    threads.emplace_back([&, a] {
      for (int i = 0; i < 20000; ++i) r.set(a, 8 + (i + a) % 9);
      r.set(a, 16);
    });
  int seen = 0;
  for (int i = 0; i < 20000; ++i) seen += r.any_lower();
  for (auto &t : threads) t.join();
  if (r.any_lower()) return 4;              // every change was counted
  r.set(5, 15);
  if (!r.any_lower()) return 5;
  r.set(5, 15);
  r.set(5, 16);
  if (r.any_lower()) return 6;
  printf("%d\n", seen);
  return 0;
}
'''


@pytest.mark.parametrize("flags", [[], ["-fsanitize=thread"]])
def test_slots_set_from_several_threads(tmp_path, flags):
    src, exe = tmp_path / "ranks.cpp", tmp_path / "ranks"
    src.write_text(SRC)
    csrc = os.path.join(ROOT, "paper_2604_07173_amd", "csrc")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-pthread", *flags, "-I", csrc, str(src), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    if "unexpected memory mapping" in out.stderr:
        pytest.skip("the sanitizer cannot run under this kernel's address layout")
    assert out.returncode == 0, out.stderr[-2000:]
