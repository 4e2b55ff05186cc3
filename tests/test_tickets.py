"""The host's wait for words that a kernel stores (no GPU: threads store them): it lasts as long as they take, sees the last of them,
and only an answer other than 0 ends it before."""
import os
import shutil
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2404_19124_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "tickets.h"
using namespace specdraft;
int main() {
  uint32_t words[4] = {7, 7, 7, 7};
  int asked = 0;
  auto store = [&](int i, int ms, uint32_t v) {
    return std::thread([&words, i, ms, v] {
      std::this_thread::sleep_for(std::chrono::milliseconds(ms));
      __atomic_store_n(words + i, v, __ATOMIC_RELEASE);
    });
  };
  auto fine = [&] { ++asked; return 0; };
  if (wait_for_tickets(words, 0, 8, fine) || wait_for_tickets(words, 4, 7, fine) || asked) return 1;
  {   // out of order, the last one long after the others, longer than any limit a wait of this kind could have had
    std::thread a = store(0, 30, 8), b = store(3, 1, 8), c = store(2, 5, 8), d = store(1, 2500, 8);
    const auto t0 = std::chrono::steady_clock::now();
    if (wait_for_tickets(words, 4, 8, fine)) return 2;
    const double s = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    a.join(); b.join(); c.join(); d.join();
    if (s < 2.4 || asked < 5 || asked > 40) return 3;
  }
  {   // nobody stores the third
    std::thread a = store(0, 1, 9), b = store(1, 1, 9);
    int n = 0;
    const int got = wait_for_tickets(words, 3, 9, [&] { return ++n == 3 ? 41 : 0; });
    a.join(); b.join();
    if (got != 41 || n != 3) return 4;
  }
  return 0;
}
"""


def test_wait(tmp_path):
    (tmp_path / "wait.cpp").write_text(PROGRAM)
    exe = str(tmp_path / "wait")
    subprocess.run([shutil.which("g++") or "g++", "-O2", "-std=c++17", "-pthread", "-I", CSRC, str(tmp_path / "wait.cpp"), "-o", exe],
                   check=True, timeout=120)
    assert subprocess.run([exe], timeout=60).returncode == 0


def test_the_library_waits_for_nothing_else():
    """A wait for the device would be one for every stream, and an error while another thread captures."""
    with open(os.path.join(CSRC, "spec_lib.hip")) as f:
        assert "hipDeviceSynchronize" not in f.read()
