"""The one-round kernel's rings (no GPU: its own step arithmetic, walked through as its waves do): what is multiplied is the step
that is due, it has landed when it is read, and no copy reaches past K, whatever K."""
import os
import shutil
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2404_19124_amd", "csrc")

PROGRAM = r"""
#include <vector>
#include "once_steps.h"
using namespace specdraft;
// A ring of `depth` slots: all of them filled, slot 0 read; then at every step the next slot is read, when all copies but those
// of the last depth - 2 slots have landed, and the slot of this step is filled again.
static int walk(int depth, int kt) {
  std::vector<int> slot(depth), when(depth);
  int copies = 0;
  auto copy = [&](int u, int step) {
    if (step < 0 || step >= kt) return false;
    slot[u % depth] = step;
    when[u % depth] = ++copies;
    return true;
  };
  for (int u = 0; u < depth; ++u)
    if (!copy(u, u)) return 1;
  int held = slot[0];
  for (int s = 0; s < kt; ++s) {
    if (held != s) return 2;
    if (s + 1 < kt && when[(s + 1) % depth] > copies - (depth - 2)) return 3;
    const int next = slot[(s + 1) % depth];
    if (!copy(s, once_next_step(s, depth, kt))) return 4;
    held = next;
  }
  return 0;
}
int main() {
  for (int kt = kOnceDW; kt <= 512; ++kt)
    for (int depth : {kOnceDW, kOnceDS})
      if (int bad = walk(depth, kt)) return bad;
  return 0;
}
"""


def test_rings(tmp_path):
    (tmp_path / "walk.cpp").write_text(PROGRAM)
    exe = str(tmp_path / "walk")
    subprocess.run([shutil.which("g++") or "g++", "-O1", "-std=c++17", "-I", CSRC, str(tmp_path / "walk.cpp"), "-o", exe], check=True,
                   timeout=120)
    assert subprocess.run([exe], timeout=60).returncode == 0


def test_the_kernel_asks_for_those_steps():
    with open(os.path.join(CSRC, "kernels_head_once.hip")) as f:
        text = f.read()
    assert text.count("copy(i, u, u);") == 1 and text.count("copy(i, u, once_next_step(base + u, DEPTH, kt));") == 1
    assert text.count("copy(i, ") == 2 and text.count("_load_lds(") == 1
