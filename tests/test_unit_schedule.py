"""The unit schedule of the Top-K kernel (csrc/schedule.h), compiled for the host:
whatever the partitions asked for, every unit is walked once and in order, a
grid of one block per unit gives every block one unit, and no block has more
units than the most even split (contiguous ranges) or whole groups (interleaved
groups) allow.
"""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_32398_amd", "csrc")

PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include <vector>
#include "schedule.h"
using dol::Sched;

// 0, or the line of the property that does not hold
static int check(int64_t units, int64_t blocks, Sched want) {
  const Sched sc = dol::plan_units(units, blocks, want);
  if (sc.lp > want.lp || blocks % (int64_t(1) << sc.lp) != 0 || sc.gu < 1) return __LINE__;
  std::vector<int> seen(units, 0), mine(blocks, 0);
  for (int64_t b = 0; b < blocks; ++b) {
    dol::UnitWalk w((uint32_t)units, (uint32_t)blocks, (uint32_t)b, sc.lp, (uint32_t)sc.gu);
    int64_t last = -1;
    for (uint32_t u = w.first(); u != (uint32_t)units; u = w.next(u)) {
      if (u >= units || (int64_t)u <= last) return __LINE__;
      last = u;
      ++seen[u];
      ++mine[b];
    }
  }
  for (int s : seen)
    if (s != 1) return __LINE__;
  const int most = *std::max_element(mine.begin(), mine.end());
  const int64_t parts = int64_t(1) << sc.lp, per_part = (units + parts - 1) / parts, gs = blocks / parts;
  const int64_t groups = (per_part + sc.gu - 1) / sc.gu;
  if (sc.gu != want.gu && most > (units + blocks - 1) / blocks) return __LINE__;
  if (sc.gu == want.gu && most > sc.gu * ((groups + gs - 1) / gs)) return __LINE__;
  if (blocks == units && most != 1) return __LINE__;
  return 0;
}

int main() {
  const Sched wants[] = {{4, 0}, {4, 3}, {4, 4}, {4, 5}, {0, 0}, {0, 3}, {1, 5}, {7, 4}};
  for (int64_t grid : {256, 512, 304, 60, 7, 1})
    for (int64_t units = 1; units <= 2600; units += units < 1100 ? 1 : 37)
      for (const Sched& w : wants) {
        const int64_t blocks = std::min(grid, units);
        const int line = check(units, blocks, w);
        if (line != 0) {
          printf("line %d: units %lld blocks %lld want gu %lld lp %d\n", line, (long long)units, (long long)blocks,
                 (long long)w.gu, w.lp);
          return 1;
        }
      }
  // counts near the 2^29 limit: sizes only
  const int64_t big = (int64_t(1) << 29) - 3;
  for (const Sched& w : wants) {
    const Sched sc = dol::plan_units(big, 256, w);
    int64_t n = 0;
    for (uint32_t b = 0; b < 256; ++b) {
      const dol::UnitWalk k((uint32_t)big, 256, b, sc.lp, (uint32_t)sc.gu);
      if (k.first() > (uint32_t)big || k.step != 256 / (1u << sc.lp) * (uint32_t)sc.gu) return 2;
      n += k.first() < (uint32_t)big;
    }
    if (n == 0) return 3;
  }
  return 0;
}
"""


def test_unit_schedule(tmp_path):
    src, exe = tmp_path / "schedule.cpp", tmp_path / "schedule"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-Wall", "-Werror", "-std=c++17", f"-I{CSRC}", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
