"""The launch shape of the fitness walk, checked by a host program over batch sizes up to the largest
that the entry point takes: every stage has a lane in some round, a dimension stays below the 2^32
threads that a launch takes, and wavefronts share stages only while the chip has room for them."""
import os
import subprocess

import paper_2606_12950_amd as M

CSRC = os.path.join(os.path.dirname(M.LIBRARY_PATH), "csrc")

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "fitness_grid.h"
using namespace maestro;

int main() {
  for (long long base = 1; base <= 1ll << 37; base *= 2)
    for (long long n = base - 1; n <= base + 1; ++n)
      for (int padded : {64, 512, 1024, 1088, 2048, 4096})
        for (int plans = 0; plans < 2; ++plans)
          for (int cus : {1, 32, 256}) {
            if (n < 1 || n > 1ll << 37) continue;
            const FitnessGrid g = fitness_grid(n, padded, plans, cus);
            const long long stages = g.threads / g.parts, step = g.blocks * stages;
            const bool ok = g.blocks >= 1 && g.blocks * g.threads < 1ll << 32 && g.blocks < 1ll << 31 &&
                            g.parts >= 1 && g.parts <= g.threads / 64 && g.threads % (64 * g.parts) == 0 &&
                            (g.parts == 1 || (plans && n * g.parts <= 1024ll * cus)) && (g.blocks - 1) * stages < n &&
                            (n + step - 1) / step >= 1;
            if (!ok)
              return std::printf("n %lld padded %d plans %d cus %d: %d threads, %d parts, %lld blocks\n", n, padded, plans, cus,
                                 g.threads, g.parts, (long long)g.blocks);
          }
  return 0;
}
"""


def test_launch_shapes(tmp_path):
    src, exe = tmp_path / "grid.cpp", tmp_path / "grid"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", f"-I{CSRC}", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.stdout == "" and r.returncode == 0
