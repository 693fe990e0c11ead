// The launch shape of the fitness walk over bound tables. Plain C++, so that a host program can check it.
#pragma once

#include <stdint.h>

namespace maestro {

struct FitnessGrid {
  int threads;                           // of a workgroup
  int parts;                             // wavefronts that share the short pairs of 64 stages
  int64_t blocks;
};

// One round of stages per workgroup while the LDS staging is small, up to four (equal ones) at 4,096
// nodes, where only two workgroups of 512 threads fit a CU and each stages 74 KB; half that width up to
// 1,024 nodes (registers admit four or five wavefronts a SIMD: 43 against 47 us on 512 nodes).
// With plans a small batch leaves most of the chip idle while each wavefront goes through up to all
// nodes that fall short, so as many wavefronts share them as fill one workgroup of 512 a CU. Two, or
// sharing up to twice as many stages, cost the batches that share nothing more than they give: 131,072
// stages 30.9 against 29.8 us, 65,536 stages 30.4 against 29.2; on 4,096 nodes without headroom the latter
// take 292 against 393 (780 without sharing, 380 scoring every pair).
inline FitnessGrid fitness_grid(int64_t n, int32_t padded, bool plans, int64_t cus) {
  FitnessGrid g{padded > 1024 ? 512 : 256, 1, 0};
  while (plans && g.parts < g.threads / 64 && n * 2 * g.parts <= cus * 512) g.parts *= 2;
  const int64_t stages = g.threads / g.parts, want = (n + stages - 1) / stages, slots = 2 * cus;
  const int64_t most_rounds = padded > 1024 ? padded / 1024 : 1;
  const int64_t fair = (want + slots - 1) / slots, rounds = fair < most_rounds ? fair : most_rounds;
  g.blocks = (want + rounds - 1) / rounds;
  const int64_t most = ((int64_t)1 << 31) / g.threads;   // a launch takes fewer than 2^32 threads a dimension
  if (g.blocks > most) g.blocks = most;
  return g;
}

}  // namespace maestro
