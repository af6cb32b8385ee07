// Host check of the attention's work decomposition (csrc/plan.h) on a device of 256 CUs that hold
// one 256-row or two 128-row bf16 workgroups each. Reads lines "bf16 B H D n_ref n_tgt" and prints
// for the queries of the whole launch and for the target queries alone: rows per workgroup, whole
// tiles, split tiles, chunks, workspace bytes, the workspace bytes of three per-segment masses, and
// the rows per workgroup without a workspace; reads "f32 B H D n_ref n_tgt" and prints subtiles x key groups.
#include <cinttypes>
#include <cstdio>
#include <cstring>

#include "plan.h"

using namespace refadapt;

int main() {
  char type[8];
  int B, H, D, nr, nt;
  while (std::scanf("%7s %d %d %d %d %d", type, &B, &H, &D, &nr, &nt) == 6) {
    if (!std::strcmp(type, "f32")) {
      const F32Split s = f32_split((int64_t)B * H, nr, nt, 256);
      std::printf("%dx%d\n", s.subtiles, s.wavefronts / s.subtiles);
      continue;
    }
    const PlanShape shape{(int64_t)B * H, D, nr, nt, AttnSlots{256, 1}, AttnSlots{256, 2}};
    const LaunchPlans l = plan_launch(shape, true), whole = plan_launch(shape, false);
    for (const bool all : {true, false}) {
      const LaunchMode m{all, !all, false};
      const QueryPlan& q = (all ? l.all : l.tgt)[l.prefers_small(m)];
      std::printf("%d %d %d %d %zu %zu %d%s", q.bm, q.plan.whole, q.plan.split_tiles, q.plan.chunks,
                  launch_ws_bytes(l, m, D), launch_seg_ws_bytes(l, m, D, 3), whole.tgt[whole.prefers_small(m)].bm,
                  all ? " " : "\n");
    }
  }
}
