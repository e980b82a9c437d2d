// Prints the routes of the nests on stdin, one a line: depth, then extent:op per level,
// then the element type (0 int32, 1 float, 2 bf16).  Host code only: the planner's sources
// are linked in.
#include <cstdio>

#include "hp_internal.h"
#include "hp_stencil_form.h"
#include "hp_units.h"

int main() {
  int depth;
  while (std::scanf("%d", &depth) == 1) {
    if (depth == 0) {
      long long rows, cols;
      int sweeps;
      if (std::scanf("%lld %lld %d", &rows, &cols, &sweeps) != 3) return 1;
      std::printf("reg %d\n", (int)hp::reg_form(rows, cols, sweeps));
      continue;
    }
    hp_nest n{};
    n.depth = depth;
    for (int l = 0; l < depth; ++l) {
      long long e;
      int o;
      if (std::scanf("%lld:%d", &e, &o) != 2) return 1;
      n.extent[l] = e;
      n.op[l] = o;
    }
    int dtype;
    if (std::scanf("%d", &dtype) != 1) return 1;
    n.dtype = dtype;
    hp::Lowered alone, task;
    if (hp::lower(&n, nullptr, 0, &alone) != HP_OK || hp::lower(&n, nullptr, 0, &task, 1) != HP_OK) return 1;
    const hp::SegRoute s = hp::seg_route(&n, nullptr, 0, alone);
    const hp::UnitRoute u = hp::unit_route(&n, 0, task, false);
    std::printf("seg_kind %d seg_parts %u seg_tail %d tail_parts %u tail_per %d tail_off %llu seg_ws %llu kernel %d "
                "unit_on %d units %lld folds %lld unit_ws %llu mparts %d lparts %d part_len %d per %d fold_waves %d "
                "fold_form %d launch_wave %lld launch_group %lld plan_ws %zu\n",
                s.kind, s.parts, s.tail, s.tail_parts, s.tail_per, (unsigned long long)s.tail_off,
                (unsigned long long)s.ws_bytes, alone.dp.kernel, u.on, (long long)u.units, (long long)u.folds,
                (unsigned long long)u.ws_bytes, u.d.mparts, u.d.lparts, u.d.part_len, u.d.per, u.d.fold_waves,
                u.d.fold_form, (long long)hp::launch_tasks(64),
                (long long)hp::launch_tasks(64 * hp::kFoldWaves), task.info.workspace_bytes);
  }
}
