// Launchers of the unit kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "hp_units.h"

namespace hp {

// n unit tasks (nest, unit) of nests of one input type, a wave each, in list order.
hp_status launch_units(int dtype, const UnitDesc* descs, const int2* tasks, int n, hipStream_t st);
// All units of one nest (n of them), in order: the baseline of one launch per nest.
hp_status launch_units_of(int dtype, const UnitDesc* desc, int n, hipStream_t st);
// Load the unit kernels: each launched with no tasks.
hp_status warm_unit_kernels(hipStream_t st);
// The nests' partial carriers: n fold tasks (nest, output), the first n_shared on a workgroup
// each (nests of kFoldWaves), the others on a wave.
hp_status launch_unit_folds(const UnitDesc* descs, const int2* tasks, int n_shared, int n, hipStream_t st);

}  // namespace hp
