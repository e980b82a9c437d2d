// Row kernels: one reduction per output over a contiguous block (hp_rows.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "hp_internal.h"

namespace hp {

// Run a nest whose plan has a row route (RowRoute::kind != ROWS_OFF); ws holds the
// partials of a split block, n_out * parts of 8 bytes: no more than the plan's workspace,
// which has 16 for each of at least as many.
hp_status launch_rows(const RowRoute& r, const void* in, void* out, void* ws, hipStream_t st);

}  // namespace hp
