// Segment kernels: int32 nests of two or three reducing segments (hp_segs.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "hp_internal.h"

namespace hp {

// Run a nest whose plan has a segment route (SegRoute::kind != SEGS_OFF); ws holds
// SegRoute::ws_bytes.
hp_status launch_segs(const SegRoute& s, const void* in, void* out, void* ws, hipStream_t st);

}  // namespace hp
