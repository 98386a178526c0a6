// The solver kernel with float32 inner solves.
#include "tick.h"

namespace pfc {

void launch_tick_f32(const TickLaunch& q, hipStream_t stream) { launch_tick_T<float>(q, stream); }
PFC_TICK_TRACE(f32)

}  // namespace pfc
