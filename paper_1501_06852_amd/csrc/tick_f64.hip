// The solver kernel with float64 inner solves.
#include "tick.h"

namespace pfc {

void launch_tick_f64(const TickLaunch& q, hipStream_t stream) { launch_tick_T<double>(q, stream); }
PFC_TICK_TRACE(f64)

}  // namespace pfc
