// Launches of the fused step (step_kernels.hip) behind the wrappers of common.h.
#pragma once

#include "common.h"

namespace lbmib {

// The step modes of launch_stream_collide and launch_stream_collide_mom.
void launch_step(const Dev& d, int storage, int mode, int share, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1);
void launch_step_mom(const Dev& d, int mode, int share, hipStream_t s);
// Advection of the last step of a sequence, in place, and the step counter.
void launch_step_end(const Dev& d, hipStream_t s);
// Near tiles of step counter + sub from the regions in d.bstate.
void launch_step_mark(const Dev& d, hipStream_t s);

}  // namespace lbmib
