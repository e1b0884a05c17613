// Host interface of the LDS-window level walk (ring.hip), used by device.hip.
#pragma once

#include "batch.h"

namespace fm {

struct RingPlan;   // tables and buffers of one batch

// Build the window tables of a batch when the rule of ring.hip takes it;
// *out stays nullptr when another kernel is the better one or the tables do
// not fit.  Work is done on the null stream and has finished on return.
int ring_create(const fm_batch* b, const std::vector<SrcDev>& src, RingPlan** out);
void ring_free(RingPlan* r);

// The walk of that direction is to be taken (r may be nullptr).
bool ring_has(const RingPlan* r, bool fwd);

// Its workgroup size, window and side slots.
void ring_sizes(const RingPlan* r, bool fwd, int32_t* threads, int32_t* window, int32_t* side);

// One walk over the batch on its stream: a.work / a.xB / a.in / a.out and the
// modes as for the other walk kernels.
hipError_t ring_walk(const fm_batch* b, bool fwd, const ApplyArgs& a);

}  // namespace fm
