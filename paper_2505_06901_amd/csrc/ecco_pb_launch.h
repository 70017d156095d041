// Host-side helpers of the launch code of the self-contained block format.
#pragma once

#include "ecco_launch.h"
#include "ecco_pb_internal.h"

namespace ecco_pb {

using ecco::aligned;

// a model can be used once it is on a device, and only while that device is the calling thread's current one: the
// kernels are launched on the current device and read the model's tables through device pointers
inline int model_ready(const ecco_pb_model* m) {
    if (!m || !m->dev || m->device < 0) return ECCO_EINVAL;
    int cur = -1;
    return (hipGetDevice(&cur) == hipSuccess && cur == m->device) ? ECCO_OK : ECCO_EINVAL;
}

}  // namespace ecco_pb
