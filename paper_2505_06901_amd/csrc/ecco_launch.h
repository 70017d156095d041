// Host-side helpers of the launch code, shared by the kernel sources of the two-chain block format.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "ecco_internal.h"

#define ECCO_HIP_CHECK(expr) do { if ((expr) != hipSuccess) return ECCO_EHIP; } while (0)

namespace ecco {

inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

// a model can be used once it is on a device, and only while that device is the calling thread's current one: the
// kernels are launched on the current device and read the model's tables through device pointers
inline int model_ready(const ecco_model* m) {
    if (!m || !m->dev || m->device < 0) return ECCO_EINVAL;
    int cur = -1;
    return (hipGetDevice(&cur) == hipSuccess && cur == m->device) ? ECCO_OK : ECCO_EINVAL;
}

// compute units of a device, asked once per device (defined in ecco_kernels.hip)
int cu_count(int device);

// tells the runtime, once per kernel and device, that the kernel may use more than 64 KB of LDS (defined in ecco_kernels.hip)
int allow_lds_once(const void* kernel, int device, size_t bytes);
template <class K>
int allow_lds(K kernel, int device, size_t bytes) { return allow_lds_once(reinterpret_cast<const void*>(kernel), device, bytes); }

}  // namespace ecco
