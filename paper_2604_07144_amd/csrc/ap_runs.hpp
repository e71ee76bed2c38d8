// The order of a list run, for the case that places came out in another; host code too, so that it can be tried without a device.
#ifndef AP_RUNS_HPP
#define AP_RUNS_HPP

#include <cstdint>

#ifndef __HIP__
#define __host__
#define __device__
#endif

// Ascending order of list[0 .. n).
__host__ __device__ inline void sort_run(uint16_t* list, uint32_t n) {
    for (uint32_t i = 1; i < n; ++i) {
        const uint16_t v = list[i];
        uint32_t k = i;
        for (; k > 0u && list[k - 1u] > v; --k) list[k] = list[k - 1u];
        list[k] = v;
    }
}

#endif  // AP_RUNS_HPP
