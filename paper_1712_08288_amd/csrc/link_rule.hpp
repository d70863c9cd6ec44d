// The free parameter l(gamma) of a cut link (paper, Section 3) and its band of
// Eq. (212), for the host's check of a new geometry and the device's link
// tables alike: rounded operation by operation, as written.
#pragma once

#include <hip/hip_runtime.h>

namespace lbe {

__host__ __device__ inline double l_of(int rule, double g) {
#pragma clang fp contract(off)
    switch (rule) {
        case 0: return g;
        case 1: return 1.5 * g;
        case 2: return 2.0 * g;
        case 3: return g * g;
        case 4: return g * g + g;
        case 5: return 0.0;
        default: return 2.0 * g - 1.0 > 0.0 ? 2.0 * g - 1.0 : 0.0;
    }
}
// dl/dgamma
__host__ __device__ inline double dl_of(int rule, double g) {
#pragma clang fp contract(off)
    switch (rule) {
        case 0: return 1.0;
        case 1: return 1.5;
        case 2: return 2.0;
        case 3: return 2.0 * g;
        case 4: return 2.0 * g + 1.0;
        case 5: return 0.0;
        default: return 2.0 * g - 1.0 > 0.0 ? 2.0 : 0.0;
    }
}
// max(0, 2 gamma - 1) <= l <= 2 gamma, Eq. (212)
__host__ __device__ inline bool l_convex(int rule, double g) {
    const double l = l_of(rule, g), lo = 2.0 * g - 1.0 > 0.0 ? 2.0 * g - 1.0 : 0.0;
    return l >= lo - 1e-12 && l <= 2.0 * g + 1e-12;
}

}  // namespace lbe
