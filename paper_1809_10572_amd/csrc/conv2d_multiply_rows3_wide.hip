// Multiply kernels of 3-row stride-1 layers with two-level lanes.
#include "conv2d_multiply.hpp"

namespace samd {

int launch_multiply_rows3_wide(const Conv2dGeom &g, int32_t *y, const void *ws, hipStream_t s, const int32_t *src) {
    if (g.rh == 1 && g.two == 1) return launch_multiply_shape<1, 3, 1>(g, y, ws, s, src);
    if (g.rh == 1 && g.two == 2) return launch_multiply_shape<1, 3, 2>(g, y, ws, s, src);
    if (g.rh == 2 && g.two == 1) return launch_multiply_shape<2, 3, 1>(g, y, ws, s, src);
    if (g.rh == 2 && g.two == 2) return launch_multiply_shape<2, 3, 2>(g, y, ws, s, src);
    return kNoInstance;
}

}  // namespace samd
