// Multiply kernels of layers without shared rows whose channels are whole batches of steps.
#include "conv2d_multiply.hpp"

namespace samd {

int launch_multiply_batches(const Conv2dGeom &g, int32_t *y, const void *ws, hipStream_t s, const int32_t *src) {
    if (g.rh == 1 && g.two == 0) return launch_multiply_shape<1, 1, 0>(g, y, ws, s, src);
    if (g.rh == 1 && g.two == 1) return launch_multiply_shape<1, 1, 1>(g, y, ws, s, src);
    if (g.rh == 1 && g.two == 2) return launch_multiply_shape<1, 1, 2>(g, y, ws, s, src);
    if (g.rh == 2 && g.two == 0) return launch_multiply_shape<2, 1, 0>(g, y, ws, s, src);
    if (g.rh == 2 && g.two == 1) return launch_multiply_shape<2, 1, 1>(g, y, ws, s, src);
    if (g.rh == 2 && g.two == 2) return launch_multiply_shape<2, 1, 2>(g, y, ws, s, src);
    return kNoInstance;
}

}  // namespace samd
