// Multiply kernels of 3-row stride-1 layers whose lanes are decoded into the tile.
#include "conv2d_multiply.hpp"

namespace samd {

int launch_multiply_rows3(const Conv2dGeom &g, int32_t *y, const void *ws, hipStream_t s, const int32_t *src) {
    if (g.rh == 1 && g.two == 0) return launch_multiply_shape<1, 3, 0>(g, y, ws, s, src);
    if (g.rh == 2 && g.two == 0) return launch_multiply_shape<2, 3, 0>(g, y, ws, s, src);
    if (g.rh == 3 && g.two == 0) return launch_multiply_shape<3, 3, 0>(g, y, ws, s, src);
    if (g.rh == 4 && g.two == 0) return launch_multiply_shape<4, 3, 0>(g, y, ws, s, src);
    return kNoInstance;
}

}  // namespace samd
