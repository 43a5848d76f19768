// Helpers shared by the HIP translation units of the library.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>

#include "samd_internal.hpp"

namespace samd {

// Blocks for a grid-stride loop over `items`, capped so huge inputs loop instead.
inline int grid_for(int64_t items, int block) {
    int64_t blocks = (items + block - 1) / block;
    return (int)std::min<int64_t>(std::max<int64_t>(blocks, 1), 65536);
}

// Map a failed launch to SAMD_EHIP with the runtime's message.
inline int check_launch(const char *what) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        set_error(std::string(what) + ": " + hipGetErrorString(e));
        return SAMD_EHIP;
    }
    return SAMD_OK;
}

// n / d = (n * mul) >> shift for 0 <= n < 2^31: divisions by launch constants as
// multiplications.
struct Division {
    uint32_t mul, shift;
};

inline Division division(uint32_t d) {
    uint32_t s = 0;
    while (((uint64_t)1 << s) < d) ++s;
    return {(uint32_t)((((uint64_t)1 << (31 + s)) + d - 1) / d), 31 + s};
}

// Requantisation shift for a layer maximum.
__device__ inline int requant_shift(int32_t layer_max, int bits) {
    const uint32_t mx = layer_max > 0 ? (uint32_t)layer_max : 0u;
    const int len = 32 - __clz(mx);   // bit length, 0 for 0
    return len > bits ? len - bits : 0;
}

// ReLU and requantisation of one accumulator.  All in 32 bits: the value is below 2^31 and
// half a step below 2^30, so their sum fits an unsigned word.
__device__ inline uint32_t requant(int32_t v, int shift, int bits) {
    const uint32_t half = shift ? 1u << (shift - 1) : 0u;
    return min(((uint32_t)max(v, 0) + half) >> shift, (1u << bits) - 1);
}

// Expands MACRO(bits, signed) for every operand format.
#define SAMD_FOR_EACH_FMT(MACRO)                                                                    \
    MACRO(1, false) MACRO(2, false) MACRO(3, false) MACRO(4, false) MACRO(5, false) MACRO(6, false) \
    MACRO(7, false) MACRO(8, false) MACRO(1, true) MACRO(2, true) MACRO(3, true) MACRO(4, true)     \
    MACRO(5, true) MACRO(6, true) MACRO(7, true) MACRO(8, true)

}  // namespace samd
