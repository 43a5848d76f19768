// SAMD 2-D convolution for gfx950: convolution by long multiplication (Sec. 5) with
// signed sign-extension and the underflow fix-up (Sec. 6).
//
// The weights' side and the launchers:
//  * prep_weights_kernel: every kernel row -> its kernel words (taps reversed, sign-
//    extended, L bits apart), laid out as one contiguous stream per group of kWaveM
//    output channels, so a wave walks its kernel words with scalar loads;
//  * filter_sum_kernel, prefix_kernel: the correction of recentred activations.
// Operand words are written by conv2d_spread.hip and multiplied by the kernel of
// conv2d_multiply.hpp.
#include <hip/hip_runtime.h>

#include <climits>
#include <map>
#include <mutex>
#include <tuple>

#include "conv2d_multiply.hpp"
#include "hip_util.hpp"

namespace samd {

namespace {

template <int B, bool S>
__device__ inline int32_t packed_field(const uint32_t *row, int col) {
    constexpr int P = 32 / B;
    const uint32_t f = (row[col / P] >> ((col % P) * B)) & ((1u << B) - 1);
    if (S) return (int32_t)(f << (32 - B)) >> (32 - B);
    return (int32_t)f;
}

// Kernel-word stream of output-channel group wb: step s = c*nrt + ky*ntw + t (or
// c*nrt + t*KH + ky on the shared-row path) holds the kWaveM words of kernel word t of
// row ky of channel c; kStreamPad zero steps pad the end.
// Also zeroes the multiply kernel's ticket counters.
template <int B, bool S>
__global__ __launch_bounds__(256) void prep_weights_kernel(const uint32_t *__restrict__ w, const Conv2dGeom g,
                                                           int32_t *__restrict__ kw, int32_t *__restrict__ queue) {
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < kQueueBytes / 4; i += 256) queue[i] = 0;
    const int64_t steps = (int64_t)g.C * g.nrt + kStreamPad;
    for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < g.kw_words; idx += (int64_t)gridDim.x * 256) {
        const int mm = (int)(idx % RM);
        const int64_t s = (idx / RM) % steps;
        const int64_t wb = idx / (RM * steps);
        const int m = (int)(wb * RM + mm);
        uint32_t word = 0;
        if (m < g.M && s < (int64_t)g.C * g.nrt) {
            const int c = (int)(s / g.nrt), rt = (int)(s % g.nrt);
            // steps of a channel: kernel-row-major, or kernel-word-major for the
            // shared-row path
            const int ky = g.rows_path ? rt % g.KH : rt / g.ntw, t = g.rows_path ? rt / g.KH : rt % g.ntw;
            const uint32_t *row = w + (((int64_t)m * g.C + c) * g.KH + ky) * g.wrw;
            const int k = g.tw_ntaps[t], a0 = g.tw_tap0[t], r = g.tw_phase[t];
            for (int si = 0; si < k; ++si) {
                const int tap = g.sw * (a0 + k - 1 - si) + r;   // reversed: lane si holds tap a0+k-1-si
                word += (uint32_t)packed_field<B, S>(row, tap) << (si * g.L);
            }
        }
        kw[idx] = (int32_t)word;
    }
}

// Correction of recentred activations whose padding is recentred too (the packed layout):
// sum[m] = xoff * (the sum of channel m's weights), one wave per output channel.
template <int B, bool S>
__global__ __launch_bounds__(256) void filter_sum_kernel(const uint32_t *__restrict__ w, const Conv2dGeom g,
                                                         int32_t *__restrict__ sum) {
    const int lane = threadIdx.x & 63;
    const int64_t rows = (int64_t)g.C * g.KH;
    for (int64_t m = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); m < g.M; m += (int64_t)gridDim.x * 4) {
        int32_t s = 0;
        for (int64_t r = lane; r < rows; r += 64) {
            const uint32_t *row = w + (m * rows + r) * g.wrw;
            for (int kx = 0; kx < g.KW; ++kx) s += packed_field<B, S>(row, kx);
        }
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
        if (lane == 0) sum[m] = g.xoff * s;
    }
}

// Correction table of recentred activations in the permanent-spacer layout: pre[m][i][j] = sum of w[m][c][ky][kx] over
// all c, ky < i, kx < j (i <= KH, j <= KW), so an output's in-image taps [ky0, ky1) x
// [kx0, kx1) sum to a rectangle of four entries.
template <int B, bool S>
__global__ __launch_bounds__(256) void prefix_kernel(const uint32_t *__restrict__ w, const Conv2dGeom g,
                                                     int32_t *__restrict__ pre) {
    const int pwid = (g.KH + 1) * (g.KW + 1);
    const int64_t total = (int64_t)g.M * pwid;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
        const int m = (int)(e / pwid), ij = (int)(e - (int64_t)m * pwid);
        const int i = ij / (g.KW + 1), j = ij - i * (g.KW + 1);
        int32_t sum = 0;
        for (int c = 0; c < g.C; ++c)
            for (int ky = 0; ky < i; ++ky) {
                const uint32_t *row = w + (((int64_t)m * g.C + c) * g.KH + ky) * g.wrw;
                for (int kx = 0; kx < j; ++kx) sum += packed_field<B, S>(row, kx);
            }
        pre[e] = sum;
    }
}

}  // namespace

int launch_conv2d_prepare(const uint32_t *w, const Conv2dGeom &g, void *ws, hipStream_t s) {
    int32_t *kw = (int32_t *)ws;
    int32_t *queue = (int32_t *)((char *)ws + conv2d_queue_offset(g));
    const int pgrid = grid_for(g.kw_words, 256);
    bool launched = false;
#define SAMD_PREP_CASE(B, SG)                                                                            \
    if (!launched && g.wbits == B && (bool)g.wsigned == SG) {                                            \
        hipLaunchKernelGGL((prep_weights_kernel<B, SG>), dim3(pgrid), dim3(256), 0, s, w, g, kw, queue);        \
        launched = true;                                                                                 \
    }
    SAMD_FOR_EACH_FMT(SAMD_PREP_CASE)
#undef SAMD_PREP_CASE
    int st = check_launch("conv2d weight preparation");
    if (st || !g.xoff) return st;
    int32_t *pre = (int32_t *)((char *)ws + conv2d_kw_bytes(g));
    const bool table = conv2d_pad_value(g.xoff, g.layout_spaced) == 0;
    const int fgrid = table ? grid_for((int64_t)g.M * (g.KH + 1) * (g.KW + 1), 256) : grid_for(g.M, 4);
    launched = false;
#define SAMD_PREFIX_CASE(B, SG)                                                                          \
    if (!launched && g.wbits == B && (bool)g.wsigned == SG) {                                            \
        if (table)                                                                                       \
            hipLaunchKernelGGL((prefix_kernel<B, SG>), dim3(fgrid), dim3(256), 0, s, w, g, pre);         \
        else                                                                                             \
            hipLaunchKernelGGL((filter_sum_kernel<B, SG>), dim3(fgrid), dim3(256), 0, s, w, g, pre);     \
        launched = true;                                                                                 \
    }
    SAMD_FOR_EACH_FMT(SAMD_PREFIX_CASE)
#undef SAMD_PREFIX_CASE
    return check_launch("conv2d correction table");
}

int resident_workgroups(const void *kernel, int block, size_t shm, int &out) {
    static std::mutex mu;
    static std::map<std::tuple<int, const void *, int, size_t>, int> cache;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        set_error("conv2d: hipGetDevice failed");
        return SAMD_EHIP;
    }
    const auto key = std::make_tuple(dev, kernel, block, shm);
    {
        std::lock_guard<std::mutex> lock(mu);
        auto it = cache.find(key);
        if (it != cache.end()) {
            out = it->second;
            return SAMD_OK;
        }
    }
    int per_cu = 0, cus = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, block, shm);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) {
        set_error(std::string("conv2d: occupancy query: ") + hipGetErrorString(e));
        return SAMD_EHIP;
    }
    out = std::max(1, per_cu) * std::max(1, cus);
    std::lock_guard<std::mutex> lock(mu);
    cache[key] = out;
    return SAMD_OK;
}

int launch_conv2d_multiply(const Conv2dGeom &g, int32_t *y, const void *ws, hipStream_t s, const int32_t *src) {
    int st = kNoInstance;
    switch (conv2d_kernel_rows(g)) {
        case 0: st = launch_multiply_general(g, y, ws, s, src); break;
        case 1: st = launch_multiply_batches(g, y, ws, s, src); break;
        case 3: st = g.two ? launch_multiply_rows3_wide(g, y, ws, s, src) : launch_multiply_rows3(g, y, ws, s, src); break;
        case 5: st = launch_multiply_rows5(g, y, ws, s, src); break;
    }
    if (st != kNoInstance) return st;
    set_error("conv2d: no kernel for this geometry");
    return SAMD_EUNSUPPORTED;
}

int launch_conv2d_samd(const uint32_t *x, const Conv2dGeom &g, int32_t *y, const void *ws, hipStream_t s) {
    const int st = launch_conv2d_spread(x, g, const_cast<void *>(ws), s, nullptr);
    if (st) return st;
    return launch_conv2d_multiply(g, y, ws, s, nullptr);
}

}  // namespace samd
