// SAMD 2-D convolution for gfx950: convolution by long multiplication (Sec. 5) with
// signed sign-extension and the underflow fix-up (Sec. 6).
//
// Three kernels:
//  * prep_weights_kernel: every kernel row -> its kernel words (taps reversed, sign-
//    extended, L bits apart), laid out as one contiguous stream per group of kWaveM
//    output channels, so a wave walks its kernel words with scalar loads;
//  * spread_kernel: every packed input row -> operand words, I values of one stride
//    phase L bits apart (temporary spacer bits), negative values sign-extended, so that
//    each word is the int32 sum_i v_i 2^(i L); rows of the zero padding are written too;
//  * conv2d_samd_kernel: a workgroup owns a tile of output rows of one image and wm*8
//    output channels.  Every lane reads its operand words straight from the spread buffer
//    with raw buffer loads (L1/L2-resident: each word is reused by the workgroup's channel
//    waves and kernel rows), every wave holds its 8 kernel words of a step in SGPRs
//    (scalar loads from its kernel-word stream) and adds the exact signed 32x32 -> 64-bit
//    products into 64-bit accumulators (v_mad_i64_i32).  Every G channels the
//    accumulators are decoded - fix-up, lane extraction - and added into an LDS tile of
//    int32 outputs (the tile is the only LDS use), which also performs the overlap-add of
//    neighbouring words' partial lanes and sums the channel-split waves; finished rows
//    are stored from the tile.
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

// Operand words xs[n][c][hp][t][q] for padded rows hp in [0, H + 2 ph), of the
// activations minus xoff (recentred unsigned activations).  A block of 256
// threads covers 256 / QP padded rows (QP, a power of two of at most 256, about nq / 2.5
// threads per row): thread (row, q) builds words q, q + QP, ... of every kernel-word
// variant t of its row from the packed input row (L1-resident; rows of the zero padding
// give zeros).
template <int B, bool S>
__global__ __launch_bounds__(256) void spread_kernel(const uint32_t *__restrict__ x, const Conv2dGeom g, int qshift,
                                                     int32_t *__restrict__ xs) {
    constexpr int P = 32 / B;
    // 32-bit row indices: the planner keeps N * C * Hp below 2^31
    const uint32_t row = blockIdx.x * (256u >> qshift) + (threadIdx.x >> qshift);   // (n*C + c)*Hp + hp
    if (row >= (uint32_t)(g.N * g.C * g.Hp)) return;
    const uint32_t nc = row / (uint32_t)g.Hp;
    const int hp = (int)(row - nc * (uint32_t)g.Hp);
    const int h = hp - g.ph;
    const bool inside = h >= 0 && h < g.H;
    const uint32_t *src = x + ((int64_t)nc * g.H + (inside ? h : 0)) * g.xrw;
    const int32_t pad = conv2d_pad_value(g.xoff, g.layout_spaced);
    // words q, q + 2^qshift, ... of the row (one pass unless the row has more than 256)
    for (int q = threadIdx.x & ((1 << qshift) - 1); q < g.nq; q += 1 << qshift) {
        int32_t *dst = xs + (int64_t)row * g.ntw * g.nq + q;
        for (int t = 0; t < g.ntw; ++t) {
            const int delta = g.tw_tap0[t] + g.tw_ntaps[t] - g.Kmax;
            const int col0 = g.sw * (q * g.I + delta) + g.tw_phase[t] - g.pw;
            uint32_t word = 0;
            if (inside || pad != 0) {
                for (int ii = 0; ii < g.I; ++ii) {
                    const int col = col0 + g.sw * ii;
                    int32_t v = pad;
                    if (inside && col >= 0 && col < g.W) {
                        const uint32_t f = (src[col / P] >> ((col % P) * B)) & ((1u << B) - 1);
                        v = (S ? ((int32_t)(f << (32 - B)) >> (32 - B)) : (int32_t)f) - g.xoff;
                    }
                    word += (uint32_t)v << (ii * g.L);
                }
            }
            dst[t * g.nq] = (int32_t)word;
        }
    }
}

// The same operand words built from unpacked 8-bit values (int8 when S, else uint8; N C H W
// row-major) instead of packed rows: the permanent-spacer layout written straight from
// the values a caller holds.  Each value enters as its low b bits (sign-extended when S).
template <int B, bool S>
__global__ __launch_bounds__(256) void spread_bytes_kernel(const uint8_t *__restrict__ x, const Conv2dGeom g,
                                                           int qshift, int32_t *__restrict__ xs) {
    const uint32_t row = blockIdx.x * (256u >> qshift) + (threadIdx.x >> qshift);   // (n*C + c)*Hp + hp
    if (row >= (uint32_t)(g.N * g.C * g.Hp)) return;
    const uint32_t nc = row / (uint32_t)g.Hp;
    const int hp = (int)(row - nc * (uint32_t)g.Hp);
    const int h = hp - g.ph;
    const bool inside = h >= 0 && h < g.H;
    const uint8_t *src = x + ((int64_t)nc * g.H + (inside ? h : 0)) * g.W;
    for (int q = threadIdx.x & ((1 << qshift) - 1); q < g.nq; q += 1 << qshift) {
        int32_t *dst = xs + (int64_t)row * g.ntw * g.nq + q;
        for (int t = 0; t < g.ntw; ++t) {
            const int delta = g.tw_tap0[t] + g.tw_ntaps[t] - g.Kmax;
            const int col0 = g.sw * (q * g.I + delta) + g.tw_phase[t] - g.pw;
            uint32_t word = 0;
            if (inside) {
                for (int ii = 0; ii < g.I; ++ii) {
                    const int col = col0 + g.sw * ii;
                    if (col >= 0 && col < g.W) {
                        const uint32_t f = src[col] & ((1u << B) - 1);
                        const int32_t v = (S ? ((int32_t)(f << (32 - B)) >> (32 - B)) : (int32_t)f) - g.xoff;
                        word += (uint32_t)v << (ii * g.L);
                    }
                }
            }
            dst[t * g.nq] = (int32_t)word;
        }
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

int launch_conv2d_spread(const uint32_t *x, const Conv2dGeom &g, void *ws, hipStream_t s, int32_t *dst) {
    int32_t *xs = dst ? dst : (int32_t *)((char *)ws + conv2d_xs_offset(g));
    // 2^qshift threads per row, each building about 2.5 of its words (words q, q + 2^qshift,
    // ...): one word per thread was 5-23 % slower at the mid-size layer
    const int qshift = spread_qshift(g.nq);
    const int64_t nrows = (int64_t)g.N * g.C * g.Hp;
    const int rpb = 256 >> qshift;
    const int64_t blocks = (nrows + rpb - 1) / rpb;   // one thread group per row, no grid-stride loop
    // the planner refuses layers that would need 2^32 threads or more (addressable())
    if (blocks * 256 > (int64_t)0xffffffff) {
        set_error("conv2d operand spread: more than 2^32 threads in one launch");
        return SAMD_EUNSUPPORTED;
    }
    const unsigned sgrid = (unsigned)blocks;
    bool launched = false;
#define SAMD_SPREAD_CASE(B, SG)                                                                            \
    if (!launched && g.xbits == B && (bool)g.xsigned == SG) {                                              \
        hipLaunchKernelGGL((spread_kernel<B, SG>), dim3(sgrid), dim3(256), 0, s, x, g, qshift, xs);        \
        launched = true;                                                                                   \
    }
    SAMD_FOR_EACH_FMT(SAMD_SPREAD_CASE)
#undef SAMD_SPREAD_CASE
    return check_launch("conv2d operand spread");
}

int launch_conv2d_spread_bytes(const void *x, const Conv2dGeom &g, int32_t *dst, hipStream_t s) {
    const int qshift = spread_qshift(g.nq);
    const int64_t nrows = (int64_t)g.N * g.C * g.Hp;
    const int rpb = 256 >> qshift;
    const int64_t blocks = (nrows + rpb - 1) / rpb;
    // the planner refuses layers that would need 2^32 threads or more (addressable())
    if (blocks * 256 > (int64_t)0xffffffff) {
        set_error("conv2d spaced pack: more than 2^32 threads in one launch");
        return SAMD_EUNSUPPORTED;
    }
    // the stored values' format: signed when the activations are (recentred unsigned
    // activations are stored unsigned and shifted by xoff inside the kernel)
    const bool sgn = g.xsigned != 0;
    bool launched = false;
#define SAMD_SPREAD_BYTES_CASE(B, SG)                                                                    \
    if (!launched && g.xbits == B && sgn == SG) {                                                        \
        hipLaunchKernelGGL((spread_bytes_kernel<B, SG>), dim3((unsigned)blocks), dim3(256), 0, s,       \
                           (const uint8_t *)x, g, qshift, dst);                                          \
        launched = true;                                                                                 \
    }
    SAMD_FOR_EACH_FMT(SAMD_SPREAD_BYTES_CASE)
#undef SAMD_SPREAD_BYTES_CASE
    return check_launch("conv2d spaced pack");
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
    if (!g.rows_path)
        st = launch_multiply_general(g, y, ws, s, src);
    else if (g.KH == 5)
        st = launch_multiply_rows5(g, y, ws, s, src);
    else if (g.two)
        st = launch_multiply_rows3_wide(g, y, ws, s, src);
    else
        st = launch_multiply_rows3(g, y, ws, s, src);
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
