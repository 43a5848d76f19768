// Operand words of the SAMD 2-D convolution: I values of one stride phase per 32-bit word, L
// bits apart (temporary spacer bits, Sec. 2.2), negative values sign-extended, for every row
// of the zero-padded image and every kernel-word variant: xs[n][c][hp][t][q], word q of
// variant t holding, lane i, the value of column sw (q I + delta_t + i) + phase_t - pw of row
// hp - ph, minus the recentring offset.  Written from packed rows, from 8-bit values, or
// from a layer's int32 accumulators (ReLU and requantisation fused in).
//
// One kernel for the three sources.  A workgroup takes a run of consecutive padded rows:
//   1. their fields go into LDS, one row of BC-bit fields per padded row, with zero fields to
//      both sides and in the rows outside the image - the only reads of global memory, all
//      in flight together;
//   2. each thread builds four consecutive words of a row and stores them in one 16-byte
//      store, row after row, so the words leave in runs of whole lines.
// A stride-1 word's I fields are cut from two neighbouring LDS words with one funnel shift
// and placed with two instructions each.
// The earlier kernel gave each padded row a few threads that read their values one by one
// from global memory: the reads' latency, one after the other, about 12 instructions per
// value and stores of half lines set its time.  Before and after, from packed rows: 13.8 MB
// of words (8 x 128 x 56 x 56, 5 to 8 bits) 9.4 and 7.5 us (a plain fill of the same bytes
// takes 4.3), 81 MB 38.7 and 21.6 us; from accumulators: 10.4 and 8.5 us, 45.4 and 28.3 us.
#include <hip/hip_runtime.h>

#include <climits>

#include "hip_util.hpp"

namespace samd {

namespace {

constexpr int kBlock = 256;
constexpr int kMaxRowLds = 32768;   // LDS bytes of a workgroup's rows

enum { kFromPacked, kFromBytes, kFromAccumulators };

struct SpreadArgs {
    int32_t H, W, Hp, ph, pw, sw, I, L, nq, ntw, xrw, xoff, xbits;
    int32_t rw;                    // words of a padded row, ntw * nq
    int32_t R;                     // padded rows per workgroup
    int32_t load_rows, word_rows;  // rows a workgroup's threads read, and build, side by side
    int32_t ls, margin;            // LDS words of a row (its last word: 1 inside the image), words before its first field
    int32_t funnel;                // stride 1 and I fields within two LDS words
    int32_t zero_pad;              // lanes outside the image are 0 although activations are recentred
    uint32_t base;                 // what every word of the recentred form takes off: xoff * sum_i 2^(i L)
    int64_t nrows;                 // N * C * Hp
    Division by_nq, by_quads, by_ls, by_Hp;
    int32_t shift0[kMaxTapWords];  // first column of word 0 of variant t: sw delta_t + phase_t - pw
};

__device__ __forceinline__ uint32_t div_by(uint32_t n, const Division &d) { return (uint32_t)(((uint64_t)n * d.mul) >> d.shift); }

// Four consecutive words, stored at once wherever they start.
typedef uint32_t Words4 __attribute__((ext_vector_type(4), aligned(4)));
// Four values of a byte row, read at once wherever they lie.
typedef uint32_t Word1 __attribute__((aligned(1)));

template <int BC, int SRC, bool S>
__global__ __launch_bounds__(kBlock) void spread_rows_kernel(const void *__restrict__ src, const SpreadArgs a,
                                                             int32_t *__restrict__ xs,
                                                             const int32_t *__restrict__ dev_max,
                                                             int32_t *__restrict__ dev_shift) {
    constexpr int P = 32 / BC;   // fields per LDS word
    extern __shared__ uint32_t rows[];
    __shared__ int32_t first[kMaxTapWords];   // shift0, where lanes can index it
    const int tid = threadIdx.x;
    if (tid < kMaxTapWords) first[tid] = a.shift0[tid];
    const int64_t r0 = (int64_t)blockIdx.x * a.R;
    const int R = (int)min((int64_t)a.R, a.nrows - r0);
    int shift = 0;
    if constexpr (SRC == kFromAccumulators) {
        shift = requant_shift(*dev_max, a.xbits);
        if (dev_shift && blockIdx.x == 0 && tid == 0) *dev_shift = shift;
    }
    // fields into LDS: a thread keeps its word of a row and walks down the rows
    const int ls = a.ls;
    {
        const int r = ls <= kBlock ? div_by(tid, a.by_ls) : 0;
        for (int c = tid - r * ls; c < ls && r < a.load_rows; c += kBlock) {
            const int w = c - a.margin;
            const int live = min(P, a.W - w * P);   // fields of this word
            const bool fields = w >= 0 && live > 0 && c < ls - 1;
#pragma unroll 2
            for (int i = r; i < R; i += a.load_rows) {
                const uint32_t row = (uint32_t)(r0 + i);   // below 2^31
                const uint32_t nc = div_by(row, a.by_Hp);
                const int h = (int)(row - nc * a.Hp) - a.ph;
                const bool inside = h >= 0 && h < a.H;
                uint32_t v = c == ls - 1 && inside ? 1 : 0;
                if (inside && fields) {
                    const int64_t line = (int64_t)nc * a.H + h;
                    if constexpr (SRC == kFromPacked) {
                        const int bits = live * BC;
                        v = ((const uint32_t *)src)[line * a.xrw + w] & (bits >= 32 ? 0xffffffffu : (1u << bits) - 1);
                    } else if constexpr (SRC == kFromBytes) {
                        // the row's last bytes as the end of the four that end there, so that every
                        // word is one read (8 x 61 x 108 x 402, 5x5, stride 4: 33.2 us byte by
                        // byte, 28.5 with the last word byte by byte, 21.9)
                        const uint8_t *s = (const uint8_t *)src + line * a.W + w * P;
                        if (a.W >= P) {
                            v = *(const Word1 *)(s - (P - live)) >> (8 * (P - live));
                        } else {
#pragma unroll
                            for (int e = 0; e < P - 1; ++e)
                                if (e < live) v |= (uint32_t)s[e] << (8 * e);
                        }
                    } else {
                        const int32_t *s = (const int32_t *)src + line * a.W + w * P;
                        int32_t q[P];
                        if (live == P) {
                            const Words4 four = *(const Words4 *)s;
#pragma unroll
                            for (int e = 0; e < P; ++e) q[e] = (int32_t)four[e];
                        } else {
#pragma unroll
                            for (int e = 0; e < P; ++e) q[e] = e < live ? s[e] : 0;
                        }
#pragma unroll
                        for (int e = 0; e < P; ++e) v |= requant(q[e], shift, a.xbits) << (8 * e);
                    }
                }
                rows[i * ls + c] = v;
            }
        }
    }
    __syncthreads();

    // words: a thread keeps its four words of a row - where their fields lie is the same in
    // every row - and walks down the rows
    const int I = a.I, L = a.L, rw = a.rw, quads = (rw + 3) / 4, xbits = SRC == kFromPacked ? BC : a.xbits;
    const int r = quads <= kBlock ? div_by(tid, a.by_quads) : 0;
    if (r >= a.word_rows) return;
    for (int quad = tid - r * quads; quad < quads; quad += kBlock) {
        int32_t *out = xs + r0 * rw + 4 * quad;
        const int nw = min(4, rw - 4 * quad);
        int at[4], sh[4], col0[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int f = min(4 * quad + e, rw - 1);
            const int t = div_by(f, a.by_nq), q = f - t * a.nq;
            // the word's first column, and the LDS word and bit of its field
            col0[e] = first[t] + a.sw * q * I;
            const uint32_t col = (uint32_t)(col0[e] + a.margin * P);
            at[e] = col / P;
            sh[e] = (col - at[e] * P) * BC;
        }
        for (int i = r; i < R; i += a.word_rows) {
            const uint32_t *row = rows + i * ls;
            uint32_t word[4] = {0u - a.base, 0u - a.base, 0u - a.base, 0u - a.base};
            if (a.funnel) {
                uint32_t bits[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t w0 = row[at[e]], w1 = row[at[e] + 1];
                    uint32_t lo = w0, hi = w1;
                    if constexpr (P * BC < 32) {
                        lo = w0 | (w1 << (P * BC));
                        hi = w1 >> (32 - P * BC);
                    }
                    bits[e] = __builtin_amdgcn_alignbit(hi, lo, sh[e]);
                }
                for (int ii = 0; ii < I; ++ii) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const uint32_t v = S ? (uint32_t)((int32_t)(bits[e] << (32 - xbits)) >> (32 - xbits))
                                             : bits[e] & ((1u << xbits) - 1);
                        word[e] += v << (ii * L);
                        bits[e] >>= BC;
                    }
                }
            } else {
                for (int ii = 0; ii < I; ++ii) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int col = col0[e] + a.sw * ii;
                        const bool in = col >= 0 && col < a.W;
                        const uint32_t k = (uint32_t)(in ? col : 0) / P;
                        uint32_t v = row[a.margin + k] >> (((in ? col : 0) - k * P) * BC);
                        v = S ? (uint32_t)((int32_t)(v << (32 - xbits)) >> (32 - xbits)) : v & ((1u << xbits) - 1);
                        word[e] += (in ? v : 0u) << (ii * L);
                    }
                }
            }
            if (a.zero_pad) {   // lanes outside the image back to 0
                const bool inside = row[ls - 1] != 0;
                for (int ii = 0; ii < I; ++ii) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int col = col0[e] + a.sw * ii;
                        if (!inside || col < 0 || col >= a.W) word[e] += (uint32_t)a.xoff << (ii * L);
                    }
                }
            }
            int32_t *o = out + i * rw;
            if (nw == 4) {
                *(Words4 *)o = Words4{word[0], word[1], word[2], word[3]};
            } else {
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    if (e < nw) o[e] = (int32_t)word[e];
            }
        }
    }
}

// Rows whose fields do not fit a workgroup's LDS (tens of thousands of columns), and layers
// of a few thousand words: a block of
// 256 threads covers 256 / QP padded rows (QP, a power of two of at most 256, about nq / 2.5
// threads per row); thread (row, q) builds words q, q + QP, ... of every kernel-word variant
// of its row, reading its values one by one.
template <int SRC, int BC, bool S>
__global__ __launch_bounds__(kBlock) void spread_direct_kernel(const void *__restrict__ src, const SpreadArgs a,
                                                             int qshift, int32_t *__restrict__ xs,
                                                             const int32_t *__restrict__ dev_max,
                                                             int32_t *__restrict__ dev_shift) {
    constexpr int P = 32 / BC;
    int shift = 0;
    if constexpr (SRC == kFromAccumulators) {
        shift = requant_shift(*dev_max, a.xbits);
        if (dev_shift && blockIdx.x == 0 && threadIdx.x == 0) *dev_shift = shift;
    }
    const uint32_t row = blockIdx.x * ((uint32_t)kBlock >> qshift) + (threadIdx.x >> qshift);   // (n*C + c)*Hp + hp
    if (row >= (uint32_t)a.nrows) return;
    const uint32_t nc = div_by(row, a.by_Hp);
    const int h = (int)(row - nc * a.Hp) - a.ph;
    const bool inside = h >= 0 && h < a.H;
    const int64_t line = (int64_t)nc * a.H + (inside ? h : 0);
    const int32_t outside = a.zero_pad ? 0 : -a.xoff;
    const int bits = SRC == kFromPacked ? BC : a.xbits;
    for (int q = threadIdx.x & ((1 << qshift) - 1); q < a.nq; q += 1 << qshift) {
        for (int t = 0; t < a.ntw; ++t) {
            uint32_t word = 0;
            for (int ii = 0; ii < a.I; ++ii) {
                const int col = a.shift0[t] + a.sw * (q * a.I + ii);
                int32_t v = outside;
                if (inside && col >= 0 && col < a.W) {
                    uint32_t f;
                    if constexpr (SRC == kFromPacked)
                        f = ((const uint32_t *)src)[line * a.xrw + col / P] >> ((col % P) * BC);
                    else if constexpr (SRC == kFromBytes)
                        f = ((const uint8_t *)src)[line * a.W + col];
                    else
                        f = requant(((const int32_t *)src)[line * a.W + col], shift, a.xbits);
                    v = (S ? (int32_t)(f << (32 - bits)) >> (32 - bits) : (int32_t)(f & ((1u << bits) - 1))) - a.xoff;
                }
                word += (uint32_t)v << (ii * a.L);
            }
            xs[((int64_t)row * a.ntw + t) * a.nq + q] = (int32_t)word;
        }
    }
}

// BC: bits of a field in LDS (the packed width, or 8)
template <int BC, int SRC, bool S>
int launch_spread(const void *src, const Conv2dGeom &g, int32_t *dst, const int32_t *dev_max, int32_t *dev_shift,
                  const char *what, hipStream_t s) {
    constexpr int P = 32 / BC;
    SpreadArgs a = {};
    a.H = g.H; a.W = g.W; a.Hp = g.Hp; a.ph = g.ph; a.pw = g.pw; a.sw = g.sw; a.I = g.I; a.L = g.L;
    a.nq = g.nq; a.ntw = g.ntw; a.xrw = g.xrw; a.xoff = g.xoff; a.xbits = g.xbits;
    a.rw = g.ntw * g.nq;
    a.nrows = (int64_t)g.N * g.C * g.Hp;
    a.zero_pad = g.xoff != 0 && conv2d_pad_value(g.xoff, g.layout_spaced) == 0;
    int lo = 0, hi = 0;   // columns a word's lanes reach, stride 1
    for (int t = 0; t < g.ntw; ++t) {
        a.shift0[t] = g.sw * (g.tw_tap0[t] + g.tw_ntaps[t] - g.Kmax) + g.tw_phase[t] - g.pw;
        lo = std::min(lo, a.shift0[t]);
        hi = std::max(hi, a.shift0[t] + g.nq * g.I);
    }
    for (int i = 0; i < g.I; ++i) a.base += (uint32_t)g.xoff << (i * g.L);
    a.funnel = g.sw == 1 && g.I <= P;
    a.margin = a.funnel ? (-lo + P - 1) / P : 0;
    const int64_t fields = (g.W + P - 1) / P;   // LDS words of a row's fields
    // the funnel reads the word after a word's first field; then the row's inside flag
    const int64_t ls = (a.funnel ? std::max<int64_t>(a.margin + fields, a.margin + (hi + P - 1) / P + 1) : fields) + 1;
    // rows per workgroup: the rows its threads build side by side, once for layers that fill
    // the chip with about that many workgroups, up to four times for larger ones (13.8 MB of
    // words: 8.9, 7.7 and 7.5 us for 1, 2 and 4; 3.6 MB: 4.6, 4.7 and 5.5 us)
    const int64_t quads = (a.rw + 3) / 4;
    const int64_t side = quads <= kBlock ? kBlock / quads : 1;
    const int64_t most = kMaxRowLds / 4 / ls;
    const int64_t passes = std::max<int64_t>(1, std::min<int64_t>(4, a.nrows / (side * 900)));
    const int64_t R = std::min<int64_t>(passes * side, most);
    const int64_t two31 = (int64_t)1 << 31;
    // a few thousand words take one chain of reads and stores rather than two phases (5184
    // words: 2.9 against 3.3 us)
    if (R < 1 || R * a.rw >= two31 || a.nrows * a.rw <= 16384) {
        const int qshift = spread_qshift(g.nq);
        const int rpb = kBlock >> qshift;
        const int64_t blocks = (a.nrows + rpb - 1) / rpb;
        // the planner refuses layers that would need 2^32 threads or more (addressable())
        if (blocks * kBlock > (int64_t)0xffffffff) {
            set_error(std::string(what) + ": more than 2^32 threads in one launch");
            return SAMD_EUNSUPPORTED;
        }
        a.by_Hp = division(g.Hp);
        hipLaunchKernelGGL((spread_direct_kernel<SRC, BC, S>), dim3((unsigned)blocks), dim3(kBlock), 0, s, src, a, qshift,
                           dst, dev_max, dev_shift);
        return check_launch(what);
    }
    a.R = (int32_t)R;
    a.ls = (int32_t)ls;
    a.load_rows = ls <= kBlock ? (int32_t)(kBlock / ls) : 1;
    a.word_rows = (int32_t)side;
    a.by_nq = division(g.nq); a.by_quads = division((uint32_t)quads); a.by_ls = division(a.ls); a.by_Hp = division(g.Hp);
    const int64_t blocks = (a.nrows + R - 1) / R;
    if (blocks * kBlock > (int64_t)0xffffffff) {
        set_error(std::string(what) + ": more than 2^32 threads in one launch");
        return SAMD_EUNSUPPORTED;
    }
    hipLaunchKernelGGL((spread_rows_kernel<BC, SRC, S>), dim3((unsigned)blocks), dim3(kBlock), (size_t)R * ls * 4, s, src,
                       a, dst, dev_max, dev_shift);
    return check_launch(what);
}

}  // namespace

int launch_conv2d_spread(const uint32_t *x, const Conv2dGeom &g, void *ws, hipStream_t s, int32_t *dst) {
    int32_t *xs = dst ? dst : (int32_t *)((char *)ws + conv2d_xs_offset(g));
#define SAMD_SPREAD_CASE(B, SG)                                                                        \
    if (g.xbits == B && (bool)g.xsigned == SG)                                                         \
        return launch_spread<B, kFromPacked, SG>(x, g, xs, nullptr, nullptr, "conv2d operand spread", s);
    SAMD_FOR_EACH_FMT(SAMD_SPREAD_CASE)
#undef SAMD_SPREAD_CASE
    set_error("conv2d operand spread: unsupported format");
    return SAMD_EINVAL;
}

int launch_conv2d_spread_bytes(const void *x, const Conv2dGeom &g, int32_t *dst, hipStream_t s) {
    // the stored values' format: signed when the activations are (recentred unsigned
    // activations are stored unsigned and shifted by xoff inside the kernel)
    return g.xsigned ? launch_spread<8, kFromBytes, true>(x, g, dst, nullptr, nullptr, "conv2d spaced pack", s)
                     : launch_spread<8, kFromBytes, false>(x, g, dst, nullptr, nullptr, "conv2d spaced pack", s);
}

int launch_relu_requant_stage(const int32_t *acc, const int32_t *dev_max, const Conv2dGeom &g, void *ws,
                              int32_t *dev_shift, hipStream_t s, int32_t *dst) {
    int32_t *xs = dst ? dst : (int32_t *)((char *)ws + conv2d_xs_offset(g));
    return launch_spread<8, kFromAccumulators, false>(acc, g, xs, dev_max, dev_shift, "relu_requant_stage", s);
}

}  // namespace samd
