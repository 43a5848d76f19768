// The multiply kernel of the SAMD 2-D convolution: operand words x kernel words, exact
// 64-bit products accumulated over input channels, lanes decoded and overlap-added, int32
// outputs stored.  A template over the launch shapes; its instances are compiled in
// conv2d_multiply_*.hip and picked by launch_conv2d_multiply (conv2d_samd.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <climits>

#include "hip_util.hpp"

namespace samd {

// Workgroups of `kernel` the current device keeps resident at once (all compute units),
// looked up once per (device, kernel, block, LDS bytes).
int resident_workgroups(const void *kernel, int block, size_t shm, int &out);

// One function per compiled group of kernels: launches the instance for g, or returns
// kNoInstance.
constexpr int kNoInstance = 1;
int launch_multiply_rows3(const Conv2dGeom &g, int32_t *y, const void *ws, hipStream_t s, const int32_t *src);
int launch_multiply_rows3_wide(const Conv2dGeom &g, int32_t *y, const void *ws, hipStream_t s, const int32_t *src);
int launch_multiply_rows5(const Conv2dGeom &g, int32_t *y, const void *ws, hipStream_t s, const int32_t *src);
int launch_multiply_batches(const Conv2dGeom &g, int32_t *y, const void *ws, hipStream_t s, const int32_t *src);
int launch_multiply_general(const Conv2dGeom &g, int32_t *y, const void *ws, hipStream_t s, const int32_t *src);

namespace {

constexpr int RM = kWaveM;

// What a launch needs, laid out in the order the kernel's phases read it.  The kernel reads
// it through the constant address space, phase by phase (args_again), so that a phase's
// values are loaded when it starts instead of being kept - in scalar registers, then in
// vector lanes - across the multiply loop.  Divisions by launch constants are
// multiplications: the item and lane set-up took about 550 instructions, 2 us of every
// launch, when it divided.
struct MultiplyArgs {
    // items and lanes
    const int32_t *xs, *kw;
    unsigned long long *tickets;
    int32_t tiles, nmb, nwg, ncs, row_tiles, wm;
    Division by_nmb, by_ncs, by_row_tiles;
    int32_t waves, wm_mul, nqs_mul;       // x / wm = (x * wm_mul) >> 16 for the few waves, likewise lanes by nqs
    int32_t nqs, groups, rows_blk, C;
    int32_t nq, ntw, nrt, Hp;
    int32_t Ho, sh, qseg, cpw, period, lds_tile;
    int64_t stream_len;                        // kernel words of one output-channel group
    uint64_t bias, odd_mask;
    // decode
    uint64_t msb_mask;
    int32_t L, nl, spacer, I, tile_rows, tile_row;
    // output
    int32_t *y;
    const int32_t *pre;
    uint64_t recip_lo, recip_hi;               // 2^64 / T (rounded down) for an XCD of the fewer, the more tiles
    int32_t rows_mul;                          // x / rows_blk = (x * rows_mul) >> 16 for the few waves
    int32_t mblk, M, Wo, cw, Kmax, xoff, pad_filled;
    int32_t KH, KW, H, W, ph, pw, sw;
};
typedef const MultiplyArgs __attribute__((address_space(4))) *ArgsPtr;

// The arguments again, opaque to the compiler: nothing read through the result moves to
// before this point.
__device__ __forceinline__ ArgsPtr args_again(ArgsPtr a) {
    asm volatile("" : "+s"(a));
    return a;
}

__device__ __forceinline__ int divide(int n, uint32_t mul, uint32_t shift) {
    return (int)(((uint64_t)(uint32_t)n * mul) >> shift);
}

// Operand words are read through a buffer resource over one image's operand words: the
// per-lane byte offset is a VGPR, the per-step offset an SGPR (no address arithmetic in
// the vector unit).  Word 3 is the gfx9 raw-buffer format (32-bit data, no swizzle).
constexpr int kBufferWord3 = 0x00020000;

__device__ __forceinline__ int32_t buffer_word(__amdgpu_buffer_rsrc_t r, int lane_bytes, int step_bytes) {
    return __builtin_amdgcn_raw_buffer_load_b32(r, lane_bytes, step_bytes, 0);
}

// Kernel words are read through the constant address space, which makes their loads scalar
// (nothing writes them while the kernel runs).
typedef const int32_t __attribute__((address_space(4))) *KernelWords;

// Empty register barrier: the accumulator is treated as rewritten here, so the products
// of successive steps cannot be summed first and added afterwards (integer addition is
// associative, and that rewrite costs one extra 64-bit add per batch); every product
// stays one v_mad_i64_i32 into its accumulator.
__device__ __forceinline__ void keep(int64_t &acc) { asm volatile("" : "+v"(acc)); }

// Waits for the wave's scalar and LDS operations (lgkmcnt 0), not for vector loads.
__device__ __forceinline__ void wait_scalar() { __builtin_amdgcn_s_waitcnt(0xc07f); }

// Sign- or zero-extended field of the low L bits (v_bfe with a uniform width).
template <bool SG>
__device__ __forceinline__ int32_t low_field(uint32_t w, int L) {
    int32_t d;
    if (SG)
        asm("v_bfe_i32 %0, %1, 0, %2" : "=v"(d) : "v"(w), "s"(L));
    else
        asm("v_bfe_u32 %0, %1, 0, %2" : "=v"(d) : "v"(w), "s"(L));
    return d;
}

// The output tile in LDS, by byte offset.
typedef int32_t __attribute__((address_space(3))) *TilePtr;
__device__ __forceinline__ void tile_add(uint32_t at, int j, int32_t v) {
    __hip_atomic_fetch_add((TilePtr)(size_t)(at + 4 * j), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Decode of one accumulator (Sec. 6).  Signed results: the accumulator started at the sign
// bits of lanes 0 .. nl-2 (MultiplyArgs::bias) instead of 0, so the carries that the
// fix-up of the signed-convolution figure adds back - a negative lane's borrow from the
// lane above - never arise, and its final xor with the same bits turns every lane's field
// into two's complement.  Lane j is the (sign-extended) field at bit j L, added into its
// output column (4 j bytes on); lane NL-1 takes all remaining bits.  Every lane is cut from
// the word directly (no chain of shifts), so the lanes' extractions are independent
// instructions.
// PS (permanent spacer bits, Sec. 6.1): every lane's MSB is a spacer bit (the planner
// keeps its values within L - 1 bits), so the xor, which only restores the MSB, is left
// out and each lane is read from its low L - 1 bits (fw).
template <bool SG, int NL, bool PS>
__device__ __forceinline__ void decode_word(uint64_t v, uint64_t msb_mask, int L, int fw, uint32_t at) {
    if (SG && !PS) v ^= msb_mask;
#pragma unroll
    for (int j = 0; j < NL - 1; ++j) tile_add(at, j, low_field<SG>((uint32_t)(v >> (j * L)), PS ? fw : L));
    const int top = (NL - 1) * L;
    tile_add(at, NL - 1, (int32_t)(SG ? (uint64_t)((int64_t)v >> top) : v >> top));
}

// The same for a lane count known only at run time.
template <bool SG, bool PS>
__device__ __forceinline__ void decode_word_n(uint64_t v, uint64_t msb_mask, int L, int fw, int nl, uint32_t at) {
    if (SG && !PS) v ^= msb_mask;
#pragma unroll 1
    for (int j = 0; j < nl - 1; ++j) tile_add(at, j, low_field<SG>((uint32_t)(v >> (j * L)), PS ? fw : L));
    const int top = (nl - 1) * L;
    tile_add(at, nl - 1, (int32_t)(SG ? (uint64_t)((int64_t)v >> top) : v >> top));
}

// Two-level lanes (Conv2dGeom::two).  A lane of L bits holds few channels when the
// products are wide for it (13-bit lanes of 4-bit operands: 7 channels, 21 products per
// accumulator and decode), and a decode into the output tile costs about as much as those
// products.  So the accumulators' lanes are not read into the tile every G channels but
// widened in registers: the accumulator starts at `bias` (half a lane's range in every
// lane below the top one), so every such lane is a non-negative field, and
//     odd  += (V >> L) & odd_mask        lanes 1, 3, ... as fields 2 L bits apart
//     all  += V                          (mod 2^64; all - (odd << L) is lanes 0, 2, ...)
// are two 64-bit sums whose fields have 2 L bits: room for 2^L such steps.  Six
// instructions per accumulator (a shift, two ands, two 64-bit adds, the restart), eight with
// the top lane apart, instead of about 22 and one LDS atomic per lane.
// The sums are decoded into the tile once, after the wave's last channel.
// TWO == 1: the top lane's sum over the whole slice fits the top bits of the word it ends
// in.  TWO == 2: it does not, and is summed in a register of its own.
template <int TWO>
struct WideLanes {
    uint64_t all = 0, odd = 0;
    int32_t top = 0;

    __device__ __forceinline__ void add(int64_t &acc, int L, int top_shift, uint64_t odd_mask, uint64_t bias) {
        odd += (uint64_t)(acc >> L) & odd_mask;
        all += (uint64_t)acc;
        if (TWO == 2) top += (int32_t)(acc >> top_shift);
        acc = (int64_t)bias;
    }

    // offset: `steps` times half a lane's range, taken off every biased lane; field: 2 L
    // low bits (all 32 when 2 L >= 32).  Both mod 2^32, as the outputs are
    template <int NL>
    __device__ __forceinline__ void decode(int L, uint32_t field, uint32_t offset, uint32_t at) const {
        const uint64_t even = all - (odd << L);
#pragma unroll
        for (int j = 0; j < NL - 1; ++j) {
            const uint64_t w = (j & 1) ? odd >> ((j - 1) * L) : even >> (j * L);
            tile_add(at, j, (int32_t)(((uint32_t)w & field) - offset));
        }
        tile_add(at, NL - 1, TWO == 2 ? top
                                      : (int32_t)((NL & 1) ? (int64_t)even >> ((NL - 1) * L)
                                                           : (int64_t)odd >> ((NL - 2) * L)));
    }

    __device__ __forceinline__ void decode_n(int L, int nl, uint32_t field, uint32_t offset, uint32_t at) const {
        const uint64_t even = all - (odd << L);
#pragma unroll 1
        for (int j = 0; j < nl - 1; ++j) {
            const uint64_t w = (j & 1) ? odd >> ((j - 1) * L) : even >> (j * L);
            tile_add(at, j, (int32_t)(((uint32_t)w & field) - offset));
        }
        tile_add(at, nl - 1, TWO == 2 ? top
                                      : (int32_t)((nl & 1) ? (int64_t)even >> ((nl - 1) * L)
                                                           : (int64_t)odd >> ((nl - 2) * L)));
    }
};
template <>
struct WideLanes<0> {};

// Work item: rows_blk output rows x all Wo columns x mblk output channels of one image,
// computed by one workgroup of wm x ks waves.  Wave (kq, mw) computes output channels
// mw*8 .. +7 of the block over its slice kq of the input channels; lane (grp, q) holds
// output word q of rows grp*RH .. +RH-1.  Operand words come straight from the spread
// buffer (global memory, L1/L2-resident: every word is reused by the block's wm waves and
// its KH kernel rows), kernel words from the wave's stream through scalar loads.  After at
// most G channels the accumulators are decoded into an LDS tile of int32 outputs whose
// atomic adds also sum the ks channel slices and overlap-add neighbouring words' partial
// lanes (TWO == 0), or widened in registers and decoded once (TWO != 0, see WideLanes).
//
// The grid holds at most as many workgroups as the chip keeps resident.  XCD x (hardware
// assigns workgroup p to XCD p % 8) owns one contiguous eighth of the spatial tiles, each
// with all its channel blocks in consecutive items, so a tile's operand words - and the
// halo rows it shares with the next row tile - are fetched into that XCD's L2 once and
// reused there.  Workgroup p first computes item p / 8 of its XCD; the items
// beyond the XCD's workgroups go to whichever workgroup frees up first, through a ticket
// counter per XCD: waves of equal work finish far apart (the SIMD issues the oldest wave
// first), and a fixed assignment would leave the chip draining for much of the launch.
// A launch takes exactly T = extra items + workgroups tickets from each counter (every
// workgroup ends on one ticket past the items), so ticket t stands for local index
// t mod T: the counters never need resetting between launches.  Each workgroup asks for
// its next ticket when it starts an item, so the atomic's latency hides behind the item.
//
// KHT: 3 or 5, the kernel rows of a stride-1 layer whose output rows share operand loads
// (rows_path): output row r with kernel row ky reads input row r + ky, so the lane's RH
// rows need RH + KHT - 1 operand words per (channel, kernel word) instead of KHT RH.  Every
// operand load costs the compute unit's texture path far more cycles than a multiply-add
// costs a SIMD, and the four SIMDs share that path.  0: any other layer, one operand word
// per (row, step); 1: such a layer whose channels have a multiple of three steps (3-row
// kernels at any stride), whose operand offsets take half of the scalar instructions.  SG: the result is signed (either operand signed), so lanes need the
// fix-up and are sign-extended.  SEG: rows are split into column segments.
//
// The multiply loop: batches of kernel words in SGPRs (scalar loads, one pointer that only
// moves forward) and operand words in VGPRs, ping-pong over two register sets A and B.
// Before a batch's kernel words are used, all outstanding scalar loads are waited for, and
// only then is the next batch requested: scalar loads return out of order, so a wait
// placed after requesting the next batch would wait for it too.  Operand loads are vector
// loads, which complete in order, so the compiler waits for exactly the batch in use.  A
// period (the batches a lane holds before it must be read) is one inner loop of pairs of
// batches with no test inside but its own: a SIMD issues its oldest wave first, so a wave's
// own scalar work and taken branches are not hidden behind the other waves.  With the test
// for the next decode in every batch and offsets recomputed per batch the loop took about
// 6.3 clocks per multiply-add and SIMD at the 8 x 128 x 56 x 56 layer at 2 bits, without
// them about 4.6.  The batch after the last one is fetched as well (its results are never
// used): it reads the next channel, which exists (the spread buffer has one spare channel
// after the last image), and the kStreamPad padding steps of the kernel-word stream.
template <int RH, int KHT, int TWO, bool SG, bool SEG>
__global__ __launch_bounds__(TWO ? kMaxWideThreads : 1024) void conv2d_samd_kernel(const MultiplyArgs by_value) {
    extern __shared__ int32_t tile[];   // the output tile, then the next item
    (void)by_value;
    const ArgsPtr args = (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
    const uint32_t tile_at = (uint32_t)(size_t)(TilePtr)tile;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int xcd = blockIdx.x % kNumXcd;
    bool fresh = true;                     // the tile has not been zeroed yet (first item)
    for (int item = blockIdx.x / kNumXcd;;) {
        const ArgsPtr a = args_again(args);
        // XCD x owns the tiles [t0, t1): a contiguous range, so neighbouring row tiles (which
        // share their halo input rows) meet in one L2
        const int t0 = (int)((int64_t)xcd * a->tiles / kNumXcd), t1 = (int)((int64_t)(xcd + 1) * a->tiles / kNumXcd);
        const int nitems = (t1 - t0) * a->nmb;       // items of this XCD
        if (item >= nitems) return;
        const int nwg = a->nwg;                      // workgroups of this XCD
        const int nextra = max(0, nitems - nwg);     // items handed out by ticket
        unsigned long long ticket = 0;
        if (nextra > 0 && tid == 0) ticket = atomicAdd(a->tickets + xcd * (kTicketStride / 8), 1ull);

        const int kq = (wave * a->wm_mul) >> 16, mw = wave - kq * a->wm;
        const int grp_raw = (lane * a->nqs_mul) >> 16;
        const bool lane_ok = grp_raw < a->groups;
        const int grp = lane_ok ? grp_raw : 0;
        const int q = lane_ok ? lane - grp_raw * a->nqs : 0;   // word within the column segment

        const int tile_of = divide(item, a->by_nmb.mul, a->by_nmb.shift);
        const int mb = item - tile_of * a->nmb;
        const int tile_id = t0 + tile_of;   // (n, row tile, column segment)
        // SEG: rows are split into column segments; without, the segment terms fold away
        const int rt_id = SEG ? divide(tile_id, a->by_ncs.mul, a->by_ncs.shift) : tile_id;
        const int cs = SEG ? tile_id - rt_id * a->ncs : 0;
        const int n = divide(rt_id, a->by_row_tiles.mul, a->by_row_tiles.shift);
        const int ho0 = (rt_id - n * a->row_tiles) * a->rows_blk;
        // the lane's word in the row; words past the row (last segment) read its last
        // word and only reach columns that are never stored
        const int nq = a->nq, ntw = a->ntw;
        const int qg = SEG ? min(cs * a->qseg + q, nq - 1) : q;

        // Operand word of step s (s = ky*ntw + t) of channel c for this lane's row r:
        // xs[n][c][hp][t][q] with hp = (ho0 + row)*sh + ky, i.e. word
        // (c*Hp*ntw + (ho0 + row)*sh*ntw + s)*nq + q of image n.  Rows past the image (the last
        // row tile, idle lanes) read the last row's inputs; their sums are not stored.
        const int ch_stride = a->Hp * ntw * nq;
        // the image's channels and one spare channel after them
        const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc(
            (void *)(a->xs + (int64_t)n * a->C * ch_stride), (short)0, (a->C + 1) * ch_stride * 4, kBufferWord3);

        // This wave's channel slice: channels cbeg .. cend-1, at least one (no plan has an empty
        // slice): the first batch is requested unconditionally.  Requested under a condition, its
        // kernel words were carried from item to item, 32 to 100 scalar registers parked in vector
        // lanes and read back: a third of the vector instructions of a layer of few channels.
        const int cbeg = min(kq * a->cpw, a->C), cend = min(cbeg + a->cpw, a->C);
        const KernelWords stream =
            (KernelWords)(a->kw + (mb * a->wm + mw) * a->stream_len + (int64_t)cbeg * a->nrt * RM);
        KernelWords kp = stream;              // the next batch's kernel words
        int sb = cbeg * ch_stride * 4;        // the next batch's operand offset
        const int period = a->period;

        int64_t acc[RH][RM];
        WideLanes<TWO> wide[RH][RM];
        int steps = 0;   // TWO: periods widened so far
        const int64_t start = SG ? (int64_t)a->bias : 0;
#pragma unroll
        for (int r = 0; r < RH; ++r)
#pragma unroll
            for (int m = 0; m < RM; ++m) acc[r][m] = start;

        // Decode: lane j of word q goes to output column q*I + j - (Kmax-1), stored at tile
        // column q*I + j.  Tile rows cover every row a wave computes, so no lane needs a
        // bounds check.  The tile address of each (row, channel) accumulator is one add away
        // from the previous one; the running address is opaque to the compiler, which would
        // otherwise keep all RH*8 addresses (times every lane-count case) live across the
        // main loop and cut the waves a SIMD can hold.
#define SAMD_DECODE_LOOP(CALL)                                                                        \
    _Pragma("unroll") for (int m = 0; m < RM; ++m) {                                                 \
        asm volatile("" : "+v"(ti));                                                                  \
        uint32_t at = ti;                                                                             \
        _Pragma("unroll") for (int r = 0; r < RH; ++r) {                                             \
            CALL;                                                                                     \
            at += row_bytes;                                                                          \
        }                                                                                             \
        ti += m_bytes;                                                                                \
    }
#define SAMD_DECODE_ADDRESSES                                                                         \
    const uint32_t row_bytes = 4 * d->tile_row, m_bytes = d->tile_rows * row_bytes;                   \
    uint32_t ti = tile_at + mw * RM * m_bytes + grp * RH * row_bytes + 4 * q * d->I;
        auto flush = [&]() __attribute__((always_inline)) {
            if constexpr (TWO != 0) {
                const ArgsPtr d = a;
                const int L = d->L, top = (d->nl - 1) * L;
                const uint64_t odd_mask = d->odd_mask;
#pragma unroll
                for (int r = 0; r < RH; ++r)
#pragma unroll
                    for (int m = 0; m < RM; ++m) wide[r][m].add(acc[r][m], L, top, odd_mask, (uint64_t)start);
                ++steps;
            } else {
                if (lane_ok) {
                    const ArgsPtr d = args_again(args);
                    SAMD_DECODE_ADDRESSES
                    const uint64_t msb = d->msb_mask;
                    const int L = d->L, fw = L - 1;
#define SAMD_DECODE_NL(NL_, PS_)                                                                      \
    case NL_:                                                                                         \
        SAMD_DECODE_LOOP((decode_word<SG, NL_, PS_>((uint64_t)acc[r][m], msb, L, fw, at)))            \
        break;
#define SAMD_DECODE_ALL(PS_)                                                                          \
    switch (d->nl) {                                                                                  \
        SAMD_DECODE_NL(2, PS_) SAMD_DECODE_NL(3, PS_) SAMD_DECODE_NL(4, PS_) SAMD_DECODE_NL(5, PS_)   \
        SAMD_DECODE_NL(6, PS_) SAMD_DECODE_NL(7, PS_) SAMD_DECODE_NL(8, PS_)                          \
    default:                                                                                          \
        SAMD_DECODE_LOOP((decode_word_n<SG, PS_>((uint64_t)acc[r][m], msb, L, fw, d->nl, at)))        \
    }
                    if constexpr (SG) {
                        if (d->spacer) {
                            SAMD_DECODE_ALL(true)
                        } else {
                            SAMD_DECODE_ALL(false)
                        }
                    } else {
                        SAMD_DECODE_ALL(false)
                    }
#undef SAMD_DECODE_ALL
#undef SAMD_DECODE_NL
                }
#pragma unroll
                for (int r = 0; r < RH; ++r)
#pragma unroll
                    for (int m = 0; m < RM; ++m) acc[r][m] = start;
            }
        };
        // the widened sums into the tile, after the wave's last channel
        auto finish = [&]() __attribute__((always_inline)) {
            if constexpr (TWO != 0) {
                if (lane_ok) {
                    const ArgsPtr d = args_again(args);
                    SAMD_DECODE_ADDRESSES
                    const int L = d->L;
                    const uint32_t field = 2 * L >= 32 ? 0xffffffffu : (1u << (2 * L)) - 1;
                    const uint32_t offset = SG ? (uint32_t)steps << (L - 1) : 0;
#define SAMD_WIDE_NL(NL_)                                                                             \
    case NL_:                                                                                         \
        SAMD_DECODE_LOOP((wide[r][m].template decode<NL_>(L, field, offset, at)))                     \
        break;
                    switch (d->nl) {
                        SAMD_WIDE_NL(3) SAMD_WIDE_NL(4) SAMD_WIDE_NL(5) SAMD_WIDE_NL(6) SAMD_WIDE_NL(7)
                    default:
                        SAMD_DECODE_LOOP((wide[r][m].decode_n(L, d->nl, field, offset, at)))
                    }
#undef SAMD_WIDE_NL
                }
            }
        };
#undef SAMD_DECODE_LOOP
#undef SAMD_DECODE_ADDRESSES
        // the tile's first zeroing, between requesting an item's first batch and using it
        auto open_tile = [&]() __attribute__((always_inline)) {
            if (fresh) {
                int4 *t4 = (int4 *)tile;   // lds_tile is a multiple of 4 words
                const int nthr = a->waves * 64;
                for (int i = tid; i < a->lds_tile / 4; i += nthr) t4[i] = int4{0, 0, 0, 0};
                __syncthreads();
                fresh = false;
            }
        };

        if constexpr (KHT == 3) {
            // batch: one kernel word of one channel, its three kernel rows (the stream is
            // kernel-word-major within a channel) and the operand words of input rows
            // hp0 + i, i < RH + 2 (rows past the padded image are clamped to its last row:
            // they only reach output rows that are never stored)
            constexpr int NA = RH + 2;
            int lbi[NA];
#pragma unroll
            for (int i = 0; i < NA; ++i)
                lbi[i] = (min(ho0 + grp * RH + i, a->Hp - 1) * ntw * nq + qg) * 4;
            // operand offsets of successive batches: to the channel's second kernel word and
            // on to the next channel (ntw == 2), or from channel to channel (ntw == 1)
            const int da = (ntw == 2 ? nq : ch_stride) * 4;
            const int db = (ntw == 2 ? ch_stride - nq : ch_stride) * 4;
            int32_t kA[3 * RM], aA[NA], kB[3 * RM], aB[NA];
            auto load = [&](int32_t(&k)[3 * RM], int32_t(&a)[NA], int step) __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < 3 * RM; ++j) k[j] = kp[j];
#pragma unroll
                for (int i = 0; i < NA; ++i) a[i] = buffer_word(xrs, lbi[i], sb);
                kp += 3 * RM;
                sb += step;
            };
            auto mac = [&](const int32_t(&k)[3 * RM], const int32_t(&a)[NA]) __attribute__((always_inline)) {
#pragma unroll
                for (int ky = 0; ky < 3; ++ky) {
#pragma unroll
                    for (int r = 0; r < RH; ++r)
#pragma unroll
                        for (int m = 0; m < RM; ++m) acc[r][m] += (int64_t)a[r + ky] * (int64_t)k[ky * RM + m];
#pragma unroll
                    for (int r = 0; r < RH; ++r)
#pragma unroll
                        for (int m = 0; m < RM; ++m) keep(acc[r][m]);
                }
            };
            int left = (cend - cbeg) * ntw;
            load(kA, aA, da);
            open_tile();
            do {
                int nb = min(left, period);
                left -= nb;
                for (; nb >= 2; nb -= 2) {
                    wait_scalar();
                    load(kB, aB, db);
                    __builtin_amdgcn_sched_barrier(0);
                    mac(kA, aA);
                    __builtin_amdgcn_sched_barrier(0);
                    wait_scalar();
                    load(kA, aA, da);
                    __builtin_amdgcn_sched_barrier(0);
                    mac(kB, aB);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (nb) {   // the slice's last batch, or periods of one
                    wait_scalar();
                    mac(kA, aA);
                    if (left > 0) load(kA, aA, da);
                }
                flush();
            } while (left > 0);
        } else if constexpr (KHT == 5) {
            // a kernel word of a channel in two batches: kernel rows 0-2 with input rows
            // 0 .. RH + 1, then kernel rows 3 and 4 with two further input rows (rows
            // 3 .. RH + 1 of the first batch are used again)
            constexpr int NA = RH + 2;
            int lbi[RH + 4];
#pragma unroll
            for (int i = 0; i < RH + 4; ++i)
                lbi[i] = (min(ho0 + grp * RH + i, a->Hp - 1) * ntw * nq + qg) * 4;
            int32_t kA[3 * RM], aA[NA], kB[2 * RM], aB[RH + 1];
            int t = 0;
            auto load_a = [&]() __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < 3 * RM; ++j) kA[j] = kp[j];
#pragma unroll
                for (int i = 0; i < NA; ++i) aA[i] = buffer_word(xrs, lbi[i], sb);
                kp += 3 * RM;
            };
            auto load_b = [&]() __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < 2 * RM; ++j) kB[j] = kp[j];
                aB[RH - 1] = buffer_word(xrs, lbi[RH + 2], sb);
                aB[RH] = buffer_word(xrs, lbi[RH + 3], sb);
                kp += 2 * RM;
                sb += nq * 4;
                if (++t == ntw) {
                    t = 0;
                    sb += (ch_stride - ntw * nq) * 4;
                }
            };
            int left = (cend - cbeg) * ntw;
            load_a();
            open_tile();
            do {
                const int nb = min(left, period);
                for (int b = 0; b < nb; ++b) {
                    wait_scalar();
                    load_b();
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int ky = 0; ky < 3; ++ky) {
#pragma unroll
                        for (int r = 0; r < RH; ++r)
#pragma unroll
                            for (int m = 0; m < RM; ++m) acc[r][m] += (int64_t)aA[r + ky] * (int64_t)kA[ky * RM + m];
#pragma unroll
                        for (int r = 0; r < RH; ++r)
#pragma unroll
                            for (int m = 0; m < RM; ++m) keep(acc[r][m]);
                    }
#pragma unroll
                    for (int i = 0; i + 1 < RH; ++i) aB[i] = aA[3 + i];
                    __builtin_amdgcn_sched_barrier(0);
                    wait_scalar();
                    load_a();
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int ky = 0; ky < 2; ++ky) {
#pragma unroll
                        for (int r = 0; r < RH; ++r)
#pragma unroll
                            for (int m = 0; m < RM; ++m) acc[r][m] += (int64_t)aB[r + ky] * (int64_t)kB[ky * RM + m];
#pragma unroll
                        for (int r = 0; r < RH; ++r)
#pragma unroll
                            for (int m = 0; m < RM; ++m) keep(acc[r][m]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                left -= nb;
                flush();
            } while (left > 0);
        } else {
            // any other layer: batches of three consecutive steps of the slice, one operand
            // word per row and step; they may straddle channels unless a channel's steps
            // are whole batches (KHT == 1)
            int lb[RH];   // byte offset of the lane's word in channel 0, step 0
#pragma unroll
            for (int r = 0; r < RH; ++r) {
                const int row = min(ho0 + min(grp * RH + r, a->rows_blk - 1), a->Ho - 1);
                lb[r] = (row * a->sh * ntw * nq + qg) * 4;
            }
            int32_t kA[3 * RM], aA[3][RH], kB[3 * RM], aB[3][RH];
            // operand offsets step by step: nq words to the next step of a channel, then on
            // to the next channel; the steps requested past the slice stop at the spare
            // channel (fewer than three steps per channel could pass it)
            int rt = 0;
            const int nrt = a->nrt;
            const int sb_max = (a->C * ch_stride + (nrt - 1) * nq) * 4;
            const int ch_skip = (ch_stride - nrt * nq) * 4;
            auto load = [&](int32_t(&k)[3 * RM], int32_t(&a)[3][RH]) __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < 3 * RM; ++j) k[j] = kp[j];
                if constexpr (KHT == 1) {
#pragma unroll
                    for (int j = 0; j < 3; ++j)
#pragma unroll
                        for (int r = 0; r < RH; ++r) a[j][r] = buffer_word(xrs, lb[r], sb + j * nq * 4);
                    sb += 3 * nq * 4;
                    rt += 3;
                    if (rt == nrt) {
                        rt = 0;
                        sb += ch_skip;
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < 3; ++j) {
#pragma unroll
                        for (int r = 0; r < RH; ++r) a[j][r] = buffer_word(xrs, lb[r], sb);
                        sb += nq * 4;
                        if (++rt == nrt) {
                            rt = 0;
                            sb += ch_skip;
                        }
                        sb = min(sb, sb_max);
                    }
                }
                kp += 3 * RM;
            };
            auto mac = [&](const int32_t(&k)[3 * RM], const int32_t(&a)[3][RH]) __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < 3; ++j) {
#pragma unroll
                    for (int r = 0; r < RH; ++r)
#pragma unroll
                        for (int m = 0; m < RM; ++m) acc[r][m] += (int64_t)a[j][r] * (int64_t)k[j * RM + m];
#pragma unroll
                    for (int r = 0; r < RH; ++r)
#pragma unroll
                        for (int m = 0; m < RM; ++m) keep(acc[r][m]);
                }
            };
            // a batch of which only the first `live` steps count
            auto mac_part = [&](const int32_t(&k)[3 * RM], const int32_t(&a)[3][RH], int live) __attribute__((always_inline)) {
                int32_t m[3][RH];
#pragma unroll
                for (int j = 0; j < 3; ++j)
#pragma unroll
                    for (int r = 0; r < RH; ++r) m[j][r] = j < live ? a[j][r] : 0;
                mac(k, m);
            };
            const int total = (cend - cbeg) * nrt;   // steps of the slice
            if (period > 0) {
                int left = total / 3;                  // whole batches
                const int rest = total - left * 3;
                load(kA, aA);
                open_tile();
                do {
                    int nb = min(left, period);
                    left -= nb;
                    // the last, partial batch joins the last period if that has room
                    bool part = left == 0 && rest != 0 && nb < period;
                    for (; nb >= 2; nb -= 2) {
                        wait_scalar();
                        load(kB, aB);
                        __builtin_amdgcn_sched_barrier(0);
                        mac(kA, aA);
                        __builtin_amdgcn_sched_barrier(0);
                        wait_scalar();
                        load(kA, aA);
                        __builtin_amdgcn_sched_barrier(0);
                        mac(kB, aB);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (nb) {   // the slice's last whole batch, or periods of one
                        wait_scalar();
                        mac(kA, aA);
                        if (left > 0 || rest != 0) load(kA, aA);
                    }
                    if (part) {
                        wait_scalar();
                        mac_part(kA, aA, rest);
                        left = -1;
                    }
                    flush();
                } while (left > 0 || (left == 0 && rest != 0));
            } else {
                // the lanes hold fewer steps than a batch (-period of them): one partial
                // batch at a time
                open_tile();
                const int spb = -period;
                int s = 0;
                do {
                    const int c = s / nrt;
                    rt = s - c * nrt;
                    sb = ((cbeg + c) * ch_stride + rt * nq) * 4;
                    kp = stream + (int64_t)s * RM;
                    load(kA, aA);
                    wait_scalar();
                    mac_part(kA, aA, min(spb, total - s));
                    flush();
                    s += spb;
                } while (s < total);
            }
        }
        finish();

        const ArgsPtr o = args_again(args);
        if (tid == 0) {
            int next = nitems;
            if (nextra > 0) {
                // ticket mod T by the rounded-down reciprocal of T, short by at most one T
                const uint64_t recip = (int)((int64_t)o->tiles - (int64_t)(t1 - t0) * kNumXcd) > 0 ? o->recip_lo : o->recip_hi;
                const unsigned long long T = nextra + nwg;
                unsigned long long r = ticket - __umul64hi(ticket, recip) * T;
                if (r >= T) r -= T;
                next = nwg + (int)r;
            }
            tile[o->lds_tile] = next;
        }
        __syncthreads();
        const int following = __builtin_amdgcn_readfirstlane(tile[o->lds_tile]);
        const bool again = following < nitems;

        // output tile -> y.  Every tile word of a segment column is zeroed for the next item, if
        // there is one, once read, also in rows past the image, channels past M and columns past
        // Wo, which another item stores.
        // Recentred activations (xoff): + xoff * (the sum of the weights over the output's
        // in-image taps).  Where the padding was written as recentred zeros (pad_filled),
        // every output takes every tap and the sum is one number per channel; in the
        // permanent-spacer layout, whose padding is 0, it is a rectangle of the prefix table.
        const int c0 = SEG ? cs * o->cw : 0, ncols = SEG ? min(o->cw, o->Wo - c0) : o->Wo;   // the segment's columns
        const int segw = SEG ? o->cw : o->Wo;
        const int rows_blk = o->rows_blk, nwaves = o->waves, M = o->M, Ho = o->Ho, mblk = o->mblk, xoff = o->xoff;
        constexpr int U = 4;
        if (segw <= 64) {
            // Rows of at most 64 outputs: each lane works out its own row, and a wave copies 2, 4 or 8
            // rows of at most 32, 16 or 8 outputs at once, four such steps at a time so that their
            // reads are in flight together.  A row of a wave of its own costs about 58 instructions whatever its
            // length, which is most of the time of layers with few input channels: 13 x 5 x 219 x
            // 32 -> 244, 3x3, 8 bits 113 -> 60 us, 10 x 3 x 182 x 23 -> 157 52 -> 23 us; one row of
            // 33 to 64 at a time is still shorter in vector than in scalar instructions: 2 x 16 x 34 x
            // 34 -> 490, 1x1, 18.3 -> 16.1 us, 12 x 46 x 26 x 54 -> 214, 3x3, 33.0 -> 30.3.
            const int lane_rows = SEG || o->Wo > 32 ? 1 : o->Wo > 16 ? 2 : o->Wo > 8 ? 4 : 8;
            const int width = 64 / lane_rows, col = lane & (width - 1);
            const int step = nwaves * lane_rows, smm = (step * o->rows_mul) >> 16, sr = step - smm * rows_blk;
            const int row = wave * lane_rows + lane / width;
            int mm = (row * o->rows_mul) >> 16, r = row - mm * rows_blk;
            int32_t *const yn = o->y + (int64_t)n * M * Ho * o->Wo;
            while (mm < mblk && col < segw) {
                int32_t v[U];
                int src[U], ms[U], hos[U];
                bool in[U], ok[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    in[u] = mm < mblk;
                    ms[u] = mb * mblk + mm;
                    hos[u] = ho0 + r;
                    ok[u] = in[u] && ms[u] < M && hos[u] < Ho && (!SEG || col < ncols);
                    src[u] = (in[u] ? (mm * o->tile_rows + r) * o->tile_row : 0) + (o->Kmax - 1) + col;
                    v[u] = tile[src[u]];
                    mm += smm;
                    r += sr;
                    if (r >= rows_blk) {
                        r -= rows_blk;
                        ++mm;
                    }
                }
                if (xoff != 0 && o->pad_filled) {
#pragma unroll
                    for (int u = 0; u < U; ++u) v[u] += o->pre[ok[u] ? ms[u] : 0];
                } else if (xoff != 0) {
                    const int kwid = o->KW + 1, wbeg = (c0 + col) * o->sw - o->pw;
                    const int kx0 = max(0, -wbeg), kx1 = max(min(o->KW, o->W - wbeg), 0);
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int hb = (ok[u] ? hos[u] : 0) * o->sh - o->ph;
                        const int ky0 = max(0, -hb) * kwid, ky1 = min(o->KH, o->H - hb) * kwid;
                        const int32_t *pm = o->pre + (int64_t)(ok[u] ? ms[u] : 0) * (o->KH + 1) * kwid;
                        v[u] += xoff * (pm[ky1 + kx1] - pm[ky0 + kx1] - pm[ky1 + kx0] + pm[ky0 + kx0]);
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (ok[u]) yn[((int64_t)ms[u] * Ho + hos[u]) * o->Wo + c0 + col] = v[u];
                    if (again && in[u]) tile[src[u]] = 0;
                }
            }
        } else {
            // Longer rows: wave w copies rows rr = w, w + nwaves, ... (rr = mm * rows_blk + r), 128
            // columns at a time.  Where the next row lies is one addition away, and the columns of
            // a row's last step are found once for all rows: layers with few input channels
            // are bound by these instructions, not by their stores.  8 x 1 x 163 x 117 -> 453, 1x1
            // (276 MB): 88 us against 116 with four rows at a time, each addressed and tested for
            // itself, and 133 with each row in steps of 4 x 64 tested columns; 75 since an item
            // carries no kernel words over.
            const int dmm = (nwaves * o->rows_mul) >> 16, dr = nwaves - dmm * rows_blk;
            int mm = (wave * o->rows_mul) >> 16, r = wave - mm * rows_blk;
            const uint32_t row_bytes = 4 * o->tile_row, blk_bytes = o->tile_rows * row_bytes;
            const uint32_t src_step = dmm * blk_bytes + dr * row_bytes, src_wrap = blk_bytes - rows_blk * row_bytes;
            const int64_t dst_step = ((int64_t)dmm * Ho + dr) * o->Wo, dst_wrap = (int64_t)(Ho - rows_blk) * o->Wo;
            uint32_t src = tile_at + mm * blk_bytes + r * row_bytes + 4 * (o->Kmax - 1 + lane);
            int32_t *dst = o->y + (((int64_t)n * M + mb * mblk + mm) * Ho + ho0 + r) * o->Wo + c0;
            const int steps128 = (ncols - 1) >> 7, last = ncols - 128 * steps128 - lane;
            const bool last0 = last > 0, last1 = last > 64;
            while (mm < mblk) {
                const int m = mb * mblk + mm, ho = ho0 + r;
                if (m < M && ho < Ho) {
                    uint32_t at = src;
                    if (xoff != 0 && !o->pad_filled) {
                        const int kwid = o->KW + 1, hb = ho * o->sh - o->ph;
                        const int ky0 = max(0, -hb) * kwid, ky1 = min(o->KH, o->H - hb) * kwid;
                        const int32_t *pm = o->pre + (int64_t)m * (o->KH + 1) * kwid;
                        for (int col = lane; col < ncols; col += 64, at += 256) {
                            const int wbeg = (c0 + col) * o->sw - o->pw;
                            const int kx0 = max(0, -wbeg), kx1 = min(o->KW, o->W - wbeg);
                            dst[col] = *(TilePtr)(size_t)at +
                                       xoff * (pm[ky1 + kx1] - pm[ky0 + kx1] - pm[ky1 + kx0] + pm[ky0 + kx0]);
                            if (again) *(TilePtr)(size_t)at = 0;
                        }
                    } else {
                        const int32_t add = xoff != 0 ? ((KernelWords)o->pre)[m] : 0;
                        uint32_t to = 4 * lane;
                        auto put = [&](uint32_t bytes, int32_t v) __attribute__((always_inline)) {
                            *(int32_t *)((char *)dst + bytes) = v + add;
                        };
                        for (int step = 0; step < steps128; ++step) {
                            const int32_t v0 = ((TilePtr)(size_t)at)[0], v1 = ((TilePtr)(size_t)at)[64];
                            put(to, v0);
                            put(to + 256, v1);
                            if (again) ((TilePtr)(size_t)at)[0] = ((TilePtr)(size_t)at)[64] = 0;
                            at += 512;
                            to += 512;
                        }
                        int32_t v0 = 0, v1 = 0;
                        if (last0) v0 = ((TilePtr)(size_t)at)[0];
                        if (last1) v1 = ((TilePtr)(size_t)at)[64];
                        if (last0) {
                            put(to, v0);
                            if (again) ((TilePtr)(size_t)at)[0] = 0;
                        }
                        if (last1) {
                            put(to + 256, v1);
                            if (again) ((TilePtr)(size_t)at)[64] = 0;
                        }
                    }
                    // the columns past Wo of the last segment
                    if (SEG && again)
                        for (int col = ncols + lane; col < segw; col += 64) ((TilePtr)(size_t)src)[col - lane] = 0;
                } else if (again) {
                    for (int col = lane; col < segw; col += 64) ((TilePtr)(size_t)src)[col - lane] = 0;
                }
                mm += dmm;
                r += dr;
                src += src_step;
                dst += dst_step;
                if (r >= rows_blk) {
                    r -= rows_blk;
                    ++mm;
                    src += src_wrap;
                    dst += dst_wrap;
                }
            }
        }
        if (!again) return;
        item = following;
        // the write-out (and the tile's re-zeroing) ends before the next item's decodes
        __syncthreads();
    }
}

// x / d = (x * mul) >> 16 for the small numbers it is used on: exact while x d < 65536 (lanes
// by words of a row, and the tile rows a workgroup copies at once - up to 8 a wave - by the
// rows of a tile, at most 4 of each of a wave's lane groups)
inline int32_t small_reciprocal(int d) { return 65536 / d + 1; }
static_assert(64 * 64 < 65536 && kMaxBlockWaves * 8 * (64 * 4) < 65536, "small_reciprocal");

template <int RH, int KHT, int TWO, bool SG, bool SEG>
int launch_multiply_instance(const Conv2dGeom &g, int32_t *y, const void *ws, hipStream_t s, const int32_t *src) {
    MultiplyArgs a = {};
    a.xs = src ? src : (const int32_t *)((const char *)ws + conv2d_xs_offset(g));
    a.kw = (const int32_t *)ws;
    a.tickets = (unsigned long long *)((char *)const_cast<void *>(ws) + conv2d_queue_offset(g));
    a.tiles = g.tiles; a.nmb = g.nmb; a.ncs = g.ncs; a.row_tiles = g.row_tiles;
    a.by_nmb = division(g.nmb); a.by_ncs = division(g.ncs); a.by_row_tiles = division(g.row_tiles);
    a.wm = g.wm; a.waves = g.wm * g.ks; a.wm_mul = small_reciprocal(g.wm); a.nqs_mul = small_reciprocal(g.nqs);
    a.nqs = g.nqs; a.groups = g.groups; a.rows_blk = g.rows_blk; a.C = g.C;
    a.nq = g.nq; a.ntw = g.ntw; a.nrt = g.nrt; a.Hp = g.Hp;
    a.Ho = g.Ho; a.sh = g.sh; a.qseg = g.qseg; a.cpw = g.cpw; a.period = g.period; a.lds_tile = g.lds_tile;
    a.stream_len = ((int64_t)g.C * g.nrt + kStreamPad) * RM;
    a.bias = g.bias; a.odd_mask = g.odd_mask;
    a.msb_mask = g.msb_mask;
    a.L = g.L; a.nl = g.nl; a.spacer = g.spacer; a.I = g.I; a.tile_rows = g.tile_rows; a.tile_row = g.tile_row;
    a.y = y;
    a.pre = (const int32_t *)((const char *)ws + conv2d_kw_bytes(g));
    a.rows_mul = small_reciprocal(g.rows_blk);
    a.mblk = g.mblk; a.M = g.M; a.Wo = g.Wo; a.cw = g.cw; a.Kmax = g.Kmax; a.xoff = g.xoff;
    a.pad_filled = conv2d_pad_value(g.xoff, g.layout_spaced) != 0;
    a.KH = g.KH; a.KW = g.KW; a.H = g.H; a.W = g.W; a.ph = g.ph; a.pw = g.pw; a.sw = g.sw;
    const int block = g.wm * g.ks * 64;
    const size_t shm = (size_t)(g.lds_words + 4) * 4;   // the tile and the next item
    const void *fn = (const void *)conv2d_samd_kernel<RH, KHT, TWO, SG, SEG>;
    int resident = 0;
    const int st = resident_workgroups(fn, block, shm, resident);
    if (st) return st;
    // every XCD gets the same number of workgroups; none gets more than its items
    const int64_t xitems = (int64_t)(g.tiles + kNumXcd - 1) / kNumXcd * g.nmb;
    const int64_t per_xcd = std::max<int64_t>(1, std::min<int64_t>(xitems, resident / kNumXcd));
    // tickets per launch and XCD: an XCD owns floor(tiles / 8) tiles or one more
    auto recip = [&](int64_t tiles) {
        const uint64_t T = (uint64_t)std::max<int64_t>(0, tiles * g.nmb - per_xcd) + per_xcd;
        return T < 2 ? ~(uint64_t)0 : (uint64_t)(((unsigned __int128)1 << 64) / T);
    };
    a.nwg = (int32_t)per_xcd;
    a.recip_lo = recip(g.tiles / kNumXcd);
    a.recip_hi = recip((g.tiles + kNumXcd - 1) / kNumXcd);
    hipLaunchKernelGGL((conv2d_samd_kernel<RH, KHT, TWO, SG, SEG>), dim3((unsigned)(per_xcd * kNumXcd)), dim3(block),
                       shm, s, a);
    return check_launch("conv2d");
}

// Picks signedness and segmentation; TWO as planned.
template <int RH, int KHT, int TWO>
int launch_multiply_shape(const Conv2dGeom &g, int32_t *y, const void *ws, hipStream_t s, const int32_t *src) {
    if (g.result_signed)
        return g.ncs > 1 ? launch_multiply_instance<RH, KHT, TWO, true, true>(g, y, ws, s, src)
                         : launch_multiply_instance<RH, KHT, TWO, true, false>(g, y, ws, s, src);
    return g.ncs > 1 ? launch_multiply_instance<RH, KHT, TWO, false, true>(g, y, ws, s, src)
                     : launch_multiply_instance<RH, KHT, TWO, false, false>(g, y, ws, s, src);
}

}  // namespace

}  // namespace samd
