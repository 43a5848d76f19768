// Host-side lane-geometry planning for the SAMD convolutions.  Pure C++: no HIP calls,
// so it runs (and is tested) without a GPU.
//
// The paper sizes lanes so that no lane can overflow into its neighbour (Sec. 5.1:
// a K-term sum of b x b-bit products needs 2b + log2 K bits) and keeps one bit of
// margin in signed lanes for the borrow a negative lane hands to the lane above it
// (Sec. 6).  Here the bound is computed exactly, per lane, for the products actually
// accumulated into it before the lanes are decoded, and the planner picks among the
// exact geometries the one with the lowest modelled cost.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdio>
#include <array>
#include <cstdint>
#include <limits>
#include <functional>
#include <map>
#include <mutex>
#include <vector>

#include "samd_internal.hpp"

namespace samd {

namespace {

typedef __int128 i128;

i128 pow2(int e) { return (i128)1 << e; }

// Range of a b-bit value.
void value_range(int bits, bool is_signed, i128 &lo, i128 &hi) {
    lo = is_signed ? -pow2(bits - 1) : 0;
    hi = is_signed ? pow2(bits - 1) - 1 : pow2(bits) - 1;
}

i128 max_abs(int bits, bool is_signed) { return is_signed ? pow2(bits - 1) : pow2(bits) - 1; }

// Does sum_{i<n} v_i 2^(i L) stay inside [lo_lim, hi_lim] for every b-bit v_i?
bool word_fits(int bits, bool is_signed, int L, int n, i128 lo_lim, i128 hi_lim) {
    if ((n - 1) * L + bits > 64) return false;
    i128 lo, hi, place = 0;
    value_range(bits, is_signed, lo, hi);
    for (int i = 0; i < n; ++i) place += pow2(i * L);
    return lo * place >= lo_lim && hi * place <= hi_lim;
}

const i128 kI32Min = -pow2(31), kI32Max = pow2(31) - 1;
const i128 kI64Max = pow2(63) - 1;

// Products of an I-value word and a k-tap word that land in lane j.
int pairs_in_lane(int j, int I, int k) {
    if (j < 0 || j > I + k - 2) return 0;
    return std::min(std::min(j + 1, k), std::min(I, I + k - 1 - j));
}

// Split `count` consecutive taps into ceil(count / kmax) near-equal groups; false (and
// nothing written) when that is more than kMaxTapWords groups.
bool split_taps(int count, int kmax, int *t0, int *nt, int &ngroups) {
    ngroups = (count + kmax - 1) / kmax;
    if (ngroups > kMaxTapWords) return false;
    int base = count / ngroups, extra = count % ngroups, at = 0;
    for (int g = 0; g < ngroups; ++g) {
        nt[g] = base + (g < extra ? 1 : 0);
        t0[g] = at;
        at += nt[g];
    }
    return true;
}

// Index ranges the kernels assume, checked for every plan before it is used or listed:
//  - one image's operand words (and one spare channel) are addressed with 32-bit byte
//    offsets, and padded rows with 32-bit indices;
//  - a wave's slice of the kernel-word stream (cpw channels, plus the padding steps) is
//    indexed with 32-bit word offsets;
//  - the operand spread and the fused epilogue give every padded row 2^q threads in one
//    launch of fewer than 2^32 threads.
bool addressable(const samd_conv2d_desc &d, const Conv2dGeom &g) {
    const int64_t two31 = (int64_t)1 << 31;
    const int64_t rows = (int64_t)d.N * d.C * g.Hp;
    const int rpb = 256 >> spread_qshift(g.nq);
    return (int64_t)(d.C + 1) * g.Hp * g.ntw * g.nq * 4 < two31 && rows < two31 &&
           ((int64_t)g.cpw * g.nrt + kStreamPad) * kWaveM < two31 &&
           (rows + rpb - 1) / rpb * 256 <= (int64_t)0xffffffff;
}

// Batches between two reads of the lanes; returns how often a wave reads them.
int64_t set_period(Conv2dGeom &t) {
    const int64_t hold = (int64_t)t.G * t.nrt;           // steps the lanes hold
    if (t.rows_path) {
        t.period = (int32_t)std::min<int64_t>((int64_t)t.G * t.ntw, INT32_MAX);
        if (t.KH == 3 && t.period > 1) t.period &= ~1;   // the multiply loop takes pairs of batches
        return ((int64_t)t.cpw * t.ntw + t.period - 1) / t.period;
    }
    t.period = (int32_t)(hold >= kStepBatch ? std::min<int64_t>(hold / kStepBatch, INT32_MAX) : -hold);
    if (t.period > 1) t.period &= ~1;                    // the multiply loop takes pairs of batches
    const int64_t per = hold >= kStepBatch ? (int64_t)t.period * kStepBatch : hold;
    return ((int64_t)t.cpw * t.nrt + per - 1) / per;
}

// The form of two-level lanes a launch can use (Conv2dGeom::two: the wave's lanes widened
// in registers after every period and decoded into the tile once, instead of decoded after
// every period), 0 for none.  Exact when every sum stays within its field: fewer than 2^L
// periods for the 2 L-bit fields, the top lane's total over the slice within the bits above
// it (1), or apart in 32 bits where an odd lane count leaves it above every widened field
// (2).  odd_mask: the odd lanes of an accumulator shifted right by one lane.
int wide_form(const Conv2dGeom &t, int64_t periods, i128 top_per_channel, uint64_t &odd_mask) {
    const int L = t.L, nl = t.nl, top = (nl - 1) * L;
    if (periods < 2 || nl < 2 || t.rh > 2 || t.wm * t.ks * 64 > kMaxWideThreads) return 0;
    if (L < 30 && periods >= ((int64_t)1 << L)) return 0;
    const i128 total = top_per_channel * t.cpw + 1;
    int form = 1;
    if (nl % 2) {
        if (total * pow2(top) > pow2(63)) form = 2;
    } else {
        const int last = (nl - 2) * L;                   // the top lane in `odd`, the highest even lane in `even`
        if (total * pow2(last) > pow2(63) || (i128)periods * pow2(L) > pow2(64 - last)) return 0;
    }
    odd_mask = 0;
    for (int j = 1; j < nl - 1; j += 2) odd_mask |= (((uint64_t)1 << L) - 1) << ((j - 1) * L);
    if (nl % 2 == 0) odd_mask |= ~(uint64_t)0 << ((nl - 2) * L);
    return form;
}

// Modelled time of one launch of the multiply kernel, in units of 4 clocks.  The form
// follows the kernel - a wave's instructions (multiply-adds, lane reads, write-out rows,
// per-batch and fixed scalar work), the issue rate of the waves a SIMD holds, the texture
// path's operand loads and the LDS atomics a compute unit's SIMDs share, a wave's own time
// as the lower bound, whole workgroups per compute unit of the busiest XCD, the tickets of
// an XCD.  Its constants were fitted to 7658 launches of about 330 layers timed on MI355X, a
// few factors then set by single layers; the write-out, the tickets and the lanes counted at run
// time were fitted again to 27727 launches of 1500 drawn layers when the write-out changed.  On
// 6063 launches of 300 other layers it is about 16 % above the time, with a spread of 15 % around
// that; its choice among a layer's timed launches is 3.2 % from the fastest on average, and
// more than 10 % from it for 7 % of the layers (4.0 % and 11 % with these terms as they were).
// All constants fitted anew brought the average to 2.8 %, but cost 8 x 128 x 56 x 56 -> 128 at 8
// bits 4 %.
// A launch that is certain to cost `most` or more is priced no further: what is returned then is
// a lower bound of at least `most`, from the terms that need no pow().
double multiply_cost(const Conv2dGeom &t, int64_t periods, double most) {
    const double waves = (double)t.wm * t.ks, acc = (double)kWaveM * t.rh;
    const double mads = acc * t.cpw * t.nrt;
    // lanes beyond those the kernel unrolls the decode for are counted at run time, twice the price
    double reads, atomics = acc * t.nl;
    if (t.two) {
        reads = 1.28 * acc * periods * (t.two == 2 ? 8.0 : 6.0) + (t.nl > 7 ? 2.4 : 1.2) * acc * (5.0 + 3.0 * t.nl);
    } else {
        reads = (t.nl > 8 ? 2.4 : 1.2) * acc * periods * (4.0 + 2.0 * t.nl);
        atomics *= periods;
    }
    // a wave's rows of the tile, as the write-out takes them: 128 columns a step, or, up to 64
    // columns, one to eight rows at a time
    const int width = t.ncs > 1 ? t.cw : t.Wo;
    const int at_once = t.ncs > 1 || width > 32 ? 1 : width > 16 ? 2 : width > 8 ? 4 : 8;
    const double rows = std::ceil((double)t.mblk * t.rows_blk / waves);
    const double out = width > 64 ? rows * (60.0 + 16.0 * ((width - 1) / 128 + 1)) : 57.6 * std::ceil(rows / at_once);
    const double loads = t.rows_path ? (double)t.cpw * t.ntw * (t.rh + t.KH - 1.0) : (double)t.cpw * t.nrt * t.rh;
    const double batches = (double)t.cpw * t.nrt / 3.0;
    const double slots = (t.rh == 1 ? 0.72 : 0.77) * mads + reads + out + 220.0 +
                         2.0 * t.lds_words / 256.0 / waves + batches * (t.rows_path ? 2.06 : t.nrt % 3 == 0 ? 9.0 : 14.9);
    // waves per SIMD the kernel's registers allow (as compiled for gfx950)
    const int regs = t.two ? (t.rh == 1 ? (t.rows_path ? 6 : 5) : (t.two == 1 && t.rows_path ? 4 : 3))
                           : (t.rh == 1 ? 7 : t.rh == 2 && t.rows_path ? 5 : 4);
    const double res = std::max(1.0, std::min(std::floor(163840.0 / (t.lds_words * 4.0 + 64.0)),
                                              std::floor(4.0 * regs / waves)));
    // workgroups per compute unit of the XCD with the most tiles (32 compute units each)
    const double items = (double)((t.tiles + kNumXcd - 1) / kNumXcd) * t.nmb / 32.0;
    const double held = std::min(res, std::max(1.0, std::ceil(items))) * waves / 4.0;   // waves per SIMD
    const double share = std::max(items, 1.0);
    // the busiest compute unit holds whole workgroups
    const double whole = items > 1.0 && items <= res ? std::ceil(items) / items - 1.0 : 0.0;
    const double tex = share * waves * loads * (t.rows_path ? 5.6 : 6.5) * (1.0 + 1.64 * whole);
    const double solo = slots * 6.0 + (t.rows_path ? 66.0 : 110.0) * (batches + 2.0);
    // rounds of equal workgroups where not all are resident
    const double rounds = items > res ? std::ceil(items / res - 0.02) : 1.0;
    const double group = std::max(solo, waves * loads * 9.5);
    // items past the resident workgroups each take a ticket from their XCD's one counter, which
    // long items hide
    const double tickets = 32.0 * 22.0 * std::max(items - res, 0.0) / (1.0 + solo / 8000.0);
    const auto total = [&](double busy) {
        busy += 0.11 * share * waves * atomics;
        if (items > res) busy *= 1.0 + 0.194 * (std::ceil(items / res) - items / res) * res / items;
        // one row per lane: three loads feed 24 products of eight accumulators; with two kernel
        // words per row the wave waits for both more than the above says
        if (t.rows_path && t.rh == 1 && t.ntw == 2 && !t.two) busy *= 1.08;
        // two-level lanes of two rows leave three or four waves per SIMD to hide those loads
        if (t.rows_path && t.rh == 2 && t.ntw == 2 && t.two) busy *= 1.13;
        // three and four rows per lane press on the registers
        if (t.rh > 2) busy *= 1.1;
        // workgroups of fewer than 4 waves do not fill a compute unit's SIMDs evenly: after
        // another kernel some SIMDs get one wave more than the rest (launches of 1792
        // 2-wave workgroups took 66-68 us instead of 56)
        if (waves < 4.0 && items > 1.0 && items <= 2.0 * res) busy *= 1.0 + 0.6 / held;
        // nor do two or three 4-wave workgroups fall on every compute unit (371 x 57 x 197 -> 85,
        // stride 2, 8 bits: 83 us with 4 waves, 66 with 8)
        else if (waves == 4.0 && items > 1.0 && items <= 3.0) busy *= 1.06;
        // the waves of a large workgroup end, and write their tile, together
        busy *= waves > 8.0 ? 1.3 : waves > 4.0 ? 1.08 : 1.0;
        return (std::max(busy, group * rounds) + 0.325 * solo + tickets) / 4.0 + 1650.0;
    };
    // issue at a clock each 4 cycles, with nothing added for the texture path
    const double least = total((1.0 - 1e-9) * std::max(share * waves * slots * (1.0 + 0.72 * whole), tex));
    if (least >= most) return least;
    const double clk = 4.0 * (1.0 + 0.366 / std::pow(held, 1.86));                      // clocks per instruction
    const double work = share * waves / 4.0 * slots * clk * (1.0 + 0.72 * whole);
    return total(std::pow(std::pow(work, 1.565) + std::pow(tex, 1.565), 1.0 / 1.565));
}

// What a search is after: the cheapest plan whose workspace is within `limit` bytes, and, with
// `all`, every such plan, priced and appended to it.
struct Search {
    std::vector<Conv2dGeom> *all = nullptr;
    size_t limit = SIZE_MAX;
};

// Launch shapes of one lane geometry: output rows per thread (rh), row groups per wave,
// output-channel waves (wm) and channel-slice waves (ks) per workgroup, and whether the
// lane's rows share operand loads (3- and 5-row, stride-1 kernels); the cheapest is kept.
// Returns false when no tile fits the LDS, or none costs less than `most`.
bool place_launch(const samd_conv2d_desc &d, Conv2dGeom &c, i128 top_per_channel, double most,
                  const Search &how, bool &range_limited) {
    const int grp_max = 64 / c.nqs;
    const bool rows_ok = d.stride_h == 1 && ((d.KH == 3 && (c.ntw == 1 || c.ntw == 2)) || d.KH == 5);
    bool found = false;
    c.spread_words = (int64_t)d.N * d.C * c.Hp * c.ntw * c.nq;
    // the operand spread (the permanent-spacer layout has none) and the multiply's first read of
    // the words, at 4 TB/s
    const double spread = (double)c.spread_words * 1e-6 * 587.5 * (c.layout_spaced ? 1.0 : 0.3 * c.I + 1.9);
    Conv2dGeom best = c, t = c;
    best.cost = most;
    for (int rows = 0; rows <= (rows_ok ? 1 : 0); ++rows) {
    for (int rh = 1; rh <= (rows && d.KH == 3 ? 4 : 2); ++rh) {
        if (rh > 1 && c.Ho < rh) continue;
        for (int gr = grp_max; gr >= 1; --gr) {
            const int rows_blk = std::min(rh * gr, c.Ho), row_tiles = (c.Ho + rows_blk - 1) / rows_blk;
            const double xcd_tiles = (d.N * row_tiles * c.ncs + kNumXcd - 1) / kNumXcd;
            // tile row stride: the columns a row needs, padded so that the rows of
            // neighbouring lane groups start on different LDS banks (row groups are
            // rh rows apart; their offset mod 32 banks should not be a multiple of
            // the lane stride I)
            int tile_row = c.nqs * c.I + c.Kmax - 1;
            for (int pad = 0; pad < c.I && c.I > 1; ++pad)
                if ((rh * (tile_row + pad)) % 32 % c.I != 0) {
                    tile_row += pad;
                    break;
                }
            for (int wm : {1, 2, 4}) {
                // at most 8 channel slices: 16-wave workgroups measured 1.0-1.8x slower than
                // 8-wave ones on 512-channel layers (all 16 waves decode into one tile)
                for (int ks : {1, 2, 4, 8}) {
                    if (wm * ks > kMaxBlockWaves) continue;
                    if (ks > 1 && (d.C + ks - 1) / ks < 1) continue;
                    t.cpw = (d.C + ks - 1) / ks;           // channels per slice
                    t.mblk = wm * kWaveM;
                    t.nmb = (d.M + t.mblk - 1) / t.mblk;
                    // most launch shapes are far from the cheapest: their multiply-adds alone
                    // show it, without a look at the rest
                    const double slots = (1.0 - 1e-9) * (0.72 * kWaveM * rh * t.cpw * c.nrt + 220.0);
                    const double waves = std::max(xcd_tiles * t.nmb / 32.0, 1.0) * wm * ks;
                    if (!how.all && (std::max(waves, 6.0) + 0.325 * 6.0) * slots / 4.0 + 1650.0 + spread >= best.cost) continue;
                    t.rows_path = rows;
                    t.rh = rh;
                    t.groups = gr;
                    t.rows_blk = rows_blk;
                    t.trows = (t.rows_blk - 1) * d.stride_h + d.KH;
                    t.wm = wm;
                    t.ks = ks;
                    t.tile_rows = gr * rh;
                    t.tile_row = tile_row;
                    t.lds_tile = (t.mblk * t.tile_rows * t.tile_row + 3) / 4 * 4;
                    t.lds_words = t.lds_tile;
                    if ((long)t.lds_words * 4 > kMaxLdsBytes) continue;
                    if (ks > 1 && (long)(ks - 1) * t.cpw >= d.C) continue;   // an empty slice
                    t.chk = t.cpw * ks;
                    t.row_tiles = row_tiles;
                    t.tiles = d.N * t.row_tiles * c.ncs;
                    t.kw_words = (int64_t)t.nmb * wm * ((int64_t)d.C * c.nrt + kStreamPad) * kWaveM;
                    if (!addressable(d, t)) {
                        range_limited = true;
                        continue;
                    }
                    if (conv2d_workspace_bytes(t) > how.limit) continue;

                    // lanes read into the tile after every period, or widened in between:
                    // whichever is cheaper
                    const int64_t periods = set_period(t);
                    const double bar = how.all ? 1e300 : best.cost - spread;
                    t.bias = t.result_signed ? t.msb_mask : 0;
                    t.two = 0;
                    t.odd_mask = 0;
                    t.cost = multiply_cost(t, periods, bar);
                    uint64_t odd_mask = 0;
                    if (const int form = wide_form(t, periods, top_per_channel, odd_mask)) {
                        t.two = form;
                        const double cost = multiply_cost(t, periods, std::min(bar, t.cost));
                        if (cost < t.cost) {
                            t.odd_mask = odd_mask;
                            t.cost = cost;
                        } else {
                            t.two = 0;
                        }
                    }
                    t.cost += spread;
                    if (how.all) how.all->push_back(t);
                    if (t.cost < best.cost) {
                        best = t;
                        found = true;
                    }
                }
            }
        }
    }
    }
    if (found) {
        const double keep = c.macs_per_mad;
        c = best;
        c.macs_per_mad = keep;
    }
    return found;
}

}  // namespace

namespace {

// xf: the activations as the lanes see them; xoff: the value subtracted from every
// stored activation before it enters a lane (0, or 2^(b-1) for recentred unsigned
// activations, which then behave as signed b-bit values).
// layout: 1 for the permanent-spacer layout (operand words held by the caller).
// msb: lanes of signed results keep their MSB as a spacer bit - their values fit L - 1
// bits - so the decode can leave out the fix-up's final xor (Sec. 6.1); it halves the
// channels a lane holds, so the planner prices both.
int search_lanes(const samd_conv2d_desc &d, samd_fmt xf, samd_fmt wf, int xoff, int layout, int msb,
                 const Search &how, Conv2dGeom &best, std::string &err) {
    Conv2dGeom g = {};
    g.N = d.N; g.C = d.C; g.H = d.H; g.W = d.W; g.M = d.M; g.KH = d.KH; g.KW = d.KW;
    g.sh = d.stride_h; g.sw = d.stride_w; g.ph = d.pad_h; g.pw = d.pad_w;
    g.Ho = (d.H + 2 * d.pad_h - d.KH) / d.stride_h + 1;
    g.Wo = (d.W + 2 * d.pad_w - d.KW) / d.stride_w + 1;
    g.xbits = xf.bits; g.xsigned = xoff ? 0 : xf.is_signed; g.wbits = wf.bits; g.wsigned = wf.is_signed;
    g.xoff = xoff;
    g.result_signed = (xf.is_signed || wf.is_signed) ? 1 : 0;
    g.layout_spaced = layout ? 1 : 0;
    g.spacer = layout && msb && g.result_signed ? 1 : 0;
    g.xrw = (int32_t)row_words(d.W, xf.bits);
    g.wrw = (int32_t)row_words(d.KW, wf.bits);

    const int S = d.stride_w;
    g.Kmax = (d.KW + S - 1) / S;
    const i128 prod = max_abs(xf.bits, xf.is_signed) * max_abs(wf.bits, wf.is_signed);
    bool found = false, range_limited = false;
    best.cost = 1e300;

    for (int L = 2; L <= 31; ++L) {
        // widest kernel word and input word that stay int32 at this lane width
        int kmax = 0;
        for (int k = 1; k <= g.Kmax; ++k)
            if (word_fits(wf.bits, wf.is_signed, L, k, kI32Min, kI32Max)) kmax = k;
        if (kmax == 0) continue;
        int imax = 0;
        for (int i = 1; i <= kMaxLanes; ++i)
            if (word_fits(xf.bits, xf.is_signed, L, i, kI32Min, kI32Max)) imax = i;
        for (int I = 1; I <= imax; ++I) {
            Conv2dGeom c = g;
            c.L = L;
            c.I = I;
            // kernel words: every stride phase's taps in groups of at most kmax
            c.ntw = 0;
            bool ok = true;
            for (int r = 0; r < S && ok; ++r) {
                int Kr = r < d.KW ? (d.KW - r + S - 1) / S : 0;
                if (Kr == 0) continue;
                int t0[kMaxTapWords], nt[kMaxTapWords], ng;
                if (!split_taps(Kr, kmax, t0, nt, ng)) {
                    ok = false;
                    break;
                }
                for (int q = 0; q < ng; ++q) {
                    if (c.ntw >= kMaxTapWords) { ok = false; break; }
                    c.tw_phase[c.ntw] = r;
                    c.tw_tap0[c.ntw] = t0[q];
                    c.tw_ntaps[c.ntw] = nt[q];
                    ++c.ntw;
                }
            }
            if (!ok) continue;
            // products per lane for one (channel, kernel row)
            if (I + c.Kmax - 1 > kMaxOutLanes) continue;
            int nj[kMaxOutLanes] = {0};
            int top = -1;
            for (int j = 0; j < I + c.Kmax - 1; ++j) {
                for (int t = 0; t < c.ntw; ++t) nj[j] += pairs_in_lane(j, I, c.tw_ntaps[t]);
                if (nj[j] > 0) top = j;
            }
            c.nl = top + 1;
            if (c.nl > kMaxOutLanes) continue;
            // largest number of channels whose sums every lane (and the whole word) holds
            const i128 cap = c.result_signed ? (c.spacer ? pow2(L - 2) - 1 : pow2(L - 1) - 1) : pow2(L) - 1;
            i128 gmax = d.C;
            i128 place = 0;
            for (int j = 0; j < c.nl; ++j) {
                if (nj[j] == 0) continue;
                i128 per = (i128)d.KH * nj[j] * prod;
                if (j < c.nl - 1) gmax = std::min(gmax, cap / per);
                if (j * L > 62) { gmax = 0; break; }
                place += (i128)nj[j] * pow2(j * L);
            }
            if (gmax >= 1) gmax = std::min(gmax, kI64Max / ((i128)d.KH * prod * place));
            if (gmax < 1) continue;
            c.G = (int32_t)gmax;
            c.msb_mask = 0;
            for (int j = 0; j < c.nl - 1; ++j) c.msb_mask |= (uint64_t)1 << (j * L + L - 1);
            c.nq = (c.Wo + c.Kmax - 1 + I - 1) / I;
            if (c.nq <= 64) {
                c.nqs = c.nq;
                c.cw = c.Wo;
                c.ncs = 1;
            } else {
                // a row too wide for one wave's lanes: column segments of cw output
                // columns (a multiple of I), each needing at most 64 words, words
                // [c0/I, (c0 + cw + Kmax - 2)/I]; the words reaching two segments are
                // computed by both
                c.nqs = 64;
                c.cw = ((c.nqs - 1) * I - (c.Kmax - 2)) / I * I;
                if (c.cw < I) continue;
                c.ncs = (c.Wo + c.cw - 1) / c.cw;
            }
            c.qseg = c.cw / I;
            c.nrt = d.KH * c.ntw;
            c.Hp = d.H + 2 * d.pad_h;
            c.macs_per_mad = (double)I * d.KW / (double)c.ntw;
            // the multiply-adds alone, spread perfectly over every SIMD, bound the cost below
            const double floor_cost = 0.72 * (double)d.N * c.Ho * c.ncs * c.nqs * d.M * d.C * c.nrt / 64.0 / 1024.0;
            if (!how.all && found && floor_cost >= best.cost) continue;
            if (!place_launch(d, c, (i128)d.KH * nj[c.nl - 1] * prod, how.all ? 1e300 : best.cost, how, range_limited)) continue;
            if (c.cost < best.cost) {
                best = c;
                found = true;
            }
        }
    }
    if (!found) {
        char buf[256];
        if (range_limited)
            snprintf(buf, sizeof buf, "the layer exceeds the kernels' index ranges (operand words of one image "
                     "above 2 GiB, a kernel-word slice above 2^31 words, or an operand spread of 2^32 threads or more)");
        else
            snprintf(buf, sizeof buf, "no exact SAMD lane geometry for %d-bit x %d-bit, KW=%d stride %d, Wo=%d",
                     xf.bits, wf.bits, d.KW, d.stride_w, g.Wo);
        err = buf;
        return SAMD_EUNSUPPORTED;
    }
    return SAMD_OK;
}

// Unsigned activations with signed weights may also be recentred: x - 2^(b-1) is a
// signed b-bit value, so products are half as large and a lane holds twice as many;
// the offset comes back exactly as 2^(b-1) times the sum of the weights over each
// output's in-image taps.  Both are planned and the cheaper kept.
int search_layout(const samd_conv2d_desc &d, samd_fmt xf, samd_fmt wf, int xoff, int layout, const Search &how,
                  Conv2dGeom &best, std::string &err) {
    int st = search_lanes(d, xf, wf, xoff, layout, 1, how, best, err);
    if (!layout || !(xf.is_signed || wf.is_signed || xoff)) return st;
    // the permanent-spacer layout of a signed result: also without the spacer MSB
    Conv2dGeom alt;
    std::string err2;
    if (search_lanes(d, xf, wf, xoff, layout, 0, how, alt, err2) == SAMD_OK && (st != SAMD_OK || alt.cost < best.cost)) {
        best = alt;
        st = SAMD_OK;
    }
    return st;
}

int search_conv2d(const samd_conv2d_desc &d, samd_fmt xf, samd_fmt wf, int spacer, const Search &how,
                  Conv2dGeom &best, std::string &err) {
    int st = search_layout(d, xf, wf, 0, spacer, how, best, err);
    if (!xf.is_signed && wf.is_signed && xf.bits >= 2) {
        Conv2dGeom alt;
        std::string err2;
        const samd_fmt xs = {xf.bits, 1};
        const size_t first = how.all ? how.all->size() : 0;
        if (search_layout(d, xs, wf, 1 << (xf.bits - 1), spacer, how, alt, err2) == SAMD_OK) {
            // the correction: in the packed layout one addition per output; in the
            // permanent-spacer layout four table lookups, issued where little hides them
            const double correction = (double)d.N * d.M * alt.Ho * alt.Wo * (spacer ? 20.0 : 0.5) / 64.0 / 1024.0;
            alt.cost += correction;
            if (how.all)
                for (size_t i = first; i < how.all->size(); ++i) (*how.all)[i].cost += correction;
            if (st != SAMD_OK || alt.cost < best.cost) {
                best = alt;
                st = SAMD_OK;
            }
        }
    }
    return st;
}

// Plans are a pure function of (shape, formats); the search prices thousands of launch
// shapes, so found plans are kept (under a lock) and later calls look them up.
using PlanKey = std::array<int32_t, 16>;
std::mutex plan_mu;
std::map<PlanKey, Conv2dGeom> plan_cache;
constexpr size_t kPlanCacheMax = 4096;
// Plans chosen by measurement (samd_conv2d_tune): they take precedence over the model's
// and are kept until cleared, since workspaces prepared under them depend on them.
std::map<PlanKey, Conv2dGeom> tuned_plans;

PlanKey plan_key(const samd_conv2d_desc &d, samd_fmt xf, samd_fmt wf, int spacer) {
    return {d.N, d.C, d.H, d.W, d.M, d.KH, d.KW, d.stride_h, d.stride_w, d.pad_h, d.pad_w,
            xf.bits, xf.is_signed, wf.bits, wf.is_signed, spacer};
}

}  // namespace

int plan_conv2d(const samd_conv2d_desc &d, samd_fmt xf, samd_fmt wf, Conv2dGeom &g, std::string &err,
                int spacer) {
    const PlanKey key = plan_key(d, xf, wf, spacer);
    {
        std::lock_guard<std::mutex> lock(plan_mu);
        auto tu = tuned_plans.find(key);
        if (tu != tuned_plans.end()) {
            g = tu->second;
            return SAMD_OK;
        }
        auto it = plan_cache.find(key);
        if (it != plan_cache.end()) {
            g = it->second;
            return SAMD_OK;
        }
    }
    int st = search_conv2d(d, xf, wf, spacer, Search{}, g, err);
    if (st == SAMD_OK && !addressable(d, g)) {
        err = "the layer exceeds the kernels' index ranges (operand words of one image above 2 GiB, a kernel-word "
              "slice above 2^31 words, or an operand spread of 2^32 threads or more)";
        st = SAMD_EUNSUPPORTED;
    }
    if (st == SAMD_OK) {
        std::lock_guard<std::mutex> lock(plan_mu);
        if (plan_cache.size() >= kPlanCacheMax) plan_cache.clear();
        plan_cache.emplace(key, g);
    }
    return st;
}

int plan_conv2d_scratch(const samd_conv2d_desc &d, samd_fmt xf, samd_fmt wf, Conv2dGeom &g, std::string &err) {
    constexpr size_t limit = SAMD_NOALLOC_SCRATCH_BYTES;
    int st = plan_conv2d(d, xf, wf, g, err);
    if (st != SAMD_OK || conv2d_workspace_bytes(g) <= limit) return st;
    PlanKey key = plan_key(d, xf, wf, 0);
    std::unique_lock<std::mutex> lock(plan_mu);
    if (tuned_plans.count(key)) return SAMD_OK;
    key.back() = -1;   // the fitting plan's own entry; one without lanes: no plan fits
    auto it = plan_cache.find(key);
    if (it == plan_cache.end()) {
        lock.unlock();
        Conv2dGeom fit;
        std::string none;
        if (search_conv2d(d, xf, wf, 0, Search{nullptr, limit}, fit, none) != SAMD_OK) fit = {};
        lock.lock();
        if (plan_cache.size() >= kPlanCacheMax) plan_cache.clear();
        it = plan_cache.emplace(key, fit).first;
    }
    if (it->second.L) g = it->second;
    return SAMD_OK;
}

int conv2d_candidates(const samd_conv2d_desc &d, samd_fmt xf, samd_fmt wf, int max_count,
                      std::vector<Conv2dGeom> &out, std::string &err, int spacer) {
    out.clear();
    // the model alone (no cache, no tuned plan): its choice, then every priced candidate
    Conv2dGeom model;
    std::vector<Conv2dGeom> all;
    int st = search_conv2d(d, xf, wf, spacer, Search{&all}, model, err);
    if (st) return st;
    if (!addressable(d, model)) {
        err = "the layer exceeds the kernels' index ranges (operand words of one image above 2 GiB, a kernel-word "
              "slice above 2^31 words, or an operand spread of 2^32 threads or more)";
        return SAMD_EUNSUPPORTED;
    }
    std::vector<Conv2dGeom> keep;
    for (const Conv2dGeom &c : all)
        if (addressable(d, c)) keep.push_back(c);
    std::stable_sort(keep.begin(), keep.end(),
                     [](const Conv2dGeom &a, const Conv2dGeom &b) { return a.cost < b.cost; });
    auto same = [](const Conv2dGeom &a, const Conv2dGeom &b) {
        return a.L == b.L && a.I == b.I && a.xoff == b.xoff && a.rows_path == b.rows_path && a.rh == b.rh &&
               a.groups == b.groups && a.wm == b.wm && a.ks == b.ks && a.spacer == b.spacer;
    };
    out.push_back(model);
    for (const Conv2dGeom &c : keep) {
        if ((int)out.size() >= max_count) break;
        bool dup = false;
        for (const Conv2dGeom &o : out) dup = dup || same(o, c);
        if (!dup) out.push_back(c);
    }
    return SAMD_OK;
}

int find_conv2d_candidate(const samd_conv2d_desc &d, samd_fmt xf, samd_fmt wf,
                          const std::function<bool(const Conv2dGeom &)> &match, Conv2dGeom &out,
                          std::string &err, int spacer) {
    // every priced candidate, unsorted (matching needs no ranking)
    Conv2dGeom model;
    std::vector<Conv2dGeom> all;
    int st = search_conv2d(d, xf, wf, spacer, Search{&all}, model, err);
    if (st) return st;
    for (const Conv2dGeom &c : all)
        if (addressable(d, c) && match(c)) {
            out = c;
            return SAMD_OK;
        }
    err = "no candidate plan of this shape matches";
    return SAMD_EINVAL;
}

void set_tuned_conv2d(const samd_conv2d_desc &d, samd_fmt xf, samd_fmt wf, const Conv2dGeom &g) {
    std::lock_guard<std::mutex> lock(plan_mu);
    tuned_plans[plan_key(d, xf, wf, g.layout_spaced)] = g;
}

void clear_tuned_conv2d(const samd_conv2d_desc *d, samd_fmt xf, samd_fmt wf) {
    std::lock_guard<std::mutex> lock(plan_mu);
    if (!d)
        tuned_plans.clear();
    else
        for (int spacer : {0, 1}) tuned_plans.erase(plan_key(*d, xf, wf, spacer));
}

// Workspace: kernel-word streams, the recentring correction table, the work queues of
// the multiply kernel, then the operand words of one call (each 256-byte aligned).
size_t conv2d_kw_bytes(const Conv2dGeom &g) { return ((size_t)g.kw_words * 4 + 255) / 256 * 256; }

size_t conv2d_pre_bytes(const Conv2dGeom &g) {
    // one sum per output channel, or the prefix table of the permanent-spacer layout
    const size_t per = g.layout_spaced ? (size_t)(g.KH + 1) * (g.KW + 1) : 1;
    return g.xoff ? ((size_t)g.M * per * 4 + 255) / 256 * 256 : 0;
}

size_t conv2d_queue_offset(const Conv2dGeom &g) { return conv2d_kw_bytes(g) + conv2d_pre_bytes(g); }

size_t conv2d_xs_offset(const Conv2dGeom &g) { return conv2d_queue_offset(g) + kQueueBytes; }

size_t conv2d_workspace_bytes(const Conv2dGeom &g) {
    // one spare channel after the last image: the batch fetched after a slice's last one
    // may read it (its products are never used)
    const size_t spare = (size_t)g.Hp * g.ntw * g.nq;
    return conv2d_xs_offset(g) + ((size_t)(g.spread_words + spare) * 4 + 255) / 256 * 256;
}

namespace {

// The geometry of L-bit lanes and I values per operand word; false where no word holds a
// tap, a lane overflows or a limit of the kernel is passed.
bool conv1d_geometry(const Conv1dGeom &g, int xbits, int kbits, const int32_t *taps, int L, int I, Conv1dGeom &c) {
    const i128 xmax = pow2(xbits) - 1, kmax_v = pow2(kbits) - 1;
    const i128 u32max = pow2(32) - 1, u64max = pow2(64) - 1;
    int kmax = 0;
    for (int k = 1; k <= g.K; ++k)
        if (word_fits(kbits, false, L, k, 0, u32max)) kmax = k;
    if (kmax == 0) return false;
    c = g;
    c.L = L;
    c.I = I;
    int t0[kMaxTapWords], nt[kMaxTapWords];
    if (!split_taps(g.K, kmax, t0, nt, c.ngroups)) return false;
    // lanes: j <-> output q*I + j - (K - 1); group g's window starts at q*I - t0[g]
    int nl = I + g.K - 1, top = -1;
    if (nl > 64) return false;
    int nj[64] = {0};
    for (int j = 0; j < nl; ++j) {
        for (int q = 0; q < c.ngroups; ++q) nj[j] += pairs_in_lane(j, I, nt[q]);
        if (nj[j]) top = j;
    }
    i128 total = 0;
    for (int j = 0; j <= top; ++j) {
        const i128 dmax = (i128)nj[j] * xmax * kmax_v;
        if (j < top && dmax > pow2(L) - 1) return false;
        if (j * L > 63 && dmax > 0) return false;
        total += dmax * pow2(j * L);
    }
    if (total > u64max) return false;
    c.nl = top + 1;
    for (int q = 0; q < c.ngroups; ++q) {
        c.g_tap0[q] = t0[q];
        c.g_ntaps[q] = nt[q];
        c.g_delta[q] = -t0[q];
        uint64_t word = 0;
        for (int s = 0; s < nt[q]; ++s) word |= (uint64_t)(uint32_t)taps[t0[q] + s] << (s * L);
        c.g_word[q] = (uint32_t)word;
    }
    c.extra = (g.K - 1 + I - 1) / I;
    if (c.extra > kMaxConv1dExtra) return false;
    c.nwords = (c.nout + I - 1) / I;
    return true;
}

}  // namespace

// The lanes depend on the widths and the number of taps alone, so the search over them (10 us
// of a call whose kernel takes 4.6) runs once for each of the 8 x 8 x 16 combinations; the
// entries are single words that any thread may write with the same value.
int plan_conv1d(int64_t n, samd_fmt xf, const int32_t *taps, int32_t K, samd_fmt kf, Conv1dGeom &best,
                std::string &err) {
    static std::atomic<uint16_t> lanes[8][8][16];
    Conv1dGeom g = {};
    g.n = n;
    g.nout = n - K + 1;
    g.bits = xf.bits;
    g.K = K;
    g.xrw = (int32_t)row_words(n, xf.bits);
    std::atomic<uint16_t> &known = lanes[xf.bits - 1][kf.bits - 1][K - 1];
    if (const int li = known.load(std::memory_order_relaxed))
        if (conv1d_geometry(g, xf.bits, kf.bits, taps, li >> 8, li & 255, best)) return SAMD_OK;
    double best_cost = 1e300;
    bool found = false;
    for (int L = 1; L <= 32; ++L) {
        int imax = 0;
        for (int i = 1; i <= 32; ++i)
            if (word_fits(xf.bits, false, L, i, 0, pow2(32) - 1)) imax = i;
        for (int I = 1; I <= std::min(imax, kConv1dMaxLanes); ++I) {
            Conv1dGeom c;
            if (!conv1d_geometry(g, xf.bits, kf.bits, taps, L, I, c)) continue;
            double cost = (double)c.ngroups * (1 + c.extra) * (2.0 + 3.0 * I) / I + 3.0 * (I + K) * (1 + c.extra) / I;
            if (cost < best_cost) {
                best_cost = cost;
                best = c;
                found = true;
            }
        }
    }
    if (!found) {
        err = "no exact SAMD lane geometry for this 1-D convolution";
        return SAMD_EUNSUPPORTED;
    }
    known.store((uint16_t)(best.L << 8 | best.I), std::memory_order_relaxed);
    return SAMD_OK;
}

}  // namespace samd
