"""The lane geometries the library plans, checked on the CPU with Python integers.

For every workload shape and bit width the planner's geometry (lane width L, values per
operand word I, kernel-word tap groups, channels per decode G) is replayed here in plain
Python, independently of the HIP code: operand and kernel words must be int32, the
64-bit accumulator must hold every partial sum, and decoding the lanes with the fix-up
of the signed-convolution figure must give the direct sums - for extreme inputs at the
bound, and for a complete small convolution compared with the oracle, which follows the
multiply kernel's form: its order of steps, when it reads the lanes, and how (decoded, or
widened and decoded at the end)."""
import functools
import itertools
import random

import numpy as np
import pytest

import paper_1809_10572_amd as samd
import samd_workloads as wl
from oracle import reference as ref
from oracle import samd_model as sm
import test_gpu_multiply_forms as multiply

I32 = (-(1 << 31), (1 << 31) - 1)


def tap_words(plan):
    return [(plan.phase[t], plan.tap0[t], plan.ntaps[t]) for t in range(plan.tap_words)]


def decode_lanes(V, L, nl, signed):
    """Lanes 0..nl-1 of an exact accumulator; the top lane takes all remaining bits."""
    if signed:
        word = V & ((1 << 64) - 1)
        mask = sum(1 << (j * L + L - 1) for j in range(nl - 1))
        s = word & mask
        fixed = ((word + s) & ((1 << 64) - 1)) ^ s
        lanes = sm.word_to_lanes(fixed, L, nl - 1, signed=True)
        top = sm.to_signed(fixed, 64) >> ((nl - 1) * L)
        return lanes + [top]
    lanes = sm.word_to_lanes(V, L, nl - 1, signed=False)
    return lanes + [V >> ((nl - 1) * L)]


def odd_lanes(L, nl):
    """The lanes 1, 3, ... of an accumulator shifted right by one lane; the top lane has every
    bit above its first."""
    mask = sum(((1 << L) - 1) << ((j - 1) * L) for j in range(1, nl - 1, 2))
    if nl % 2 == 0:
        mask |= (1 << 64) - (1 << ((nl - 2) * L))
    return mask


def read_slice(words, plan, form):
    """Lane sums of one wave's slice of the channels: words holds, per channel, the products of
    its steps (kernel row ky, kernel word t), and the accumulator is read after every period."""
    L, nl = plan.lane_bits, plan.out_lanes
    top, M64 = (nl - 1) * L, (1 << 64) - 1
    if form.kernel_rows >= 3:     # a batch: one kernel word of one channel, all its kernel rows
        batches = [sum(w[ky][t] for ky in range(len(w))) for w in words for t in range(plan.tap_words)]
        size = form.period
    else:                         # batches of three steps, or periods of fewer
        batches = [p for w in words for row in w for p in row]
        size = 3 * form.period if form.period > 0 else -form.period
    # accumulators of signed results start with half a lane's range in every lane below the top
    bias = sum(1 << (j * L + L - 1) for j in range(nl - 1)) if form.result_signed else 0
    lanes, every, odd, apart, reads = [0] * nl, 0, 0, 0, 0
    for i in range(0, len(batches), size):
        v = bias + sum(batches[i:i + size])
        assert -(1 << 63) <= v < (1 << 63)
        reads += 1
        if form.widened:
            every, odd, apart = (every + v) & M64, (odd + ((v >> L) & form.odd_mask)) & M64, apart + (v >> top)
        elif form.result_signed:
            fixed = (v & M64) ^ bias
            got = sm.word_to_lanes(fixed, L, nl - 1, signed=True) + [sm.to_signed(fixed, 64) >> top]
            lanes = [a + b for a, b in zip(lanes, got)]
        else:
            lanes = [a + b for a, b in zip(lanes, decode_lanes(v, L, nl, False))]
    if form.widened:
        even = (every - (odd << L)) & M64
        field = min(2 * L, 32)
        offset = reads << (L - 1) if form.result_signed else 0
        for j in range(nl - 1):
            word = odd >> ((j - 1) * L) if j % 2 else even >> (j * L)
            lanes[j] = sm.to_signed(((word & ((1 << field) - 1)) - offset) & 0xffffffff, 32)
        inside = sm.to_signed(even, 64) >> top if nl % 2 else sm.to_signed(odd, 64) >> ((nl - 2) * L)
        lanes[nl - 1] = apart if form.widened == 2 else inside
    return lanes


def planned_conv2d(x, w, shape, xf, wf, plan, form, filters=None, rows=None):
    """The planned SAMD convolution on Python integers: operand words of I phase values,
    kernel words of reversed taps, exact products, the lanes of every channel slice read as the
    form says and added into the outputs they belong to (of all filters and rows, or of some)."""
    N, C, H, W, M, KH, KW, sh, sw, ph, pw = shape
    Ho, Wo = ref.out_hw(shape)
    L, I, Kmax = plan.lane_bits, plan.lanes, plan.taps_max
    nq, off = plan.words_per_row, plan.x_offset
    tws = tap_words(plan)
    assert form.result_signed == int(xf.is_signed or wf.is_signed)
    if form.widened:
        assert form.odd_mask == odd_lanes(L, plan.out_lanes)
    y = np.zeros((N, M, Ho, Wo), dtype=np.int64)

    def xval(n, c, h, col):
        # recentred activations enter the lanes as x - off, the zero padding too
        return (int(x[n, c, h, col]) if 0 <= h < H and 0 <= col < W else 0) - off

    def xword(n, c, h, t, q):
        r, a0, k = tws[t]
        A = sum(xval(n, c, h, sw * (q * I + a0 + k - Kmax + i) + r - pw) << (i * L) for i in range(I))
        assert I32[0] <= A <= I32[1]
        return A

    def wword(m, c, ky, t):
        r, a0, k = tws[t]
        B = sum(int(w[m, c, ky, sw * (a0 + k - 1 - s) + r]) << (s * L) for s in range(k))
        assert I32[0] <= B <= I32[1]
        return B

    filters, rows = filters or range(M), rows or range(Ho)
    kernel = {(m, c, ky, t): wword(m, c, ky, t) for m in filters for c in range(C) for ky in range(KH) for t in range(len(tws))}
    per = plan.chunk_channels // plan.split_waves        # channels of a wave's slice
    for n, ho, q in itertools.product(range(N), rows, range(nq)):
        A = [[[xword(n, c, ho * sh + ky - ph, t, q) for t in range(len(tws))] for ky in range(KH)] for c in range(C)]
        for m in filters:
            for c0 in range(0, C, per):
                words = [[[A[c][ky][t] * kernel[m, c, ky, t] for t in range(len(tws))] for ky in range(KH)]
                         for c in range(c0, min(c0 + per, C))]
                for j, d in enumerate(read_slice(words, plan, form)):
                    o = q * I + j - (Kmax - 1)
                    if 0 <= o < Wo:
                        y[n, m, ho, o] += d
    # add back off * the sum of the filter's weights: every output takes every tap
    return y + off * np.asarray(w, dtype=np.int64).sum(axis=(1, 2, 3))[None, :, None, None]


SMALL = [
    (wl.Conv2dShape(1, 5, 4, 11, 2, 3, 3, 1, 1, 1, 1), [(1, 0, 4, 1), (4, 0, 4, 1), (8, 0, 8, 1), (3, 1, 3, 1),
                                                       (6, 1, 6, 1), (2, 1, 5, 0)]),
    (wl.Conv2dShape(1, 2, 9, 13, 2, 11, 11, 4, 4, 2, 2), [(4, 0, 4, 1), (8, 0, 8, 1), (2, 1, 2, 1)]),
    (wl.Conv2dShape(1, 3, 6, 9, 2, 5, 5, 1, 1, 2, 2), [(2, 0, 2, 1), (8, 0, 8, 1), (5, 1, 5, 1)]),
]


@pytest.mark.parametrize("shape,fmts", SMALL, ids=["3x3", "11x11s4", "5x5"])
def test_planned_convolution_matches_oracle(shape, fmts):
    rng = np.random.default_rng(sum(shape.as_tuple()))
    for bx, sx, bw, sw_ in fmts:
        xf, wf = samd.Fmt(bx, sx), samd.Fmt(bw, sw_)
        plan = samd.conv2d_plan(shape, xf, wf)
        gen = wl.half_extremes
        x = gen(rng, (shape.N, shape.C, shape.H, shape.W), bx, bool(sx))
        w = gen(rng, (shape.M, shape.C, shape.KH, shape.KW), bw, bool(sw_))
        got = planned_conv2d(x, w, shape.as_tuple(), xf, wf, plan, samd.conv2d_form(shape, xf, wf))
        np.testing.assert_array_equal(got, ref.conv2d(x, w, shape.as_tuple()), err_msg=str((bx, sx, bw, sw_)))


# layers of every way to read the lanes, with the plans that the GPU test of the forms runs:
# 3-, 5- and 7-row kernels, signed and unsigned results, the top lane's sum inside its word and apart
@pytest.mark.parametrize("kind", ["mixed", "low", "high", "opposite"])
@pytest.mark.parametrize("case", [0, 1, 4, 5, 6, 7])
def test_every_way_to_read_the_lanes_matches_oracle(case, kind):
    shape, xb, xs, wb, ws, _ = multiply.FORMS[case]
    xf, wf = samd.Fmt(xb, xs), samd.Fmt(wb, ws)
    x, w = multiply._operands(kind, shape, xb, xs, wb, ws)
    want = ref.conv2d(x, w, shape)
    filters, rows = [0, 8], [0, 3]
    for form, key in form_plans(case).items():
        try:
            samd.conv2d_use_plan(shape, xf, wf, key)
            got = planned_conv2d(x, w, shape, xf, wf, samd.conv2d_plan(shape, xf, wf), samd.conv2d_form(shape, xf, wf),
                                 filters, rows)
        finally:
            samd.conv2d_untune(shape, xf, wf)
        pick = np.ix_([0], filters, rows, range(want.shape[3]))
        np.testing.assert_array_equal(got[pick], want[pick], err_msg=str((form, key)))


@functools.lru_cache(maxsize=None)
def form_plans(case):
    return multiply.form_plans(case)


@pytest.mark.parametrize("shape,xfmt,wfmt,steps", multiply.FEW_STEPS)
def test_few_steps_per_decode_match_oracle(shape, xfmt, wfmt, steps):
    xf, wf = samd.Fmt(*xfmt), samd.Fmt(*wfmt)
    form = samd.conv2d_form(shape, xf, wf)
    assert form.period == -steps
    x, w = multiply._operands("mixed", shape, *xfmt, *wfmt)
    want = ref.conv2d(x, w, shape)
    filters, rows = [0, shape[4] - 1], [0, shape[2] - 1]
    got = planned_conv2d(x, w, shape, xf, wf, samd.conv2d_plan(shape, xf, wf), form, filters, rows)
    pick = np.ix_(range(shape[0]), filters, rows, range(want.shape[3]))
    np.testing.assert_array_equal(got[pick], want[pick])


def full_shapes():
    out = []
    for cfg, shape in ((1, wl.SINGLE), (3, wl.MID), (4, wl.STRESS)):
        for b in range(1, 9):
            xs, ws = (True, True) if cfg == 4 else (False, True)
            if cfg == 4 and b == 1:
                continue
            out.append((f"cfg{cfg}-b{b}", shape, samd.Fmt(b, xs), samd.Fmt(b, ws)))
    for li, shape in enumerate(wl.ALEXNET_LAYERS):
        for b in (2, 4, 8):
            out.append((f"alex{li + 1}-b{b}", shape, samd.Fmt(b, False), samd.Fmt(b, True)))
    return out


@pytest.mark.parametrize("name,shape,xf,wf", full_shapes(), ids=[f[0] for f in full_shapes()])
def test_planned_geometry_is_exact_at_the_bound(name, shape, xf, wf):
    """Every lane of a word accumulated over G channels of extreme products decodes
    exactly; operand and kernel words are int32 for every value in range."""
    plan = samd.conv2d_plan(shape, xf, wf)
    L, I, Kmax, G = plan.lane_bits, plan.lanes, plan.taps_max, plan.flush_channels
    assert 1 <= G <= shape.C and plan.macs_per_mad > 0
    tws = tap_words(plan)
    assert sum(k for (_, _, k) in tws) == shape.KW
    # recentred unsigned activations reach the lanes as signed b-bit values
    xlo, xhi = wl.value_range(xf.bits, bool(xf.is_signed) or plan.x_offset != 0)
    wlo, whi = wl.value_range(wf.bits, bool(wf.is_signed))
    for lo, hi, n in [(xlo, xhi, I)] + [(wlo, whi, k) for (_, _, k) in tws]:
        place = sum(1 << (i * L) for i in range(n))
        assert lo * place >= I32[0] and hi * place <= I32[1]
    signed = bool(xf.is_signed or wf.is_signed or plan.x_offset)
    rnd = random.Random(hash(name) & 0xFFFF)
    rows = G * shape.KH
    # adversarial operands: every product at its most positive / most negative value,
    # then random mixtures of the extremes
    cases = []
    for mode in ("max", "min", "mix", "mix"):
        xs, wsv = [], []
        for _ in range(rows):
            for (r, a0, k) in tws:
                if mode == "max":
                    xv, wv = (xhi, whi) if xhi * whi >= xlo * wlo else (xlo, wlo)
                    xw = [xv] * I, [wv] * k
                elif mode == "min":
                    xv, wv = (xhi, wlo) if xhi * wlo <= xlo * whi else (xlo, whi)
                    xw = [xv] * I, [wv] * k
                else:
                    xw = [rnd.choice((xlo, xhi)) for _ in range(I)], [rnd.choice((wlo, whi)) for _ in range(k)]
                xs.append(xw[0])
                wsv.append(xw[1])
        cases.append((xs, wsv))
    nl = plan.out_lanes
    assert nl <= I + Kmax - 1
    for xs, wsv in cases:
        acc = 0
        want = [0] * (I + Kmax - 1)
        for idx, (xv, wv) in enumerate(zip(xs, wsv)):
            r, a0, k = tws[idx % len(tws)]
            A = sum(v << (i * L) for i, v in enumerate(xv))
            B = sum(v << (s * L) for s, v in enumerate(wv))
            acc += A * B
            assert -(1 << 63) <= acc < (1 << 63)
            for j, d in enumerate(np.convolve(xv, wv)):
                want[j] += int(d)
        assert all(v == 0 for v in want[nl:])
        assert decode_lanes(acc, L, nl, signed) == want[:nl], name


def test_plan_prefers_more_lanes_for_fewer_bits():
    shape = wl.MID
    mpm = [samd.conv2d_plan(shape, samd.Fmt(b, False), samd.Fmt(b, True)).macs_per_mad for b in (1, 2, 4, 8)]
    assert mpm[0] >= mpm[1] >= mpm[2] >= mpm[3] and mpm[0] > mpm[3]


def test_plan_rejects_what_cannot_be_exact():
    # a 16-tap-wide kernel row of 8-bit values leaves no exact geometry within 32-bit words
    with pytest.raises(samd.SamdError) as e:
        samd.conv2d_plan(wl.Conv2dShape(1, 1, 4, 200, 1, 1, 100, 1, 1, 0, 0), samd.Fmt(8, False), samd.Fmt(8, True))
    assert e.value.status in (samd.SAMD_EUNSUPPORTED,)


def planned_conv1d(x, k, plan):
    """The planned 1-D convolution on Python integers: unsigned operand words of I values
    L bits apart, one kernel word per tap group (natural order), 32x32 -> 64-bit
    products, lanes read out and added into the outputs they belong to."""
    n, K = len(x), len(k)
    L, I, nl = plan.lane_bits, plan.lanes, plan.out_lanes
    nout = n - K + 1
    y = [0] * nout
    nwords = -(-nout // I)
    for q in range(nwords + plan.extra):
        acc = 0
        for g in range(plan.groups):
            t0, kk = plan.tap0[g], plan.ntaps[g]
            A = sum(int(x[q * I - t0 + i]) << (i * L) for i in range(I) if 0 <= q * I - t0 + i < n)
            B = sum(int(k[t0 + s]) << (s * L) for s in range(kk))
            assert A < (1 << 32) and B < (1 << 32)
            acc += A * B
        assert acc < (1 << 64)
        lanes = [(acc >> (j * L)) & ((1 << L) - 1) for j in range(nl - 1)] + [acc >> ((nl - 1) * L)]
        for j, d in enumerate(lanes):
            o = q * I + j - (K - 1)
            if 0 <= o < nout:
                y[o] += d
    return y


@pytest.mark.parametrize("bits", range(1, 9))
def test_planned_conv1d_matches_oracle(bits):
    rng = np.random.default_rng(bits)
    top = (1 << bits) - 1
    for K in (1, 2, 3, 5, 7, 16):
        for n in (K, K + 1, 41, 200):
            for x, k in ((np.full(n, top), np.full(K, top)), (wl.uniform(rng, (n,), bits, False),
                                                             wl.uniform(rng, (K,), bits, False))):
                plan = samd.conv1d_plan(n, bits, k.tolist(), bits)
                assert sum(plan.ntaps[g] for g in range(plan.groups)) == K
                assert planned_conv1d(x, k, plan) == list(ref.conv1d(x, k)), (bits, K, n)
