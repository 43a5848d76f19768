"""The operand-word writer, from its three sources (packed rows, 8-bit values, int32
accumulators), checked through the convolution against the oracle: layers large enough for
its workgroups of rows and ones that are not, strided ones, several values to a word - more
than an LDS word holds fields among them -, recentred words with and without a filled
padding, rows that end inside a word, and rows too long for a workgroup's LDS."""
import numpy as np
import pytest
import torch

import paper_1809_10572_amd as samd
import samd_workloads as wl
from oracle import reference as ref

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# under the plans of their own: few output channels, so mostly one value to a word
CASES = [
    ((2, 9, 31, 61, 4, 3, 3, 1, 1, 1, 1), 1, 1),
    ((2, 9, 31, 62, 4, 3, 3, 1, 1, 1, 1), 3, 3),
    ((2, 9, 30, 59, 4, 3, 3, 1, 1, 1, 1), 5, 5),      # packed words with unused bits
    ((2, 9, 30, 57, 4, 3, 3, 1, 1, 1, 1), 8, 8),
    ((1, 6, 41, 75, 4, 5, 5, 1, 1, 2, 2), 7, 7),      # several kernel words per row
    ((2, 5, 41, 83, 4, 3, 3, 2, 2, 1, 1), 4, 4),      # two stride phases
    ((2, 3, 61, 93, 4, 7, 11, 4, 4, 2, 5), 2, 2),
    ((3, 25, 40, 53, 4, 1, 1, 1, 1, 0, 0), 2, 3),     # 1x1
    ((1, 1, 2, 40000, 3, 3, 3, 1, 1, 1, 1), 8, 8),    # rows beyond a workgroup's LDS
]


@pytest.mark.parametrize("signed", [False, True])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_every_source_matches_the_oracle(case, signed):
    shape, xb, wb = CASES[case]
    N, C, H, W, M, KH, KW = shape[:7]
    rng = np.random.default_rng(100 + case)
    x = wl.half_extremes(rng, (N, C, H, W), xb, signed)
    w = wl.uniform(rng, (M, C, KH, KW), wb, True)
    xf, wf = samd.Fmt(xb, signed), samd.Fmt(wb, True)
    want = ref.conv2d(x, w, shape)
    xv = torch.from_numpy(x.astype(np.int8 if signed else np.uint8)).to(DEV)
    wp = samd.pack(torch.from_numpy(w.astype(np.int8)).to(DEV), wb, True)
    got = {"packed": samd.conv2d(samd.pack(xv, xb, signed), xf, wp, wf, shape)}
    wss = samd.conv2d_spaced_prepare(wp, wf, shape, xf)
    words = samd.conv2d_spaced_pack(xv, xf, wf, shape)
    got["bytes"] = samd.conv2d_spaced(words, xf, wf, shape, wss)
    if not signed:
        # accumulators whose requantised values are x: shift 0 when the maximum is the range's
        acc = torch.from_numpy(x.astype(np.int32)).to(DEV)
        acc[acc == 0] = -5
        mx = torch.full((1,), (1 << xb) - 1, dtype=torch.int32, device=DEV)
        got["accumulators"] = samd.conv2d_spaced(samd.relu_requant_spaced(acc, mx, xb, wf, shape), xf, wf, shape, wss)
        ws = samd.conv2d_prepare(wp, wf, shape, xf)
        samd.relu_requant_stage(acc, mx, xb, wf, shape, ws)
        got["staged"] = samd.conv2d_accumulate(xf, wf, shape, ws)
    torch.cuda.synchronize()
    for name, y in got.items():
        np.testing.assert_array_equal(y.cpu().numpy(), want, err_msg=name)


# (shape, bits, weight bits, values per word, lane bits, recentring offset): pinned plans of
# several values to a word.  The last but one holds more fields to a word than a 32-bit LDS word
# of 8-bit fields, so its words are not cut with a funnel shift; a stride's never are.
PINNED = [
    ((2, 36, 31, 61, 4, 3, 3, 1, 1, 1, 1), 1, 1, 5, 6, 0),
    ((2, 36, 31, 62, 4, 3, 3, 1, 1, 1, 1), 3, 3, 3, 10, 4),
    ((2, 40, 30, 57, 4, 3, 3, 1, 1, 1, 1), 8, 8, 2, 20, 128),
    ((2, 40, 41, 75, 4, 5, 5, 1, 1, 2, 2), 5, 5, 2, 15, 16),
    ((2, 36, 41, 83, 4, 3, 3, 2, 2, 1, 1), 4, 4, 3, 12, 8),
    ((2, 36, 41, 83, 4, 3, 3, 2, 2, 1, 1), 4, 4, 3, 12, 0),
    ((3, 50, 40, 53, 4, 1, 1, 1, 1, 0, 0), 1, 1, 5, 3, 0),
    ((3, 50, 40, 53, 4, 1, 1, 2, 1, 0, 0), 2, 1, 6, 4, 2),
]


@pytest.mark.parametrize("case", range(len(PINNED)))
def test_several_values_to_a_word(case):
    shape, xb, wb, lanes, lane_bits, xoff = PINNED[case]
    N, C, H, W, M, KH, KW = shape[:7]
    xf, wf = samd.Fmt(xb, False), samd.Fmt(wb, True)
    rng = np.random.default_rng(200 + case)
    x = wl.half_extremes(rng, (N, C, H, W), xb, False)
    w = wl.half_extremes(rng, (M, C, KH, KW), wb, True)
    want = ref.conv2d(x, w, shape)
    xv = torch.from_numpy(x.astype(np.uint8)).to(DEV)
    wp = samd.pack(torch.from_numpy(w.astype(np.int8)).to(DEV), wb, True)
    # accumulators that a shift of 3, rounding half up, takes to x: up to 4 below and 3 above 8 x
    acc = torch.from_numpy((8 * x + rng.integers(-4, 4, x.shape)).astype(np.int32)).to(DEV)
    mx = torch.full((1,), 8 * ((1 << xb) - 1), dtype=torch.int32, device=DEV)
    shift = torch.full((1,), -1, dtype=torch.int32, device=DEV)
    try:
        for spaced in (0, 1):
            samd.conv2d_use_plan(shape, xf, wf, dict(
                lane_bits=lane_bits, lanes=lanes, x_offset=xoff, shared_rows=int(shape[7] == 1 and KH > 1),
                rows_per_thread=1, rows_per_block=1, mblock=8, split_waves=1, layout_spaced=spaced))
        plan = samd.conv2d_spaced_plan(shape, xf, wf)
        assert plan.lanes == lanes and plan.x_offset == xoff == samd.conv2d_plan(shape, xf, wf).x_offset
        # above what the one-chain writer takes
        assert N * C * (H + 2 * shape[9]) * plan.tap_words * plan.words_per_row > 16384
        xp = samd.pack(xv, xb, False)
        wss, ws = samd.conv2d_spaced_prepare(wp, wf, shape, xf), samd.conv2d_prepare(wp, wf, shape, xf)
        words = {"spaced bytes": samd.conv2d_spaced_pack(xv, xf, wf, shape),
                 "spaced packed": samd.conv2d_spaced_from_packed(xp, xf, wf, shape),
                 "spaced accumulators": samd.relu_requant_spaced(acc, mx, xb, wf, shape, dev_shift=shift)}
        got = {name: samd.conv2d_spaced(v, xf, wf, shape, wss) for name, v in words.items()}
        got["packed"] = samd.conv2d_prepared(xp, xf, wf, shape, ws)
        samd.relu_requant_stage(acc, mx, xb, wf, shape, ws)
        got["accumulators"] = samd.conv2d_accumulate(xf, wf, shape, ws)
    finally:
        samd.conv2d_untune(shape, xf, wf)
    assert int(shift.item()) == 3
    for name, y in got.items():
        np.testing.assert_array_equal(y.cpu().numpy(), want, err_msg=name)


def test_bytes_are_read_as_fast_as_packed_rows():
    # 8-bit values take the same room either way, and give the same words; read one byte at a time
    # they took 1.3 times as long
    shape, xf, wf = (8, 61, 108, 402, 51, 5, 5, 4, 4, 0, 0), samd.Fmt(8, True), samd.Fmt(8, True)
    x = torch.randint(-128, 128, shape[:4], device=DEV, dtype=torch.int16).to(torch.int8)
    xp, out = samd.pack(x, 8, True), samd.conv2d_spaced_pack(x, xf, wf, shape)

    def microseconds(call):
        start, end, times = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True), []
        for _ in range(16):
            start.record()
            for _ in range(30):
                call()
            end.record()
            end.synchronize()
            times.append(start.elapsed_time(end) / 30 * 1e3)
        return min(times[4:])

    packed = microseconds(lambda: samd.conv2d_spaced_from_packed(xp, xf, wf, shape, out=out))
    plain = microseconds(lambda: samd.conv2d_spaced_pack(x, xf, wf, shape, out=out))
    print(f"from bytes {plain:.1f} us, from packed rows {packed:.1f} us")
    assert plain < 1.15 * packed, (plain, packed)


@pytest.mark.parametrize("width", [1, 2, 3, 4, 5, 6, 7, 8, 11])
@pytest.mark.parametrize("bits,signed", [(8, True), (5, False)])
def test_short_rows_of_bytes(width, bits, signed):
    # rows narrower than the four bytes of one read, and rows whose last read begins inside them,
    # each row at another alignment; the last row ends the buffer
    shape, xf, wf = (31, 67, 9, width, 16, 3, 1, 1, 1, 1, 0), samd.Fmt(bits, signed), samd.Fmt(4, True)
    lo, hi = wl.value_range(bits, signed)
    x = torch.randint(lo, hi + 1, shape[:4], device=DEV, dtype=torch.int16).to(torch.int8 if signed else torch.uint8)
    plan = samd.conv2d_spaced_plan(shape, xf, wf)
    words = 31 * 67 * 11 * plan.words_per_row * plan.tap_words   # a spare channel follows, never written
    assert words > 16384
    got = samd.conv2d_spaced_pack(x, xf, wf, shape)
    want = samd.conv2d_spaced_from_packed(samd.pack(x, bits, signed), xf, wf, shape)
    assert torch.equal(got[:words], want[:words])
