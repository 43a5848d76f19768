"""Every form of the multiply kernel - rows shared by 3- and 5-row kernels, the general
path, lanes decoded every period or widened in registers (two-level lanes, with the top
lane inside its word and apart), signed and unsigned results, column segments - against the
oracle, bit-exact, at shapes where each begins or ends: odd channel counts and slices,
periods of one batch or less, rows past the image, filters past M, and operands that drive
every lane to its bound; and the write-out of short output rows."""
import itertools

import numpy as np
import pytest
import torch

import paper_1809_10572_amd as samd
import samd_workloads as wl
from oracle import reference as ref

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (shape, x bits, x signed, w bits): 13-bit lanes of 4-bit operands hold 7 channels (both
# layouts of the top lane), 9-bit lanes of 2-bit operands 7 or 4, 22-bit lanes of 8-bit 10;
# 1x1 and strided kernels take the general path; 300 columns take column segments
CASES = [
    ((1, 41, 7, 19, 9, 3, 3, 1, 1, 1, 1), 4, False, 4),
    ((2, 40, 6, 11, 17, 3, 3, 1, 1, 1, 1), 2, True, 2),
    ((1, 37, 5, 13, 8, 3, 3, 1, 1, 1, 1), 8, True, 8),
    ((1, 33, 4, 9, 8, 3, 3, 1, 1, 0, 1), 5, False, 5),
    ((1, 23, 9, 14, 10, 5, 5, 1, 1, 2, 2), 4, False, 4),
    ((1, 19, 6, 10, 8, 5, 3, 1, 1, 2, 1), 8, False, 8),
    ((1, 66, 3, 17, 9, 1, 1, 1, 1, 0, 0), 4, True, 4),
    ((1, 21, 11, 12, 8, 3, 3, 2, 2, 1, 1), 6, True, 4),
    ((1, 9, 13, 23, 8, 11, 11, 4, 4, 2, 2), 4, False, 4),
    ((1, 30, 3, 300, 8, 3, 3, 1, 1, 1, 1), 4, False, 4),
    ((1, 20, 4, 9, 8, 3, 3, 1, 1, 1, 1), 3, False, 3),
]


def _operands(kind, shape, xb, xs, wb, ws=True):
    N, C, H, W, M, KH, KW = shape[:7]
    xlo, xhi = wl.value_range(xb, xs)
    wlo, whi = wl.value_range(wb, ws)
    if kind == "mixed":
        rng = np.random.default_rng(sum(shape) + xb)
        return wl.half_extremes(rng, (N, C, H, W), xb, xs), wl.half_extremes(rng, (M, C, KH, KW), wb, ws)
    x = xlo if kind == "low" else xhi       # every product at one extreme
    return np.full((N, C, H, W), x), np.full((M, C, KH, KW), wlo if kind != "high" else whi)


def _variants(cands):
    """The candidates, and their lane geometries under launch shapes the list leaves out:
    several rows per lane, one or more channel slices, shared rows or not."""
    keys = [samd.plan_key(p) for p in cands]
    seen = set()
    for k in list(keys):
        geometry = (k["lane_bits"], k["lanes"], k["x_offset"])
        if geometry in seen or len(seen) >= 6:
            continue
        seen.add(geometry)
        keys += [dict(k, shared_rows=shared, rows_per_thread=rows, rows_per_block=rows * groups, mblock=m, split_waves=ks)
                 for shared in (0, 1) for rows in (1, 2, 3, 4) for groups in (1, 2) for m, ks in ((8, 1), (16, 2), (8, 4))]
    return keys


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("kind", ["mixed", "low", "high", "opposite"])
def test_every_candidate_matches_the_oracle(case, kind):
    shape, xb, xs, wb = CASES[case]
    x, w = _operands(kind, shape, xb, xs, wb)
    xf, wf = samd.Fmt(xb, xs), samd.Fmt(wb, True)
    want = ref.conv2d(x.astype(np.int32), w.astype(np.int32), shape)
    dev = lambda a, s: torch.from_numpy(a.astype(np.int8 if s else np.uint8)).to(DEV)
    xp, wp = samd.pack(dev(x, xs), xb, xs), samd.pack(dev(w, True), wb, True)
    cands = samd.conv2d_candidates(shape, xf, wf, samd.MAX_CANDIDATES)
    keys, ran = _variants(cands), 0
    # the mixed operands go through every variant, the others through every fourth
    try:
        for p in keys if kind == "mixed" else keys[::4]:
            try:
                samd.conv2d_use_plan(shape, xf, wf, p)
            except samd.SamdError:
                if not isinstance(p, dict):
                    raise           # a listed plan
                continue            # a launch shape this layer does not have
            ran += 1
            y = samd.conv2d(xp, xf, wp, wf, shape)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(y.cpu().numpy(), want, err_msg=str(p))
    finally:
        samd.conv2d_untune(shape, xf, wf)
    assert ran >= len(cands) // 4


# Layers that between them run every instance of the kernel: (shape, x bits, x signed, w bits,
# w signed) and the forms of each, as (kernel_rows, rows per lane, widened) of a plan.
# Result signedness and column segments (the rows of 261 columns) are the layer's own.
ROWS3 = set(itertools.product((1, 3), (1, 2), (0, 1, 2))) | {(3, 3, 0), (3, 4, 0)}
ROWS5 = set(itertools.product((0, 5), (1, 2), (0, 1, 2)))
FORMS = [
    ((1, 47, 7, 19, 9, 3, 3, 1, 1, 1, 1), 4, False, 4, True, ROWS3),
    ((1, 47, 7, 19, 9, 3, 3, 1, 1, 1, 1), 8, False, 8, False, ROWS3),
    ((1, 47, 7, 261, 9, 3, 3, 1, 1, 1, 1), 8, False, 8, False, ROWS3),
    ((1, 97, 5, 261, 9, 3, 3, 1, 1, 1, 1), 8, True, 8, True, ROWS3),
    ((1, 47, 7, 19, 9, 5, 5, 1, 1, 2, 2), 3, False, 3, False, ROWS5),
    ((1, 47, 7, 19, 9, 5, 5, 1, 1, 2, 2), 4, False, 4, True, {f for f in ROWS5 if f[2] < 2}),
    ((1, 47, 7, 19, 9, 5, 5, 1, 1, 2, 2), 8, True, 8, True, {(5, 1, 2), (5, 2, 2)}),
    ((1, 47, 7, 19, 9, 7, 7, 1, 1, 3, 3), 8, True, 8, True, {(0, 1, 2), (0, 2, 2)}),
    ((1, 47, 7, 261, 9, 5, 5, 1, 1, 2, 2), 4, False, 4, True, {f for f in ROWS5 if f[2] < 2}),
    ((1, 47, 7, 261, 9, 5, 5, 1, 1, 2, 2), 8, True, 8, True, {(5, 1, 2), (5, 2, 2)}),
    ((1, 47, 7, 261, 9, 7, 7, 1, 1, 3, 3), 8, True, 8, True, {(0, 1, 2), (0, 2, 2)}),
    ((1, 47, 7, 261, 9, 5, 5, 1, 1, 2, 2), 4, False, 4, False,
     {f for f in ROWS5 if f[2] < 2} - {(0, 2, 0)} | {(5, 1, 2)}),
    ((1, 47, 7, 261, 9, 5, 5, 1, 1, 2, 2), 8, False, 8, False, {(5, 2, 2)}),
    ((1, 47, 7, 261, 9, 7, 7, 1, 1, 3, 3), 7, False, 7, False, {(0, 1, 2), (0, 2, 0), (0, 2, 2)}),
]


def form_plans(case):
    """Plans of a layer of FORMS, the first found of each of its forms."""
    shape, xb, xs, wb, ws, forms = FORMS[case]
    xf, wf = samd.Fmt(xb, xs), samd.Fmt(wb, ws)
    found = {}
    try:
        for k in map(lambda p: p if isinstance(p, dict) else samd.plan_key(p),
                     _variants(samd.conv2d_candidates(shape, xf, wf, samd.MAX_CANDIDATES))):
            try:
                samd.conv2d_use_plan(shape, xf, wf, k)
            except samd.SamdError:
                continue
            f = samd.conv2d_form(shape, xf, wf)
            assert f.result_signed == (xs or ws)
            found.setdefault((f.kernel_rows, k["rows_per_thread"], f.widened), k)
            if forms <= set(found):
                break
    finally:
        samd.conv2d_untune(shape, xf, wf)
    return {f: found.get(f) for f in sorted(forms)}


@pytest.mark.parametrize("case", range(len(FORMS)))
def test_every_form_matches_the_oracle(case):
    shape, xb, xs, wb, ws, _ = FORMS[case]
    xf, wf = samd.Fmt(xb, xs), samd.Fmt(wb, ws)
    plans = form_plans(case)
    assert None not in plans.values(), plans
    dev = lambda a, s: torch.from_numpy(a.astype(np.int8 if s else np.uint8)).to(DEV)
    runs = []
    for kind in ("mixed", "low", "high", "opposite"):
        x, w = _operands(kind, shape, xb, xs, wb, ws)
        runs.append((kind, samd.pack(dev(x, xs), xb, xs), samd.pack(dev(w, ws), wb, ws), ref.conv2d(x, w, shape)))
    try:
        for form, key in plans.items():
            samd.conv2d_use_plan(shape, xf, wf, key)
            for kind, xp, wp, want in runs:
                y = samd.conv2d(xp, xf, wp, wf, shape)
                np.testing.assert_array_equal(y.cpu().numpy(), want, err_msg=f"{form} {kind} {key}")
    finally:
        samd.conv2d_untune(shape, xf, wf)


# default plans whose lanes hold two, or one, product: (shape, formats, steps)
FEW_STEPS = [
    ((1, 7, 25, 35, 138, 1, 1, 1, 1, 0, 0), (2, False), (2, True), 2),
    ((2, 2, 33, 22, 155, 1, 1, 1, 1, 0, 0), (4, True), (2, True), 1),
    ((2, 7, 33, 78, 168, 1, 1, 1, 1, 0, 0), (2, True), (7, False), 1),
]


@pytest.mark.parametrize("shape,xfmt,wfmt,steps", FEW_STEPS)
def test_default_plans_of_few_steps_per_decode(shape, xfmt, wfmt, steps):
    xf, wf = samd.Fmt(*xfmt), samd.Fmt(*wfmt)
    assert samd.conv2d_form(shape, xf, wf).period == -steps
    x, w = _operands("mixed", shape, *xfmt, *wfmt)
    want = ref.conv2d(x, w, shape)
    dev = lambda a, s: torch.from_numpy(a.astype(np.int8 if s else np.uint8)).to(DEV)
    y = samd.conv2d(samd.pack(dev(x, xfmt[1]), *xfmt), xf, samd.pack(dev(w, wfmt[1]), *wfmt), wf, shape)
    np.testing.assert_array_equal(y.cpu().numpy(), want)


def test_few_steps_per_decode_on_the_general_path():
    # one-bit 1x1 layers list lane geometries that hold fewer products than one batch of
    # three steps (2-bit lanes, one product) or one batch (3-bit lanes); every listed one of
    # the narrowest lanes is run
    shape, xf, wf = (1, 13, 3, 20, 8, 1, 1, 1, 1, 0, 0), samd.Fmt(1, False), samd.Fmt(1, True)
    rng = np.random.default_rng(5)
    x = wl.uniform(rng, (1, 13, 3, 20), 1, False)
    w = wl.uniform(rng, (8, 13, 1, 1), 1, True)
    want = ref.conv2d(x, w, shape)
    xp = samd.pack(torch.from_numpy(x.astype(np.uint8)).to(DEV), 1, False)
    wp = samd.pack(torch.from_numpy(w.astype(np.int8)).to(DEV), 1, True)
    seen = set()
    for bits in (2, 3, 4, 5):
        for lanes in range(2, 9):
            for rows in (1, 2, 3):
                for ks in (1, 2):
                    key = dict(lane_bits=bits, lanes=lanes, x_offset=0, shared_rows=0, rows_per_thread=1,
                               rows_per_block=rows, mblock=8, split_waves=ks, layout_spaced=0, spacer_msb=0)
                    try:
                        samd.conv2d_use_plan(shape, xf, wf, key)
                    except samd.SamdError:
                        continue
                    seen.add(samd.conv2d_form(shape, xf, wf).period)
                    y = samd.conv2d(xp, xf, wp, wf, shape)
                    torch.cuda.synchronize()
                    samd.conv2d_untune(shape, xf, wf)
                    np.testing.assert_array_equal(y.cpu().numpy(), want, err_msg=str(key))
    assert {-1, 1} <= seen


def test_a_layer_whose_fastest_plan_passes_the_scratch_array_still_runs_there():
    # 5-bit operands, signed 1-bit weights, 7x7: the model's choice needs 75 MB of workspace,
    # other plans of the layer under 64 MiB
    shape, xf, wf = (1, 692, 36, 205, 707, 7, 7, 1, 1, 3, 3), samd.Fmt(5, False), samd.Fmt(1, True)
    assert samd.conv2d_workspace(shape, xf, wf) > samd.NOALLOC_SCRATCH_BYTES
    g = torch.Generator(device=DEV).manual_seed(5)
    x = torch.randint(0, 32, (1, 692, 36, 205), generator=g, device=DEV, dtype=torch.uint8)
    w = torch.randint(-1, 1, (707, 692, 7, 7), generator=g, device=DEV, dtype=torch.int8)
    xp, wp = samd.pack(x, 5, False), samd.pack(w, 1, True)
    want = samd.conv2d(xp, xf, wp, wf, shape)
    out = torch.empty_like(want)
    for _ in range(2):
        samd.conv2d_noalloc(xp, xf, wp, wf, shape, out=out.fill_(-1))
        assert torch.equal(out, want)


@pytest.mark.parametrize("width", [1, 7, 8, 9, 16, 17, 32, 33])
@pytest.mark.parametrize("bits,signed", [(8, False), (3, True)])
def test_rows_written_several_at_a_time(width, bits, signed):
    # 8, 4 or 2 output rows leave a wave at once up to 8, 16 and 32 columns; 13 filters and 11
    # rows leave channel blocks and lanes part empty
    shape, xf, wf = (3, 6, 11, width, 13, 3, 3, 1, 1, 1, 1), samd.Fmt(bits, signed), samd.Fmt(bits, True)
    x, w = _operands("mixed", shape, bits, signed, bits)
    want = torch.from_numpy(np.asarray(ref.conv2d(x, w, shape))).to(DEV, torch.int32)
    xt = torch.from_numpy(x.astype(np.int8 if signed else np.uint8)).to(DEV)
    wp = samd.pack(torch.from_numpy(w.astype(np.int8)).to(DEV), bits, True)
    assert torch.equal(samd.conv2d(samd.pack(xt, bits, signed), xf, wp, wf, shape), want)
    ws = samd.conv2d_spaced_prepare(wp, wf, shape, xf)
    assert torch.equal(samd.conv2d_spaced(samd.conv2d_spaced_pack(xt, xf, wf, shape), xf, wf, shape, ws), want)


@pytest.mark.parametrize("spaced", [False, True])
@pytest.mark.parametrize("width", [1, 7, 8, 9, 16, 17, 32, 33, 63, 64, 65])
@pytest.mark.parametrize("bits,signed,lane_bits,rows", [(8, False, 21, 3), (3, True, 11, 4)])
def test_write_out_of_full_tiles(bits, signed, lane_bits, rows, width, spaced):
    # tiles of 3 or 4 rows of 11, the last part empty, four channel blocks of 32 filters, the last
    # part empty, and more 16-wave workgroups per XCD than its 32 compute units hold (2 each), so
    # that a tile is cleared for the next item; 8-bit layers recentred, with one correction per
    # filter (packed) or a table of them (spaced).  Rows of 65 outputs take the other copy.
    shape, xf, wf = (48, 8, 11, width, 125, 3, 3, 1, 1, 1, 1), samd.Fmt(bits, signed), samd.Fmt(bits, True)
    x, w = _operands("mixed", shape, bits, signed, bits)
    want = torch.from_numpy(np.asarray(ref.conv2d(x, w, shape))).to(DEV, torch.int32)
    xt = torch.from_numpy(x.astype(np.int8 if signed else np.uint8)).to(DEV)
    wp = samd.pack(torch.from_numpy(w.astype(np.int8)).to(DEV), bits, True)
    key = dict(lane_bits=lane_bits, lanes=2, x_offset=0 if signed else 1 << (bits - 1), shared_rows=1,
               rows_per_thread=rows, rows_per_block=rows, mblock=32, split_waves=4, layout_spaced=int(spaced))
    try:
        samd.conv2d_use_plan(shape, xf, wf, key)
        plan = (samd.conv2d_spaced_plan if spaced else samd.conv2d_plan)(shape, xf, wf)
        assert (plan.rows_per_block, plan.mblock, plan.split_waves) == (rows, 32, 4)
        assert plan.col_segments == 1 and plan.x_offset == key["x_offset"]
        assert 48 * -(-11 // rows) // 8 * 4 > 2 * 32       # tiles of an XCD x channel blocks
        if spaced:
            ws = samd.conv2d_spaced_prepare(wp, wf, shape, xf)
            y = samd.conv2d_spaced(samd.conv2d_spaced_pack(xt, xf, wf, shape), xf, wf, shape, ws)
        else:
            y = samd.conv2d(samd.pack(xt, bits, signed), xf, wp, wf, shape)
    finally:
        samd.conv2d_untune(shape, xf, wf)
    assert torch.equal(y, want)


def _pinned(shape, xf, wf, key, x, w):
    """The layer's output under a pinned plan, and the plan."""
    spaced, signed, bits = bool(key["layout_spaced"]), bool(xf.is_signed), xf.bits
    xt = torch.from_numpy(x.astype(np.int8 if signed else np.uint8)).to(DEV)
    wp = samd.pack(torch.from_numpy(w.astype(np.int8)).to(DEV), wf.bits, True)
    try:
        samd.conv2d_use_plan(shape, xf, wf, key)
        if spaced:
            plan = samd.conv2d_spaced_plan(shape, xf, wf)
            ws = samd.conv2d_spaced_prepare(wp, wf, shape, xf)
            y = samd.conv2d_spaced(samd.conv2d_spaced_pack(xt, xf, wf, shape), xf, wf, shape, ws)
        else:
            plan = samd.conv2d_plan(shape, xf, wf)
            y = samd.conv2d(samd.pack(xt, bits, signed), xf, wp, wf, shape)
        torch.cuda.synchronize()
    finally:
        samd.conv2d_untune(shape, xf, wf)
    return y, plan


# (bits, signed, lane bits, lanes, widths): rows of one to three steps of 128 columns, each ending
# at, before and after a 64 and a 128; then segments, the last of them narrower, of more and of at
# most 64 columns
LONG_ROWS = [(8, False, 21, 2, (65, 126)), (8, False, 21, 2, (127, 187, 300)), (2, True, 9, 3, (127, 128, 129, 190)),
             (1, True, 6, 5, (191, 192, 193, 255, 256, 257, 318)), (1, True, 6, 5, (319, 400)), (1, True, 6, 1, (65, 150))]


@pytest.mark.parametrize("spaced", [False, True])
@pytest.mark.parametrize("bits,signed,lane_bits,lanes,width", [(*c[:4], w) for c in LONG_ROWS for w in c[4]])
def test_write_out_of_long_rows(bits, signed, lane_bits, lanes, width, spaced):
    # tiles of 3 rows of 11, the last part empty, 16 channel blocks, the last part empty, and more
    # workgroups per XCD than its 32 compute units hold (4 each by registers), so that a tile is
    # cleared for the next item; 8-bit layers recentred
    shape, xf, wf = (32, 4, 11, width, 125, 3, 3, 1, 1, 1, 1), samd.Fmt(bits, signed), samd.Fmt(bits, True)
    x, w = _operands("mixed", shape, bits, signed, bits)
    key = dict(lane_bits=lane_bits, lanes=lanes, x_offset=0 if signed else 1 << (bits - 1), shared_rows=1,
               rows_per_thread=3, rows_per_block=3, mblock=8, split_waves=4, layout_spaced=int(spaced), spacer_msb=0)
    y, plan = _pinned(shape, xf, wf, key, x, w)
    assert (plan.rows_per_block, plan.mblock, plan.x_offset) == (3, 8, key["x_offset"])
    assert (plan.col_segments > 1) == (width + 2 > 64 * lanes)
    assert plan.col_segments * 32 * 4 // 8 * 16 > 4 * 32       # tiles of an XCD x channel blocks
    np.testing.assert_array_equal(y.cpu().numpy(), ref.conv2d(x, w, shape))


def test_the_write_out_of_long_rows_keeps_up_with_a_fill():
    # one channel, 1x1: 276 MB of outputs and hardly a product.  1.9 times the time of a fill of the
    # same bytes; 2.9 when four rows at a time were addressed and tested one by one
    shape, xf, wf = (8, 1, 163, 117, 453, 1, 1, 1, 1, 0, 0), samd.Fmt(8, True), samd.Fmt(8, True)
    x = torch.randint(-128, 128, shape[:4], device=DEV, dtype=torch.int16).to(torch.int8)
    w = torch.randint(-128, 128, (453, 1, 1, 1), device=DEV, dtype=torch.int16).to(torch.int8)
    xp, wp = samd.pack(x, 8, True), samd.pack(w, 8, True)
    y = torch.empty((8, 453, 163, 117), dtype=torch.int32, device=DEV)

    def microseconds(call):
        start, end, times = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True), []
        for _ in range(12):
            start.record()
            for _ in range(10):
                call()
            end.record()
            end.synchronize()
            times.append(start.elapsed_time(end) * 100)
        return min(times[4:])

    key = dict(lane_bits=16, lanes=2, x_offset=0, shared_rows=0, rows_per_thread=2, rows_per_block=2, mblock=32,
               split_waves=1, layout_spaced=0, spacer_msb=0)
    try:
        samd.conv2d_use_plan(shape, xf, wf, key)
        ws = samd.conv2d_stage(xp, xf, wf, shape, samd.conv2d_prepare(wp, wf, shape, xf))
        layer = microseconds(lambda: samd.conv2d_accumulate(xf, wf, shape, ws, out=y))
    finally:
        samd.conv2d_untune(shape, xf, wf)
    fill = microseconds(lambda: y.fill_(1))
    print(f"layer {layer:.1f} us, fill {fill:.1f} us")
    assert layer < 2.5 * fill, (layer, fill)
