"""The planner's search on the CPU: a plan's first look-up prices only launches that may be
the cheapest, and finds the one that pricing every launch finds."""
import ctypes
import glob
import os
import random
import re
import statistics
import time

import pytest

import paper_1809_10572_amd as samd
import test_gpu_multiply_forms as multiply


def _layers(count, seed):
    rng = random.Random(seed)
    for _ in range(count):
        k, s = rng.choice((1, 3, 3, 5, 7, 11)), rng.choice((1, 1, 2, 4))
        shape = (rng.randint(1, 8), rng.randint(3, 200), rng.randint(11, 120), rng.randint(11, 300), rng.randint(8, 200),
                 k, k, s, s, k // 2, k // 2)
        yield shape, samd.Fmt(rng.randint(1, 8), rng.random() < 0.5), samd.Fmt(rng.randint(1, 6), rng.random() < 0.8)


def test_the_bounded_search_finds_the_cheapest_plan():
    planned = 0
    for shape, xf, wf in _layers(60, 3):
        try:
            plan = samd.conv2d_plan(shape, xf, wf)
        except samd.SamdError:
            continue
        first, *rest = samd.conv2d_candidates(shape, xf, wf, 4)   # prices every launch
        assert bytes(plan) == bytes(first), (shape, xf, wf)
        assert all(plan.model_cost <= c.model_cost for c in rest)
        planned += 1
    assert planned > 40


def _seconds(call, *args):
    t = time.perf_counter()
    call(*args)
    return time.perf_counter() - t


@pytest.mark.parametrize("shape,bits", [((8, 128, 56, 56, 128, 3, 3, 1, 1, 1, 1), 4),
                                        ((4, 96, 40, 40, 64, 5, 5, 1, 1, 2, 2), 4)])
def test_a_first_plan_prices_few_launches(shape, bits):
    # against a listing, which prices every launch of the layer: 3 to 5 % of its time (15 to 40 %
    # when every launch within reach of the multiply-adds' bound was priced in full)
    xf, wf = samd.Fmt(bits, False), samd.Fmt(bits, True)
    shares = []
    for i in range(15):
        new = shape[:4] + (shape[4] + i,) + shape[5:]     # a layer not planned yet
        shares.append(_seconds(samd.conv2d_plan, new, xf, wf) / _seconds(samd.conv2d_candidates, new, xf, wf, 1))
    assert statistics.median(shares) < 0.11, shares


def test_a_layer_too_large_for_the_scratch_array_is_searched_once():
    # no plan of this layer fits the array; the refusal, which comes before any HIP call, is
    # remembered
    shape, xf, wf = (16, 512, 57, 57, 384, 3, 3, 1, 1, 1, 1), samd.Fmt(8, False), samd.Fmt(8, True)
    d = samd.Conv2dDesc.of(shape)
    call = lambda: samd.lib().samd_conv2d_noalloc(256, xf, 256, wf, ctypes.byref(d), 256, None)
    refused = lambda: _seconds(lambda: statuses.append(call()))
    statuses = []
    first, later = refused(), min(refused() for _ in range(5))
    assert set(statuses) == {samd.SAMD_ENOSPC} and "scratch array" in samd.lib().samd_last_error().decode()
    assert later < 0.2 * first, (first, later)


def test_the_multiply_tests_name_every_compiled_form():
    # the layers of tests/test_gpu_multiply_forms.py against the instances in the sources
    sources = os.path.join(os.path.dirname(samd.LIB_PATH), "csrc", "conv2d_multiply_*.hip")
    compiled = set()
    for path in glob.glob(sources):
        for rh, kht, two in re.findall(r"launch_multiply_shape<(\d), (\d), (\d)>", open(path).read()):
            compiled |= {(int(kht), int(rh), int(two), sg, seg) for sg in (0, 1) for seg in (0, 1)}
    named = set()
    for shape, xb, xs, wb, ws, forms in multiply.FORMS:
        segments = samd.conv2d_plan(shape, samd.Fmt(xb, xs), samd.Fmt(wb, ws)).col_segments > 1
        named |= {f + (int(xs or ws), int(segments)) for f in forms}
    assert named == compiled and len(compiled) == 104


@pytest.mark.parametrize("case", [0, 6, 12])
def test_named_forms_have_plans(case):
    assert None not in multiply.form_plans(case).values()


# (shape, x format, w bits): the multiply's us with the plans of before, one value per word in
# segments of 64 columns or words of 11 lanes, and with the present ones
WIDE_ROWS = [((2, 2, 157, 262, 252, 1, 1, 1, 1, 0, 0), (8, False), 8),       # 61.8, 37.8
             ((6, 1, 221, 166, 202, 2, 2, 1, 1, 1, 0), (8, False), 4),       # 112.4, 80.0
             ((15, 8, 44, 152, 371, 1, 1, 1, 1, 0, 0), (8, False), 7),       # 108.2, 82.0
             ((13, 2, 129, 299, 259, 1, 7, 2, 2, 0, 3), (1, False), 1)]      # 57.7, 41.2


@pytest.mark.parametrize("shape,xfmt,wbits", WIDE_ROWS)
def test_layers_of_few_channels_and_wide_rows_fill_their_words(shape, xfmt, wbits):
    plan = samd.conv2d_plan(shape, samd.Fmt(*xfmt), samd.Fmt(wbits, True))
    assert plan.lanes >= 2 and (plan.col_segments == 1 or plan.segment_columns > 64)
    assert plan.out_lanes <= 8
