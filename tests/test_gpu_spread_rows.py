"""The operand-word writer, from its three sources (packed rows, 8-bit values, int32
accumulators), checked through the convolution against the oracle: layers large enough for
its workgroups of rows, strided ones, words of more fields than an LDS word holds, rows
that end inside a word, and rows too long for a workgroup's LDS."""
import numpy as np
import pytest
import torch

import paper_1809_10572_amd as samd
import samd_workloads as wl
from oracle import reference as ref

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    ((2, 9, 31, 61, 4, 3, 3, 1, 1, 1, 1), 1, 1),      # four values per word
    ((2, 9, 31, 62, 4, 3, 3, 1, 1, 1, 1), 3, 3),
    ((2, 9, 30, 59, 4, 3, 3, 1, 1, 1, 1), 5, 5),      # packed words with unused bits
    ((2, 9, 30, 57, 4, 3, 3, 1, 1, 1, 1), 8, 8),
    ((1, 6, 41, 75, 4, 5, 5, 1, 1, 2, 2), 7, 7),      # several kernel words per row
    ((2, 5, 41, 83, 4, 3, 3, 2, 2, 1, 1), 4, 4),      # two stride phases
    ((2, 3, 61, 93, 4, 7, 11, 4, 4, 2, 5), 2, 2),
    ((3, 25, 40, 53, 4, 1, 1, 1, 1, 0, 0), 2, 3),     # 1x1: many values per word
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
