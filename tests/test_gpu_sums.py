"""Accuracy of the long FP32 sums behind the decoder gradients.  n identical rays
through one voxel give n identical contributions, so every bias gradient is n
times that of one ray (a single contribution, exact).  Adding equal terms to a
running sum errs the same way at every step, so a sum that runs over a block's
whole share, or over all blocks, is far off one that adds in groups.

Tolerance: all terms of an entry are equal, so each addition on the longest path
to the result errs by at most 2^-24 of its sum.  The path: 7 additions in a
16-hit step's 8 hits of a lane, the window's steps - 1, the block's windows - 1,
1 for the lane groups, 3 for the waves; then the blocks' partial sums, of which a
quarter's 16 accumulators take every 16th: ceil(rows / 64) - 1, 4 to combine
them, 3 for the quarters."""

import math

import numpy as np
import pytest

from synth.configs import lf_inputs, lf_widths, xavier_params

pytestmark = pytest.mark.gpu


def _bias_entries(widths, at=0):
    out = []
    for i, o in zip(widths[:-1], widths[1:]):
        out += range(at + i * o, at + i * o + o)
        at += i * o + o
    return out, at


# model, rays, hits of a window, most windows of a block per 256 blocks
# (deterministic: items stay on their blocks; light field: the last two of 8
# rounds of items go to whichever block is free, so up to four times a block's
# share), most rows of partials
CASES = {
    "16": ((16, 64, 64, 64, 4), 1 << 19, 128, 16, 512),
    "8": ((8, 32, 32, 4), 8192, 16, 1, 512),
    "lf": (None, 1 << 18, 64, 4 * 16, 256),
}


@pytest.mark.parametrize("model", list(CASES))
def test_equal_contributions(gpu_lib, model):
    import torch
    svlf = gpu_lib
    widths, n, win, windows, rows = CASES[model]
    leaf = np.array([[3, 5, 2]], np.int32)
    lo = -1 + leaf[0] * 0.25
    o = np.array([-2.0, -1.7, -2.3], np.float32)
    d = (lo + [0.11, 0.13, 0.09] - o).astype(np.float32)
    o, d = (torch.from_numpy(np.tile(x, (n, 1))).cuda() for x in (o, d))
    rng = np.random.default_rng(5)
    if model == "lf":
        F, p = lf_inputs(7, 8)
        wt, wc = lf_widths()
        bt, at = _bias_entries(wt)
        entries = bt + _bias_entries(wc, at)[0]
        scene = svlf.DeviceScene.lf_from_host(leaf, 3, F)
    else:
        p = xavier_params(rng, widths)
        p[-1] = 0.7
        entries = _bias_entries(widths)[0]
        scene = svlf.DeviceScene.from_host(leaf, 3, rng.normal(0, 0.3, (8, widths[0])).astype(np.float32))
    params = torch.from_numpy(p.astype(np.float32)).cuda()
    opts = svlf.make_opts(1, "voxel", "fp32", 0 if model == "lf" else svlf.FLAG_DETERMINISTIC)

    def bias_gradients(m, scale):
        g_rgb = torch.tensor([0.9, -1.3, 0.6], device="cuda").mul(scale).repeat(m, 1)
        g_dep = torch.full((m,), 0.7 * scale, device="cuda")
        gF, gp = torch.zeros_like(scene.features), torch.zeros_like(params)
        a = ([scene], [m], params) + (() if model == "lf" else (widths,))
        (svlf.lf_render_backward if model == "lf" else svlf.render_backward)(
            *a, opts, o[:m], d[:m], g_rgb, g_dep, None, [gF], gp)
        return gp[entries].double().cpu().numpy()

    tol = (7 + math.ceil(win / 16) - 1 + windows - 1 + 1 + 3 + math.ceil(rows / 64) - 1 + 4 + 3) * 2.0 ** -24
    worst = 0.0
    for scale in (1.0, 1.3, 1.7, 1.9):      # other mantissas
        one = bias_gradients(1, scale)
        used = one != 0
        assert used.sum() > len(entries) / 4
        got = bias_gradients(n, scale)
        assert not got[~used].any()
        worst = max(worst, np.abs(got[used] / (n * one[used]) - 1).max())
    print(model, "error", worst * 2 ** 24, "of", tol * 2 ** 24, "x 2^-24")
    assert worst <= tol
