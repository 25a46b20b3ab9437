"""How a call's rays are divided into work items must not show in its results:
the same rays rendered in calls of different sizes (item sizes from the
smallest up, one to several rounds of the grid, ragged ends, one and two
scenes) give the same bits, and gradients that agree up to the order of their
FP32 sums."""

import numpy as np
import pytest

from synth.configs import lf_inputs, tiny_workload

pytestmark = pytest.mark.gpu

N_ALL = 70001
SIZES = (1, 15, 17, 4095, 4097, 12289, 65537)


MODELS = {  # decoder, hits per ray, view direction
    "8": ((8, 32, 32, 4), 6, False),
    "8vd": ((11, 32, 32, 4), 16, True),
    "16": ((16, 64, 64, 64, 4), 7, False),
    "32": ((32, 64, 64, 64, 4), 8, False),
    "32vd": ((35, 64, 64, 64, 4), 16, True),
    "lf": ((8, 32, 32, 4), 6, False),
}


def _inputs(widths, K, viewdir):
    import torch
    w = tiny_workload(5, 5, widths[0] - (3 if viewdir else 0), widths, K)
    rng = np.random.default_rng(11)
    o = rng.normal(size=(N_ALL, 3))
    o = 3.0 * o / np.linalg.norm(o, axis=1, keepdims=True)
    d = rng.uniform(-0.6, 0.6, (N_ALL, 3)) - o
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    t = rng.uniform(0, 1, (N_ALL, 4))
    return w, [torch.from_numpy(np.ascontiguousarray(x, np.float32)).cuda() for x in (o, d, t[:, :3], 3 * t[:, 3])]


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("model", list(MODELS))
def test_item_sizes(gpu_lib, model, precision):
    import torch
    svlf = gpu_lib
    w, (o, d, rgb_t, dep_t) = _inputs(*MODELS[model])
    sc = w.scene()
    if model == "lf":
        F, p = lf_inputs(7, sc.n_vertices)
        scene = svlf.DeviceScene.lf_from_host(sc.leaf_ijk, sc.depth, F)
    else:
        p = w.params()
        p[-1] = 0.6
        scene = svlf.DeviceScene.from_host(sc.leaf_ijk, sc.depth, w.features())
    params = torch.from_numpy(p).cuda()
    opts = svlf.make_opts(w.K, "voxel", precision, svlf.FLAG_VIEWDIR if MODELS[model][2] else 0)

    def call(lo, counts, grads=True):
        n = sum(counts)
        sl = slice(lo, lo + n)
        scenes = [scene] * len(counts)
        a = (scenes, counts, params) + (() if model == "lf" else (w.widths,)) + (opts, o[sl], d[sl])
        out = (svlf.lf_render if model == "lf" else svlf.render)(*a)
        if not grads:
            return out, None, None
        gF, gp = torch.zeros_like(scene.features), torch.zeros_like(params)
        step = svlf.lf_train_step if model == "lf" else svlf.train_step
        step(*a, rgb_t[sl].contiguous(), dep_t[sl], 0.1, 1.0 / N_ALL, [gF] * len(counts), gp)
        return out, gF, gp

    whole, gF, gp = call(0, [N_ALL])
    assert (whole[2] > 0).float().mean() > 0.2
    for n in SIZES:
        for counts in ([n], [n // 3, n - n // 3]):
            lo = (N_ALL - n) // 2
            got, _, _ = call(lo, counts, grads=False)
            for x, y in zip(got, whole):
                assert torch.equal(x, y[lo:lo + n]), (model, precision, counts)
    # gradients: the whole call against calls over its parts
    parts = [(0, [4095]), (4095, [40000, 17]), (44112, [N_ALL - 44112])]
    sF, sp = torch.zeros_like(gF), torch.zeros_like(gp)
    for lo, counts in parts:
        _, f, q = call(lo, counts)
        sF += f
        sp += q
    assert (sF - gF).abs().max() <= 1e-5 * gF.abs().max()
    assert (sp - gp).abs().max() <= 1e-4 * gp.abs().max()
