"""Work items over the live rays of a call against items over all its rays, for
every kernel family: rays of one scene, in one call (2^15 rays and more: live
rays) and as two scenes that are the same one (several scenes: all rays).
Images bit for bit, gradients and losses up to the order of their FP32 sums;
and the same call on reused hits, whose live-ray arrays are made from the
counts."""

import numpy as np
import pytest

from synth.configs import lf_inputs, tiny_workload

pytestmark = pytest.mark.gpu

MODELS = {  # decoder, hits per ray, view direction
    "8": ((8, 32, 32, 4), 6, False),
    "8vd": ((11, 32, 32, 4), 16, True),
    "16": ((16, 64, 64, 64, 4), 7, False),
    "32": ((32, 64, 64, 64, 4), 8, False),
    "32vd": ((35, 64, 64, 64, 4), 16, True),
    "lf": ((8, 32, 32, 4), 6, False),
}


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("model", list(MODELS))
@pytest.mark.parametrize("n", [1 << 15, 70001])
def test_plans_agree(gpu_lib, n, model, precision):
    import torch
    svlf = gpu_lib
    widths, K, vd = MODELS[model]
    w = tiny_workload(5, 5, widths[0] - (3 if vd else 0), widths, K)
    sc = w.scene()
    rng = np.random.default_rng(n)
    o = rng.normal(size=(n, 3))
    o = 3.0 * o / np.linalg.norm(o, axis=1, keepdims=True)
    d = rng.uniform(-0.5, 0.5, (n, 3)) - o
    d[rng.random(n) < 0.7] *= -1.0                   # most rays miss
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    t = rng.uniform(0, 1, (n, 4))
    o, d, rgb_t, dep_t = [torch.from_numpy(np.ascontiguousarray(x, np.float32)).cuda()
                          for x in (o, d, t[:, :3], 3 * t[:, 3])]
    if model == "lf":
        F, p = lf_inputs(7, sc.n_vertices)
        scene = svlf.DeviceScene.lf_from_host(sc.leaf_ijk, sc.depth, F)
    else:
        p = w.params()
        p[-1] = 0.6
        scene = svlf.DeviceScene.from_host(sc.leaf_ijk, sc.depth, w.features())
    params = torch.from_numpy(p).cuda()
    dec = () if model == "lf" else (w.widths,)
    ws = svlf.Workspace()

    def call(counts, flags):
        opts = svlf.make_opts(K, "voxel", precision, flags | (svlf.FLAG_VIEWDIR if vd else 0))
        a = ([scene] * len(counts), counts, params) + dec + (opts, o, d)
        images = (svlf.lf_render if model == "lf" else svlf.render)(*a, workspace=ws)
        gF, gp, loss = torch.zeros_like(scene.features), torch.zeros_like(params), torch.zeros(1, device="cuda")
        rgb, dep = torch.full((n, 3), -1.0, device="cuda"), torch.full((n,), -1.0, device="cuda")
        (svlf.lf_train_step if model == "lf" else svlf.train_step)(
            *a, rgb_t, dep_t, 0.1, 1.0 / n, [gF] * len(counts), gp, out_rgb=rgb, out_depth=dep, loss_out=loss,
            workspace=ws)
        return list(images) + [rgb, dep, gF, gp, loss]

    live = call([n], 0)
    reused = call([n], svlf.FLAG_REUSE_HITS)
    every = call([n // 3, n - n // 3], 0)
    hit = (live[2] > 0).float().mean()
    assert 0.05 < hit < 0.4
    for other in (reused, every):
        for i, (x, y) in enumerate(zip(live, other)):
            if i < 5:
                assert torch.equal(x, y), i
            else:
                assert (x - y).abs().max() <= 1e-4 * y.abs().max(), i
