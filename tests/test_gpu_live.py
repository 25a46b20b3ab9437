"""Work items planned over the live rays (rays with hits) of a call against
items over all its rays: the same images bit for bit, and gradients and losses
that agree up to the order of their FP32 sums.  A call that reuses hits is
planned over all rays, so both plans run on the same hits.  Cases: ray counts
at the edges of the live plan and of a traversal block (64 rays) and a
thread's share of blocks; no, one, few and all rays live, and live rays in one
stretch only."""

import numpy as np
import pytest

from synth.configs import lf_inputs, tiny_workload

pytestmark = pytest.mark.gpu

N_MIN, N_MAX = 1 << 15, 1 << 22


def _live(pattern, n, rng):
    if pattern == "none":
        return np.zeros(n, bool)
    if pattern == "all":
        return np.ones(n, bool)
    if pattern == "fifth":
        return rng.random(n) < 0.2
    m = np.zeros(n, bool)
    if pattern == "last":
        m[-1] = True
    elif pattern == "stretch":
        m[n // 3:n // 3 + 3001] = True
    else:                                   # every ray of some blocks, none of others
        m[:] = (np.arange(n) // 64) % 5 == 2
    return m


CASES = [(N_MIN - 1, "fifth"), (N_MIN, "fifth"), (N_MIN, "none"), (N_MIN + 1, "last"), (N_MIN + 63, "all"),
         (40009, "stretch"), (65537, "blocks"), (262144 + 65, "fifth"), (262144 + 4097, "stretch"),
         (1 << 20, "blocks"), (N_MAX, "blocks"), (N_MAX, "last"), (N_MAX + 1, "fifth")]


@pytest.mark.parametrize("model", ["render", "lf"])
@pytest.mark.parametrize("n,pattern", CASES)
def test_live_plan(gpu_lib, model, n, pattern):
    import torch
    svlf = gpu_lib
    K = 5
    w = tiny_workload(5, 5, 8, (8, 32, 32, 4), K)
    sc = w.scene()
    rng = np.random.default_rng(n)
    live = _live(pattern, n, rng)
    o = rng.normal(size=(n, 3))
    o = 3.0 * o / np.linalg.norm(o, axis=1, keepdims=True)
    d = rng.uniform(-0.3, 0.3, (n, 3)) - o
    d[~live] *= -1.0
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
    widths = () if model == "lf" else (w.widths,)
    render = svlf.lf_render if model == "lf" else svlf.render
    step = svlf.lf_train_step if model == "lf" else svlf.train_step
    ws = svlf.Workspace()
    got = {}
    for name, flags in (("own", 0), ("reused", svlf.FLAG_REUSE_HITS)):
        a = ([scene], [n], params) + widths + (svlf.make_opts(K, "voxel", "fp32", flags), o, d)
        images = render(*a, workspace=ws)
        gF, gp = torch.zeros_like(scene.features), torch.zeros_like(params)
        loss = torch.zeros(1, device="cuda")
        rgb, dep = torch.full((n, 3), -1.0, device="cuda"), torch.full((n,), -1.0, device="cuda")
        step(*a, rgb_t, dep_t, 0.1, 1.0 / n, [gF], gp, out_rgb=rgb, out_depth=dep, loss_out=loss, workspace=ws)
        got[name] = [x.clone() for x in images] + [rgb, dep, gF, gp, loss]
    hit = got["own"][2] > 0
    assert not hit.cpu().numpy()[~live].any()
    assert pattern in ("none", "last") or hit.sum() > 0.3 * live.sum()
    for i, (x, y) in enumerate(zip(got["own"], got["reused"])):
        if i < 5:
            assert torch.equal(x, y), i
        else:
            assert (x - y).abs().max() <= 1e-4 * y.abs().max(), i


def test_deterministic_same_bits_on_reused_hits(gpu_lib):
    """A deterministic train step gives the same bits whether it traverses
    the rays itself or reuses the hits of an earlier call."""
    import torch
    svlf = gpu_lib
    n, K = 40009, 5
    w = tiny_workload(5, 5, 8, (8, 32, 32, 4), K)
    sc = w.scene()
    rng = np.random.default_rng(3)
    o = rng.normal(size=(n, 3))
    o = 3.0 * o / np.linalg.norm(o, axis=1, keepdims=True)
    d = rng.uniform(-0.3, 0.3, (n, 3)) - o
    d[rng.random(n) < 0.8] *= -1.0
    t = rng.uniform(0, 1, (n, 4))
    o, d, rgb_t, dep_t = [torch.from_numpy(np.ascontiguousarray(x, np.float32)).cuda()
                          for x in (o, d, t[:, :3], 3 * t[:, 3])]
    scene = svlf.DeviceScene.from_host(sc.leaf_ijk, sc.depth, w.features())
    params = torch.from_numpy(w.params()).cuda()
    ws = svlf.Workspace()
    got = []
    for flags in (0, svlf.FLAG_REUSE_HITS):
        gF, gp, loss = torch.zeros_like(scene.features), torch.zeros_like(params), torch.zeros(1, device="cuda")
        opts = svlf.make_opts(K, "voxel", "fp32", svlf.FLAG_DETERMINISTIC | flags)
        svlf.train_step([scene], [n], params, w.widths, opts, o, d, rgb_t, dep_t, 0.1, 1.0 / n, [gF], gp,
                        loss_out=loss, workspace=ws)
        got.append((gF, gp, loss))
    assert got[0][0].abs().max() > 0
    for x, y in zip(*got):
        assert torch.equal(x, y)
