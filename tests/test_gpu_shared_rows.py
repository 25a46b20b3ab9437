"""A feature row that consecutive hits of a ray share is added once by the
atomic backward (the sum is handed from hit to hit); the deterministic one keeps
every hit's share and sums them per vertex.  Both must agree, for chains of hits
through the 26 kinds of neighbouring cells: rays from cell centres of a full
grid along every sign combination, which cross faces, edges (two axes at once)
or corners (three), and random rays, whose chains mix them."""

import itertools

import numpy as np
import pytest

from synth.configs import xavier_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("widths", [(8, 32, 32, 4), (16, 64, 64, 64, 4), (32, 64, 64, 64, 4)])
def test_shared_rows(gpu_lib, widths, precision):
    import torch
    svlf = gpu_lib
    depth, K = 4, 16
    side = 1 << depth
    ijk = np.stack(np.meshgrid(*[np.arange(side)] * 3, indexing="ij"), -1).reshape(-1, 3).astype(np.int32)
    rng = np.random.default_rng(2)
    signs = np.array([s for s in itertools.product((-1, 0, 1), repeat=3) if any(s)], np.float32)
    d = np.concatenate([np.repeat(signs, 40, 0), rng.normal(size=(1500, 3)).astype(np.float32)])
    cells = rng.integers(0, side, d.shape)
    cells = np.where(rng.random(d.shape) < 0.7, np.where(d < 0, side - 1, np.where(d > 0, 0, cells)), cells)   # long chains
    o = (-1 + (cells + 0.5) * (2.0 / side)).astype(np.float32)
    p = rng.permutation(len(d))
    n = len(d)
    o, d = (torch.from_numpy(np.ascontiguousarray(x[p])).cuda() for x in (o, d))
    F = rng.normal(0, 0.3, ((side + 1) ** 3, widths[0])).astype(np.float32)
    scene = svlf.DeviceScene.from_host(ijk, depth, F)
    w = xavier_params(rng, widths)
    w[-1] = 0.1                                        # long chains stay visible
    params = torch.from_numpy(w.astype(np.float32)).cuda()
    count = svlf.trace_hits(scene.octree, o, d, K)[3]
    assert (count >= 8).float().mean() > 0.3 and count.max() == K
    g_rgb = torch.from_numpy(rng.normal(size=(n, 3)).astype(np.float32)).cuda()
    g_dep = torch.from_numpy(rng.normal(size=n).astype(np.float32)).cuda()
    got = []
    for flags in (0, svlf.FLAG_DETERMINISTIC):
        gF, gp = torch.zeros_like(scene.features), torch.zeros_like(params)
        svlf.render_backward([scene], [n], params, widths, svlf.make_opts(K, "voxel", precision, flags), o, d, g_rgb,
                             g_dep, None, [gF], gp)
        got.append(gF)
    # the same terms in another order: at most some hundred per entry
    assert got[1].abs().max() > 0
    assert (got[0] - got[1]).abs().max() <= 1e-5 * got[1].abs().max()
