"""Timed cases of the SVLF render path, through the public entry points of
paper_2205_07058_amd: views rendered with either decoder form, train passes of
one scene and of several, whole optimisation steps, and a differentiable
render under torch.autograd.

listed()            the cases, small to large
draw(rng)           one more case of the same ranges
prepare(case, seed) scene, features, decoder weights, rays, targets and buffers
run(state)          one pass, returning its outputs
exact(case, seed)   the same outputs in 64 bits (plain torch, no library code)
work(case)          bytes and flops that one pass cannot do without

A case is a dict:

  op         "render" | "train" | "step" | "autograd" | "lf_render" | "lf_train" | "lf_stage"
  scene      "shell" (a spherical shell), "solid" (12 ellipsoids, filled) or
             "surface" (the surfaces of ellipsoids and boxes)
  depth      octree depth; scenes > 1: depths depth, depth + 1, ... in one call
  view       side of a square view (0: a batch)
  rays       rays of a batch: pixels drawn from 50 views, in (view, pixel) order
  C, K       features per vertex (single decoder), hits per ray
  precision, tau, viewdir, deterministic, stage: options of the entry points
"""

import math

import numpy as np
import torch

from paper_2205_07058_amd import autograd, svlf, train

DEV = "cuda"
HIDDEN = {8: (32, 32), 16: (64, 64, 64), 32: (64, 64, 64)}      # hidden layers by C
LF_T, LF_C, LF_H = 64, 32, 128                                  # light-field sizes
LAMBDA_DEPTH, LAMBDA_ETA, LAMBDA_TAU = 0.1, 1.0, 0.1


def _case(name, op, scene, depth, view=0, rays=0, scenes=1, C=32, K=8, precision="bf16", tau="voxel",
          viewdir=False, deterministic=False, stage=""):
    c = dict(op=op, scene=scene, depth=depth, view=view, rays=rays, scenes=scenes, C=C, K=K,
             precision=precision, tau=tau, viewdir=viewdir, deterministic=deterministic, stage=stage)
    return dict(c, name=name) if name else c


def listed():
    return [
        # An interactive preview of a small scene: 4,096 rays, where the launches are the cost.
        _case("view_64_d4_fp32", "render", "shell", 4, view=64, C=8, K=4, precision="fp32"),
        # A frame of a solid scene at full precision.
        _case("view_800_d7_fp32", "render", "solid", 7, view=800, C=16, precision="fp32"),
        # A full-resolution frame of a paper-scale scene, as it is served.
        _case("view_1600_d9_bf16", "render", "surface", 9, view=1600),
        # A small fitting step: the usual few thousand rays, then Adam on everything.
        _case("step_4096_d8_bf16", "step", "surface", 8, rays=4096),
        # Training at full precision on a mid-size batch.
        _case("train_262144_d7_fp32", "train", "solid", 7, rays=1 << 18, C=16, precision="fp32"),
        # Training at paper scale.
        _case("train_1048576_d9_bf16", "train", "surface", 9, rays=1 << 20),
        # A reproducible run with the view direction as an input, on a ragged batch.
        _case("train_det_100003_d8_bf16", "train", "surface", 8, rays=100003, K=11, viewdir=True,
              deterministic=True),
        # A render inside a user's own autograd graph: ragged, long hit lists, full precision.
        _case("autograd_20011_d6_fp32", "autograd", "solid", 6, rays=20011, C=8, K=16, precision="fp32",
              tau="world", viewdir=True),
        # Several scenes of different depths that share one decoder, in one call.
        _case("train_3_scenes_d7_bf16", "train", "surface", 7, rays=400009, scenes=3),
        # A frame of the light-field model.
        _case("lf_view_800_d8_bf16", "lf_render", "surface", 8, view=800, tau="direct"),
        # The light-field model's staged training: one pass of the first stage.
        _case("lf_stage_262144_d9_bf16", "lf_stage", "surface", 9, rays=1 << 18, tau="direct", stage="surface"),
        # Light-field training at full precision on a small scene.
        _case("lf_train_40009_d7_fp32", "lf_train", "surface", 7, rays=40009, tau="direct", precision="fp32"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["render", "render", "render", "train", "train", "train", "step", "autograd", "lf_render",
                     "lf_train", "lf_stage"])
    scene = rng.choice(["solid", "surface", "surface"])
    depth = rng.randint(5, 9) if scene == "surface" else rng.randint(4, 7)
    precision = rng.choice(["fp32", "bf16", "bf16"])
    lf = op.startswith("lf")
    C = 32 if lf else rng.choice([8, 16, 32, 32])
    tau = rng.choice(["direct", "direct", "voxel"] if lf else ["voxel", "voxel", "world"])
    c = dict(C=C, K=rng.randint(4, 16), precision=precision, tau=tau,
             viewdir=(lf or C != 16) and rng.random() < 0.25)
    if op == "render":
        return _case("", op, scene, depth, view=_log(rng, 48, 1500), **c)
    if op == "lf_render":
        return _case("", op, scene, depth, view=_log(rng, 48, 800), **c)
    if lf:
        stage = rng.choice(["surface", "volume"]) if op == "lf_stage" else ""
        return _case("", op, scene, depth, rays=_log(rng, 2000, 200000 if precision == "bf16" else 40000),
                     stage=stage, **c)
    if op == "train":
        several = rng.choice([1, 1, 2, 3]) if scene == "surface" else 1
        return _case("", op, scene, min(depth, 10 - several), rays=_log(rng, 2000, 700000), scenes=several,
                     deterministic=several == 1 and rng.random() < 0.25, **c)
    return _case("", op, scene, depth, rays=_log(rng, 2000, 300000), **c)


# ------------------------------------------------------------------ inputs


def _objects(case, g):
    """(centre, rotation, semi-axes, is_box, albedo) of the scene's objects."""
    if case["scene"] == "shell":
        return [(torch.zeros(3), torch.eye(3), torch.full((3,), 0.6), False, torch.rand(3, generator=g))]
    # "surface": 60 objects of a paper-scale scene (about 1% of the leaves at depth 9), or 18
    # objects in each of several scenes
    solid = case["scene"] == "solid"
    n_ell, n_box, scale = (12, 0, 1.0) if solid else (40, 20, 0.8) if case["scenes"] == 1 else (12, 6, 1.0)
    out = []
    for i in range(n_ell + n_box):
        a = (0.05 + 0.25 * torch.rand(3, generator=g)) * scale
        box = i >= n_ell
        q = torch.nn.functional.normalize(torch.randn(4, generator=g), dim=0).tolist()
        w, x, y, z = q
        rot = torch.tensor([[1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w)],
                            [2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w)],
                            [2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)]])
        r = a.norm().item() if box else a.max().item()
        c = (2 * torch.rand(3, generator=g) - 1) * (1 - r)
        out.append((c, torch.eye(3) if box else rot, a, box, torch.rand(3, generator=g)))
    return out


def _implicit(obj, x, y, z):
    """Negative inside; sign changes on the surface."""
    c, rot, a, box, _ = obj
    p = [x - c[0].item(), y - c[1].item(), z - c[2].item()]
    if box:
        q = [p[k].abs() - a[k].item() for k in range(3)]
        return torch.maximum(torch.maximum(q[0], q[1]), q[2])
    return sum(((rot[0, k].item() * p[0] + rot[1, k].item() * p[1] + rot[2, k].item() * p[2]) / a[k].item()) ** 2
               for k in range(3)) - 1


def _spread(v):
    v = (v | v << 32) & 0x1F00000000FFFF
    v = (v | v << 16) & 0x1F0000FF0000FF
    v = (v | v << 8) & 0x100F00F00F00F00F
    v = (v | v << 4) & 0x10C30C30C30C30C3
    return (v | v << 2) & 0x1249249249249249


def _compact(v):
    v = v & 0x1249249249249249
    v = (v | v >> 2) & 0x10C30C30C30C30C3
    v = (v | v >> 4) & 0x100F00F00F00F00F
    v = (v | v >> 8) & 0x1F0000FF0000FF
    v = (v | v >> 16) & 0x1F00000000FFFF
    return (v | v >> 32) & 0x1FFFFF


def _morton(ijk):
    return _spread(ijk[..., 0]) | _spread(ijk[..., 1]) << 1 | _spread(ijk[..., 2]) << 2


def _leaves(case, objects, depth):
    """Occupied leaves in ascending Morton order, int64 [n][3]."""
    n, h = 1 << depth, 2.0 / (1 << depth)
    codes = []
    for obj in objects:
        c, rot, a, box, _ = obj
        ext = a if box else ((rot ** 2) @ (a ** 2)).sqrt()
        if case["scene"] == "shell":
            ext = ext + 0.05
        lo = [max(0, int((c[k].item() - ext[k].item() + 1) / h) - 1) for k in range(3)]
        hi = [min(n, int((c[k].item() + ext[k].item() + 1) / h) + 2) for k in range(3)]
        x, y, z = (torch.arange(lo[k], hi[k] + 1, device=DEV, dtype=torch.float32) * h - 1 for k in range(3))
        x, y, z = x[:, None, None], y[None, :, None], z[None, None, :]
        if case["scene"] == "shell":
            f = ((x * x + y * y + z * z).sqrt() - 0.6).abs() - 0.05
        else:
            f = _implicit(obj, x, y, z)
        f_lo, f_hi = f, f
        for k in range(3):
            m = f_lo.shape[k] - 1
            f_lo = torch.minimum(f_lo.narrow(k, 0, m), f_lo.narrow(k, 1, m))
            f_hi = torch.maximum(f_hi.narrow(k, 0, m), f_hi.narrow(k, 1, m))
        keep = f_lo <= 0
        if case["scene"] == "surface":
            keep &= f_hi >= 0
        ijk = keep.nonzero() + torch.tensor(lo, device=DEV)
        codes.append(_morton(ijk))
    code = torch.unique(torch.cat(codes))
    return torch.stack([_compact(code >> k) for k in range(3)], 1)


def _rays(case, g, n):
    """Rays of one view, or of pixels drawn from 50 views; FP32 [n][3]."""
    view = case["view"]
    side, views = (view, 1) if view else (800, 50)
    pos = torch.nn.functional.normalize(torch.randn(views, 3, generator=g, dtype=torch.float64), dim=1)
    pos = (3.0 if case["scene"] == "shell" else 4.0) * pos
    f = -torch.nn.functional.normalize(pos, dim=1)
    right = torch.nn.functional.normalize(torch.linalg.cross(f, torch.tensor([[0.0, 0.0, 1.0]], dtype=f.dtype).expand_as(f)), dim=1)
    up = torch.linalg.cross(right, f)
    if view:
        flat = torch.arange(n, device=DEV)
    else:
        dg = torch.Generator(device=DEV).manual_seed(int(torch.randint(1 << 40, (1,), generator=g)))
        flat = torch.randint(0, views * side * side, (n,), generator=dg, device=DEV).sort().values
    v, pix = flat // (side * side), flat % (side * side)
    t = math.tan(math.radians(25.0))
    px = ((pix % side).double() + 0.5) / side * 2 - 1
    py = 1 - ((pix // side).double() + 0.5) / side * 2
    pos, f, right, up = (a.to(DEV)[v] for a in (pos, f, right, up))
    d = torch.nn.functional.normalize(f + px[:, None] * t * right + py[:, None] * t * up, dim=1)
    return pos.float().contiguous(), d.float().contiguous()


def _targets(objects, g, o, d):
    """Lambertian colour and depth of the first object on each ray (0 on a miss)."""
    light = torch.nn.functional.normalize(torch.randn(3, generator=g), dim=0).to(DEV)
    best = torch.full((o.shape[0],), math.inf, device=DEV)
    rgb = torch.zeros_like(o)
    for c, rot, a, box, albedo in objects:
        c, rot, a, albedo = (x.to(DEV) for x in (c, rot, a, albedo))
        p, v = ((o - c) @ rot) / a, (d @ rot) / a
        if box:
            t0, t1 = (-1 - p) / v, (1 - p) / v
            near = torch.minimum(t0, t1)
            t = near.max(1).values
            ok = (t < torch.maximum(t0, t1).min(1).values) & (t > 0)
            k = near.argmax(1, keepdim=True)
            nrm = torch.zeros_like(p).scatter(1, k, -torch.sign(v.gather(1, k)))
        else:
            aa, b, cc = (v * v).sum(1), (p * v).sum(1), (p * p).sum(1) - 1
            disc = b * b - aa * cc
            t = (-b - disc.clamp(min=0).sqrt()) / aa
            ok = (disc > 0) & (t > 0)
            nrm = torch.nn.functional.normalize(((p + t[:, None] * v) / a) @ rot.T, dim=1)
        new = ok & (t < best)
        best = torch.where(new, t, best)
        rgb = torch.where(new[:, None], albedo * (nrm @ light).clamp(min=0)[:, None], rgb)
    return rgb.contiguous(), torch.where(best < math.inf, best, torch.zeros_like(best))


def _widths(case):
    return (case["C"] + (3 if case["viewdir"] else 0),) + HIDDEN[case["C"]] + (4,)


def _lf_widths(case):
    return (2 * LF_T + 6, LF_H, 2), (LF_C + 6 + (3 if case["viewdir"] else 0), LF_H, LF_H, LF_H, 3)


def _xavier(g, widths, bias_at, bias):
    """Xavier-uniform weights, zero biases but for the density output's."""
    parts = []
    for a, b in zip(widths[:-1], widths[1:]):
        parts += [(2 * torch.rand(b * a, generator=g) - 1) * math.sqrt(6.0 / (a + b)), torch.zeros(b)]
    if bias_at is not None:
        parts[-1][bias_at] = bias
    return torch.cat(parts)


def _inputs(case, seed):
    """Everything made from the seed, before any library call."""
    g = torch.Generator().manual_seed(seed)
    dg = torch.Generator(device=DEV).manual_seed(seed + 1)
    lf = case["op"].startswith("lf")
    n = case["view"] ** 2 or case["rays"]
    counts = [n] if case["scenes"] == 1 else [n // (2 << i) for i in range(case["scenes"])]
    if case["scenes"] > 1:
        counts[-1] += n - sum(counts)
    s = dict(case=case, counts=counts, scenes=[])
    o, d, trgb, tdep = [], [], [], []
    for i, m in enumerate(counts):
        # the scene is the case's own (its octree sizes the feature table); the seed gives
        # the features, the weights, the cameras, the rays and the light
        objects = _objects(case, torch.Generator().manual_seed(100 + i))
        leaves = _leaves(case, objects, case["depth"] + i)
        corners = (leaves[:, None, :] + torch.tensor([[j & 1, j >> 1 & 1, j >> 2] for j in range(8)], device=DEV))
        verts, corner = torch.unique(_morton(corners), return_inverse=True)
        c_all = LF_T + LF_C if lf else case["C"]
        F = 0.1 * torch.randn(verts.numel() * c_all, generator=dg, device=DEV)
        s["scenes"].append(dict(leaves=leaves, corners=corner, depth=case["depth"] + i, nv=verts.numel(),
                                F=F if lf else F.view(-1, c_all)))
        ro, rd = _rays(case, g, m)
        tr, td = _targets(objects, g, ro, rd)
        for out, x in ((o, ro), (d, rd), (trgb, tr), (tdep, td)):
            out.append(x)
    s["o"], s["d"], s["trgb"], s["tdep"] = torch.cat(o), torch.cat(d), torch.cat(trgb), torch.cat(tdep)
    if lf:
        wt, wc = _lf_widths(case)
        s["params"] = torch.cat([_xavier(g, wt, 0, 0.5), _xavier(g, wc, None, 0)]).to(DEV)
    else:
        s["params"] = _xavier(g, _widths(case), 3, 1.0).to(DEV)
    # upstream gradients of the differentiable render
    s["g_rgb"] = torch.randn(n, 3, generator=dg, device=DEV) / n
    s["g_depth"] = torch.randn(n, generator=dg, device=DEV) / n
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    n, op = s["o"].shape[0], case["op"]
    bf16 = case["precision"] == "bf16"
    dev = []
    for sc in s["scenes"]:
        scene = svlf.DeviceScene(svlf.DeviceOctree(sc["leaves"].int().cpu().numpy(), sc["depth"], DEV), sc["F"])
        if bf16:
            scene.refresh_bf16()
        dev.append(scene)
    flags = (svlf.FLAG_VIEWDIR if case["viewdir"] else 0) | (svlf.FLAG_DETERMINISTIC if case["deterministic"] else 0)
    st = dict(case=case, n=n, counts=s["counts"], scenes=dev, o=s["o"], d=s["d"], trgb=s["trgb"], tdep=s["tdep"],
              params=s["params"], opts=svlf.make_opts(case["K"], case["tau"], case["precision"], flags),
              ws=svlf.Workspace())
    if op in ("train", "lf_train", "lf_stage"):
        st.update(rgb=torch.empty(n, 3, device=DEV), depth=torch.empty(n, device=DEV), loss=torch.empty(1, device=DEV),
                  gF=[torch.zeros_like(x.features) for x in dev], gp=torch.zeros_like(s["params"]))
    if op == "lf_stage":
        st["kind"] = svlf.make_lf_loss(case["stage"], LAMBDA_ETA, LAMBDA_TAU if case["stage"] == "surface" else 0.0,
                                       1.0 / n, case["stage"] == "volume")
    if op == "step":
        st["trainer"] = train.Trainer(dev[0], s["params"], _widths(case), case["K"], case["precision"], case["tau"],
                                      viewdir=case["viewdir"])
    if op == "autograd":
        st.update(g_rgb=s["g_rgb"], g_depth=s["g_depth"], F=dev[0].features.requires_grad_(),
                  params=s["params"].requires_grad_())
    return st


# ------------------------------------------------------------------ one pass


def run(st):
    case, op = st["case"], st["case"]["op"]
    if op == "render":
        return svlf.render(st["scenes"], st["counts"], st["params"], _widths(case), st["opts"], st["o"], st["d"],
                           workspace=st["ws"])
    if op == "lf_render":
        return svlf.lf_render(st["scenes"], st["counts"], st["params"], st["opts"], st["o"], st["d"],
                              workspace=st["ws"])
    if op == "step":
        t = st["trainer"]
        loss = t.step(st["o"], st["d"], st["trgb"], st["tdep"])
        return dict(loss=loss, features=t.scene.features, params=t.params, mF=t.mF, vF=t.vF, mp=t.mp, vp=t.vp)
    if op == "autograd":
        rgb, depth, acc = autograd.render(st["scenes"][0], st["params"], _widths(case), st["o"], st["d"], case["K"],
                                          case["tau"], case["precision"], features=st["F"], viewdir=case["viewdir"])
        gF, gp = torch.autograd.grad([rgb, depth], [st["F"], st["params"]], [st["g_rgb"], st["g_depth"]])
        return rgb.detach(), depth.detach(), acc.detach(), gF, gp
    out = dict(grad_features=st["gF"], grad_params=st["gp"])     # gradients accumulate, as over micro-batches
    kept = dict(out_rgb=st["rgb"], out_depth=st["depth"], loss_out=st["loss"], workspace=st["ws"])
    if op == "train":
        svlf.train_step(st["scenes"], st["counts"], st["params"], _widths(case), st["opts"], st["o"], st["d"],
                        st["trgb"], st["tdep"], LAMBDA_DEPTH, 1.0 / st["n"], **out, **kept)
    elif op == "lf_train":
        svlf.lf_train_step(st["scenes"], st["counts"], st["params"], st["opts"], st["o"], st["d"], st["trgb"],
                           st["tdep"], LAMBDA_DEPTH, 1.0 / st["n"], **out, **kept)
    else:
        svlf.lf_train_stage(st["scenes"], st["counts"], st["params"], st["opts"], st["o"], st["d"], st["trgb"],
                            st["tdep"], st["kind"], **out, **kept)
    return dict(out, rgb=st["rgb"], depth=st["depth"], loss=st["loss"])


# ------------------------------------------------------------------ 64 bits


def _first_hits(sc, o, d, K):
    """(ray, leaf, t_in, t_out) of each ray's first K leaves, in order. The slab test is binary32 with separate
    roundings, as the library's interface defines it; levels are expanded one after the other."""
    depth, code = sc["depth"], _morton(sc["leaves"])
    inv = (1.0 / d.double()).float()

    def meets(ray, cell, level):
        h = 2.0 / (1 << level)
        t_in, t_out = torch.zeros(ray.numel(), device=DEV), torch.full((ray.numel(),), math.inf, device=DEV)
        for k in range(3):
            lo = _compact(cell >> k).float() * h - 1
            oo, iv = o[ray, k], inv[ray, k]
            t0, t1 = (lo - oo) * iv, (lo + h - oo) * iv
            a, b = torch.minimum(t0, t1), torch.maximum(t0, t1)
            flat, inside = torch.isinf(iv), (lo <= oo) & (oo < lo + h)
            a = torch.where(flat, torch.where(inside, -math.inf, math.inf), a)
            b = torch.where(flat, math.inf, b)
            t_in, t_out = torch.maximum(t_in, a), torch.minimum(t_out, b)
        return t_in, t_out

    out, step = [], 1 << 18
    for first in range(0, o.shape[0], step):
        ray = torch.arange(first, min(first + step, o.shape[0]), device=DEV)
        cell = torch.zeros_like(ray)
        for level in range(depth + 1):
            if level:
                nodes = torch.unique_consecutive(code >> 3 * (depth - level))
                lo, hi = (torch.searchsorted(nodes, (cell + e) << 3) for e in (0, 1))
                m = hi - lo
                start = torch.repeat_interleave(lo - (m.cumsum(0) - m), m)
                cell = nodes[start + torch.arange(start.numel(), device=DEV)]
                ray = torch.repeat_interleave(ray, m)
            t_in, t_out = meets(ray, cell, level)
            keep = t_in < t_out
            ray, cell, t_in, t_out = ray[keep], cell[keep], t_in[keep], t_out[keep]
        order = t_in.sort(stable=True).indices
        order = order[ray[order].sort(stable=True).indices]
        ray, cell, t_in, t_out = ray[order], cell[order], t_in[order], t_out[order]
        n = torch.bincount(ray - first, minlength=1)
        slot = torch.arange(ray.numel(), device=DEV) - (n.cumsum(0) - n)[ray - first]
        k = slot < K
        out.append((ray[k], torch.searchsorted(code, cell[k]), t_in[k], t_out[k], slot[k]))
    return [torch.cat(x) for x in zip(*out)]


def _psi(F, corners, u):
    """Trilinear interpolation of rows F[corner] at u in [0, 1]^3."""
    out = 0
    for j in range(8):
        w = 1
        for k in range(3):
            w = w * (u[:, k] if j >> k & 1 else 1 - u[:, k])
        out = out + w[:, None] * F.index_select(0, corners[:, j])
    return out


def _mlp(p, widths, x):
    at = 0
    for i, (a, b) in enumerate(zip(widths[:-1], widths[1:])):
        x = x @ p[at:at + a * b].view(b, a).T + p[at + a * b:at + a * b + b]
        at += a * b + b
        if i + 2 < len(widths):
            x = torch.relu(x)
    return x


def _composite(n, K, ray, slot, tau, c, t):
    """Eq. 3 over each ray's hits: rgb, depth, acc."""
    at = ray * K + slot
    tau = torch.zeros(n * K, dtype=tau.dtype, device=DEV).index_put((at,), tau).view(n, K)
    val = torch.zeros(n * K, 5, dtype=c.dtype, device=DEV).index_put(
        (at,), torch.cat([c, t[:, None], torch.ones_like(t)[:, None]], 1)).view(n, K, 5)
    w = torch.exp(-(tau.cumsum(1) - tau)) * -torch.expm1(-tau)
    r = (w[:, :, None] * val).sum(1)
    return r[:, :3], r[:, 3], r[:, 4]


def exact(case, seed):
    s = _inputs(case, seed)
    op, K, lf = case["op"], case["K"], case["op"].startswith("lf")
    grads = op not in ("render", "lf_render")
    params = s["params"].double().requires_grad_(grads)
    feats = [sc["F"].double().requires_grad_(grads) for sc in s["scenes"]]
    o, d, n = s["o"].double(), s["d"].double(), s["o"].shape[0]
    rays, slots, taus, cols, ts, extra = [], [], [], [], [], []
    begin = 0
    for sc, F, m in zip(s["scenes"], feats, s["counts"]):
        ray, leaf, t0, t1, slot = _first_hits(sc, s["o"][begin:begin + m], s["d"][begin:begin + m], K)
        f_in, f_out = t0, t1
        ray, h = ray + begin, 2.0 / (1 << sc["depth"])
        begin += m
        oo, dd, t0, t1 = o[ray], d[ray], t0.double(), t1.double()
        lo = sc["leaves"][leaf].double() * h - 1
        corners = sc["corners"][leaf]
        scale = {"voxel": (t1 - t0) / h, "world": t1 - t0, "direct": torch.ones_like(t0)}[case["tau"]]

        def cell(t):
            return ((oo + t[:, None] * dd - lo) / h).clamp(0, 1)
        if not lf:
            t = (t0 + t1) / 2
            x = _psi(F, corners, cell(t))
            y = _mlp(params, _widths(case), torch.cat([x, dd], 1) if case["viewdir"] else x)
            c, tau = torch.sigmoid(y[:, :3]), torch.relu(y[:, 3]) * scale
        else:
            wt, wc = _lf_widths(case)
            n_t = sum(a * b + b for a, b in zip(wt[:-1], wt[1:]))
            Z_T, Z_C = F[:sc["nv"] * LF_T].view(-1, LF_T), F[sc["nv"] * LF_T:].view(-1, LF_C)
            y = oo - (lo + h / 2)
            a, b = (dd * dd).sum(1), (dd * y).sum(1)
            root = (b * b - a * ((y * y).sum(1) - 0.75 * h * h)).clamp(min=0).sqrt()
            r = torch.cat([torch.nn.functional.normalize(y + ((-b + e * root) / a)[:, None] * dd, dim=1)
                           for e in (-1, 1)], 1)
            z = _mlp(params[:n_t], wt, torch.cat([_psi(Z_T, corners, cell(t0)), _psi(Z_T, corners, cell(t1)), r], 1))
            tau, eta = torch.relu(z[:, 0]) * scale, torch.sigmoid(z[:, 1])
            t = eta * t0 + (1 - eta) * t1
            x = [_psi(Z_C, corners, cell(t)), r] + ([dd] if case["viewdir"] else [])
            c = torch.sigmoid(_mlp(params[n_t:], wc, torch.cat(x, 1)))
            if op == "lf_stage":
                want = s["tdep"][ray]
                at = (f_in <= want) & (want < f_out)
                far = (t1 - want.double()) / (t1 - t0)
                e = LAMBDA_ETA * (eta - far) ** 2
                if case["stage"] == "surface":
                    e = e + ((c - s["trgb"][ray].double()) ** 2).sum(1) + LAMBDA_TAU * torch.exp(-2 * tau)
                extra.append(e[at].sum())
        for out, v in ((rays, ray), (slots, slot), (taus, tau), (cols, c), (ts, t)):
            out.append(v)
    rgb, depth, acc = _composite(n, K, *(torch.cat(v) for v in (rays, slots, taus, cols, ts)))
    if not grads:
        return rgb, depth, acc
    trgb, tdep = s["trgb"].double(), s["tdep"].double()
    if op == "autograd":
        loss = (rgb * s["g_rgb"].double()).sum() + (depth * s["g_depth"].double()).sum()
    elif op == "lf_stage":
        loss = sum(extra) / n
        if case["stage"] == "volume":
            loss = loss + ((rgb - trgb) ** 2).sum() / n
    else:
        loss = (((rgb - trgb) ** 2).sum() / 3 + LAMBDA_DEPTH * (depth - tdep).abs().sum()) / n
    gp, *gF = torch.autograd.grad(loss, [params] + feats)
    if op == "lf_stage" and case["stage"] == "volume":      # the colour side is frozen
        gp[n_t:] = 0
        for sc, x in zip(s["scenes"], gF):
            x[sc["nv"] * LF_T:] = 0
    rgb, depth, loss = rgb.detach(), depth.detach(), loss.detach().view(1)
    if op == "autograd":
        return rgb, depth, acc.detach(), gF[0], gp
    if op != "step":
        return dict(grad_features=gF, grad_params=gp, rgb=rgb, depth=depth, loss=loss)
    out = dict(loss=loss)
    for name, m, v, p, x in (("features", "mF", "vF", feats[0], gF[0]), ("params", "mp", "vp", params, gp)):
        b1, b2, eps, lr = (float(np.float32(b)) for b in (0.9, 0.999, 1e-8, 1e-3))
        out[m], out[v] = (1 - b1) * x, (1 - b2) * x * x
        out[name] = p.detach() - lr * x / (x.abs() + eps)     # the first step's bias corrections
    return out


# ------------------------------------------------------------------ work


def work(case):
    """One read of every ray, target and touched feature row, leaf and octree node, one write of every output;
    gradients of the touched rows read and written; Adam's state where it runs. The decoder's multiply-adds for
    each hit, three times as many with a backward pass."""
    s = _inputs(case, 0)
    op, n = case["op"], s["o"].shape[0]
    lf, grads = op.startswith("lf"), op not in ("render", "lf_render")
    c_all = LF_T + LF_C if lf else case["C"]
    n_params = s["params"].numel()
    if lf:
        macs = sum(a * b for w in _lf_widths(case) for a, b in zip(w[:-1], w[1:]))
    else:
        macs = sum(a * b for a, b in zip(_widths(case)[:-1], _widths(case)[1:]))
    bytes_ = n * (24 + 16 + (4 if not grads or op == "autograd" else 0) + (16 if grads else 0)) + 4 * n_params
    hits = begin = 0
    for sc, m in zip(s["scenes"], s["counts"]):
        _, leaf, *_ = _first_hits(sc, s["o"][begin:begin + m], s["d"][begin:begin + m], case["K"])
        begin += m
        hits += leaf.numel()
        leaf = torch.unique(leaf)
        rows = torch.unique(sc["corners"][leaf]).numel()
        bytes_ += leaf.numel() * 32 + rows * c_all * (2 if case["precision"] == "bf16" else 4)
        code = _morton(sc["leaves"])[leaf]
        bytes_ += 8 * sum(torch.unique_consecutive(code >> 3 * k).numel() for k in range(1, sc["depth"] + 1))
        if op == "step":
            bytes_ += sc["nv"] * c_all * (30 if case["precision"] == "bf16" else 28) + rows * c_all * 4
        elif grads:
            bytes_ += rows * c_all * 8
        if op == "autograd":                                   # the gradient is a new tensor
            bytes_ += (sc["nv"] - rows) * c_all * 4
    if op == "step":
        bytes_ += 24 * n_params
    return {"bytes": bytes_, "flops": 2 * macs * hits * (3 if grads else 1)}
