"""Workloads whose speed is measured, each a call that programs on this
framework make: training steps (one view, and a batch of views), frames
rendered without gradients, seeding from a point cloud (plain and learned),
training of the seeding network, bundle adjustment and multi-view stereo.

A case is a dict of plain values; `kind` says which entry points it goes
through.  `prepare` makes what a program holds before the call, `run` is one
pass, `work` the bytes and operations the pass cannot do without, and `exact`
the outputs in float64 from plain torch.
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_2601_17354_amd import ba, seed_mlp
from paper_2601_17354_amd.batch import MIXED_SIZES, BatchedStep
from paper_2601_17354_amd.mvs import MVS, MVSParams
from paper_2601_17354_amd.raster import Rasterizer, param_rows
from paper_2601_17354_amd.train import Trainer, learning_rates, seed_pca

DEV = "cuda"
F64 = torch.float64


def listed():
    return [
        # The smallest step: the parity workload's 1000 Gaussians, where launches and host calls count.
        dict(name="train_1k_128", kind="train", n=1000, sh=0, w=128, h=128, lam=0.0, cached=True, check=True),
        # A preview-sized step on a ragged image, as `train` runs it: flags read every step, recompute backward.
        dict(name="train_20k_317x243", kind="train", n=20000, sh=1, w=317, h=243, lam=0.2, cached=False, check=True),
        # 100k Gaussians with view-dependent colour (SH degree 3), one 1024x768 view, L1 loss, recompute backward.
        dict(name="train_100k_sh3_1024", kind="train", n=100000, sh=3, w=1024, h=768, lam=0.0, cached=False,
             check=False),
        # The headline training step: 300k Gaussians at 1920x1440 with the replay trace.
        dict(name="train_300k_1920", kind="train", n=300000, sh=0, w=1920, h=1440, lam=0.2, cached=True,
             check=False),
        # Viewing a trained model: frames without trace or gradients.
        dict(name="render_300k_1920", kind="render", n=300000, sh=0, w=1920, h=1440),
        # The largest: eight views of uneven resolution in one step, 1M Gaussians at SH degree 3.
        dict(name="batch_1m_sh3_8views", kind="batch", n=1000000, sh=3, views=8, first=0, cached=True),
        # Plain seeding of the benchmark's cloud: 16 nearest neighbours and the disc seed.
        dict(name="seed_300k", kind="seed", m=300000),
        # Learned seeding of a fresh scene's cloud: neighbours, features, network, fall back.
        dict(name="learned_seed_200k", kind="learned", m=200000),
        # One optimisation step of the seeding network at its training batch size.
        dict(name="seednet_16384", kind="seednet", m=16384),
        # One Levenberg-Marquardt iteration of a whole capture: 60 keyframes, 100k points, up to 8 views each.
        dict(name="ba_60x100k", kind="ba", cams=60, points=100000, iters=0),
        # A short adjustment while a capture runs: few keyframes, five iterations with their accept tests.
        dict(name="ba_12x2k_lm5", kind="ba", cams=12, points=2000, iters=5),
        # Dense stereo of a batch of eight 960x720 targets at 128 planes: census to fused cloud.
        dict(name="mvs_8x960x720x128", kind="mvs", targets=8, views=16, w=960, h=720, planes=128),
    ]


def _logint(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["train", "train", "train", "render", "batch", "seed", "learned", "seednet", "ba", "mvs"])
    if kind in ("train", "render"):
        w = _logint(rng, 64, 1920)
        c = dict(kind=kind, n=_logint(rng, 500, 300000), sh=rng.randrange(4), w=w,
                 h=max(32, int(w * rng.uniform(0.55, 1.0))))
        if kind == "train":
            c.update(lam=rng.choice([0.0, 0.2]), cached=rng.random() < 0.5, check=rng.random() < 0.5)
        return c
    if kind == "batch":
        v = rng.randint(1, 8)
        return dict(kind=kind, n=_logint(rng, 5000, 600000), sh=rng.randrange(4), views=v, first=rng.randint(0, 8 - v),
                    cached=rng.random() < 0.5)
    if kind in ("seed", "learned"):
        return dict(kind=kind, m=_logint(rng, 2000, 300000))
    if kind == "seednet":
        return dict(kind=kind, m=_logint(rng, 40, 65536))
    if kind == "ba":
        cams = _logint(rng, 3, 70)
        iters = rng.choice([0, 0, 3])
        return dict(kind=kind, cams=cams, points=_logint(rng, 60, 100000 if iters == 0 else 20000), iters=iters)
    w = _logint(rng, 64, 960)
    return dict(kind=kind, targets=rng.randint(1, 8), views=rng.randint(8, 16), w=w, h=max(40, int(w * rng.uniform(0.6, 0.8))),
                planes=rng.choice([64, 128, 128, 192, 256]) if w < 640 else rng.choice([64, 128]))


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


class _Scene:
    """Twenty spheres, a floor and two walls with a procedural texture."""

    def __init__(self, seed):
        r = np.random.default_rng(seed)
        rd, th = 2.5 * np.sqrt(r.uniform(0, 1, 20)), r.uniform(0, 2 * np.pi, 20)
        t = lambda a: torch.as_tensor(a, dtype=torch.float32, device=DEV)  # noqa: E731
        self.centres = t(np.stack([rd * np.cos(th), r.uniform(-0.5, 1.5, 20), rd * np.sin(th)], 1))
        radii = r.uniform(0.2, 1.0, 20)
        self.radii = t(radii)
        # origin, two unit axes, normal, extents
        self.planes = [([-6, -1.5, -6], [1, 0, 0], [0, 0, 1], [0, 1, 0], 12.0, 12.0),
                       ([-6, -1.5, -6], [1, 0, 0], [0, 1, 0], [0, 0, 1], 12.0, 6.0),
                       ([-6, -1.5, -6], [0, 0, 1], [0, 1, 0], [1, 0, 0], 12.0, 6.0)]
        self.areas = np.concatenate([4 * np.pi * radii ** 2, [p[4] * p[5] for p in self.planes]])
        self.base, self.freq = t(r.uniform(0.15, 0.85, (23, 3))), t(r.uniform(2.0, 9.0, (23, 3)))
        self.phase = t(r.uniform(0, 2 * np.pi, (23, 3)))

    def colour(self, sid, p):
        b, f, ph = self.base[sid], self.freq[sid], self.phase[sid]
        s = torch.sin(f * p + ph) * torch.sin(0.7 * f * p[:, [1, 2, 0]] + 1.3 * ph)
        chk = torch.remainder(torch.floor(2 * p).sum(1), 2)
        return torch.clamp(b + 0.25 * s + 0.08 * (chk[:, None] - 0.5), 0.02, 0.98)

    def sample(self, n, g):
        """n points, normals and colours on the surfaces, by area."""
        sid = torch.multinomial(torch.as_tensor(self.areas / self.areas.sum(), device=DEV), n, replacement=True,
                                generator=g)
        d = torch.nn.functional.normalize(torch.randn((n, 3), generator=g, device=DEV), dim=1)
        k = sid.clamp(max=19)
        pts, nrm = self.centres[k] + self.radii[k, None] * d, d.clone()
        uv = torch.rand((n, 2), generator=g, device=DEV)
        for i, (o, ua, va, nn, ul, vl) in enumerate(self.planes):
            o, ua, va, nn = (torch.tensor(x, dtype=torch.float32, device=DEV) for x in (o, ua, va, nn))
            on = (sid == 20 + i)[:, None]
            pts = torch.where(on, o + uv[:, :1] * ul * ua + uv[:, 1:] * vl * va, pts)
            nrm = torch.where(on, nn.expand(n, 3), nrm)
        return pts, nrm, self.colour(sid, pts)


def _camera(w, h, eye, target, hfov=60.0):
    eye = np.asarray(eye, np.float64)
    f = np.asarray(target, np.float64) - eye
    f /= np.linalg.norm(f)
    r = np.cross(f, [0.0, 1.0, 0.0])
    r /= np.linalg.norm(r)
    R = np.stack([r, np.cross(f, r), f])
    fx = float(np.float32(w / (2 * math.tan(math.radians(hfov) / 2))))
    vm = np.concatenate([R, (-R @ eye)[:, None]], 1).astype(np.float32)
    return dict(width=w, height=h, fx=fx, fy=fx, cx=w / 2.0, cy=h / 2.0, viewmat=vm)


def _ring(w, h, angle, height=0.8, radius=4.5):
    return _camera(w, h, (radius * math.sin(angle), height, radius * math.cos(angle)), (0.0, 0.3, 0.0))


def _gaussians(n, sh, seed):
    """Canonical parameters [F][n]: a random cube of Gaussians below 5000,
    else flat Gaussians on a scene's surfaces with a spread of sizes and
    opacities, as a model in training has."""
    g = _gen(seed)
    P = torch.zeros((param_rows(sh), n), dtype=torch.float32, device=DEV)
    if n < 5000:
        P[0:3] = 2 * torch.rand((3, n), generator=g, device=DEV) - 1
        P[2] += 4.0
        P[3:6] = -3.0 + 0.5 * torch.randn((3, n), generator=g, device=DEV)
        P[6:10] = torch.nn.functional.normalize(torch.randn((4, n), generator=g, device=DEV), dim=0)
        P[10] = torch.randn(n, generator=g, device=DEV)
        P[11:14] = math.sqrt(math.pi) * (2 * torch.rand((3, n), generator=g, device=DEV) - 1)
    else:
        scene = _Scene(seed)
        pts, nrm, col = scene.sample(n, g)
        s = math.log(0.6 * math.sqrt(float(scene.areas.sum()) / n))
        P[0:3] = pts.T
        P[3:6] = s + 0.3 * torch.randn((3, n), generator=g, device=DEV)
        P[5] -= 1.5
        qa = torch.stack([1 + nrm[:, 2], -nrm[:, 1], nrm[:, 0], torch.zeros(n, device=DEV)], 1)
        qa[qa[:, 0] < 1e-4] = torch.tensor([0.0, 1.0, 0.0, 0.0], device=DEV)
        qa = torch.nn.functional.normalize(qa, dim=1)
        a = math.pi * torch.rand(n, generator=g, device=DEV)
        c, z = torch.cos(a), torch.sin(a)
        w_, x_, y_ = qa[:, 0], qa[:, 1], qa[:, 2]
        P[6:10] = torch.stack([w_ * c, x_ * c + y_ * z, y_ * c - x_ * z, w_ * z])
        P[10] = 0.5 + 1.5 * torch.randn(n, generator=g, device=DEV)
        P[11:14] = ((col - 0.5) * (2 * math.sqrt(math.pi))).T
    if sh:
        P[14:] = 0.05 * torch.randn((P.shape[0] - 14, n), generator=g, device=DEV)
    return P


def _image(w, h, seed):
    """A smooth picture with some fine detail, in [0, 1]."""
    g = _gen(seed)
    lo = torch.rand((1, 3, 12, 12), generator=g, device=DEV)
    im = torch.nn.functional.interpolate(lo, size=(h, w), mode="bilinear", align_corners=False)[0]
    return torch.clamp(im + 0.05 * torch.randn((3, h, w), generator=g, device=DEV), 0, 1).contiguous()


def _view(case, seed):
    if case["n"] < 5000:
        f = float(max(case["w"], case["h"]))
        vm = np.zeros((3, 4), np.float32)
        vm[:, :3] = np.eye(3)
        return dict(width=case["w"], height=case["h"], fx=f, fy=f, cx=case["w"] / 2.0, cy=case["h"] / 2.0, viewmat=vm)
    return _ring(case["w"], case["h"], 2 * math.pi * (seed % 60) / 60)


def _batch_views(case, seed):
    return [_ring(*MIXED_SIZES[case["first"] + v], 2 * math.pi * (v / 8 + (seed % 7) / 60)) for v in range(case["views"])]


def _cloud(m, seed):
    g = _gen(seed)
    pts, _, col = _Scene(seed).sample(m, g)
    pts = pts + 0.01 * torch.randn((m, 3), generator=g, device=DEV)
    return pts.T.contiguous(), col.T.contiguous()


def _rotation_of(q):
    w, x, y, z = q.unbind(-1)
    return torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                        2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                        2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], -1).reshape(*q.shape[:-1], 3, 3)


def _net_batch(m, seed):
    """Feature rows, base seeds and targets as scene pairs have them: offsets
    of a few s_t in the local frame, a disc base, a target near it."""
    g = _gen(seed)
    rnd = lambda *s: torch.randn(s, generator=g, device=DEV)  # noqa: E731
    x = torch.zeros((m, 64), device=DEV)
    off = 1.5 * rnd(m, 16, 3)
    off[:, :, 2] *= 0.2
    x[:, :48] = off.reshape(m, 48)
    d = off - off.mean(1, keepdim=True)
    x[:, 48:57] = (d.transpose(1, 2) @ d / 16).reshape(m, 9)
    q = torch.nn.functional.normalize(rnd(m, 4), dim=1)
    ls = -4.0 + 0.5 * rnd(m)
    s = torch.stack([ls, ls, ls + math.log(0.1)], 1)
    R = _rotation_of(q)
    base = torch.cat([R.reshape(m, 9), s, q], 1).contiguous()
    s2 = 2 * (s + 0.3 * rnd(m, 3))
    M = R @ torch.diag_embed(s2) @ R.transpose(1, 2)
    t = torch.stack([M[:, 0, 0], M[:, 1, 1], M[:, 2, 2], M[:, 0, 1], M[:, 0, 2], M[:, 1, 2],
                     0.5 + 1.5 * rnd(m), torch.zeros(m, device=DEV)], 1).contiguous()
    return x, base, t


def _net_weights(seed):
    w = seed_mlp.load_weights(device=DEV)
    return w + 0.01 * torch.randn(w.shape, generator=_gen(seed + 77), device=DEV)


def _tracks(case, seed):
    """Ring keyframes and surface points seen by up to 8 of them: pixel noise
    of 0.5, 1% of wrong matches, a perturbed start (as numpy arrays)."""
    C, M = case["cams"], case["points"]
    g = _gen(seed)
    cams = [_ring(1920, 1440, 2 * math.pi * i / C) for i in range(C)]
    vm = np.stack([c["viewmat"].astype(np.float64) for c in cams])
    U, _, Vt = np.linalg.svd(vm[:, :, :3])
    R = U @ Vt
    centre = -np.einsum("cji,cj->ci", R, vm[:, :, 3])
    pts = _Scene(seed).sample(M + M // 4 if C >= 8 else 4 * M, g)[0].to(F64)
    Rt, ct = torch.as_tensor(R, device=DEV), torch.as_tensor(centre, device=DEV)
    f, cx, cy = cams[0]["fx"], 960.0, 720.0
    xc = torch.einsum("cij,mcj->mci", Rt, pts[:, None] - ct[None])
    z = xc[..., 2]
    uv = torch.stack([f * xc[..., 0] / z + cx, f * xc[..., 1] / z + cy], -1)
    vis = (z > 0.2) & (uv[..., 0] >= 0) & (uv[..., 0] < 1920) & (uv[..., 1] >= 0) & (uv[..., 1] < 1440)
    key = torch.where(vis, torch.rand(vis.shape, generator=g, device=DEV), 2.0)
    rank = key.argsort(1).argsort(1)
    vis &= rank < 8
    keep = (vis.sum(1) >= 2).nonzero()[:, 0]
    keep = keep.repeat(-(-M // keep.numel()))[:M]
    vis, uv, pts = vis[keep], uv[keep], pts[keep]
    o = vis.nonzero()
    obs = uv[o[:, 0], o[:, 1]]
    k = o.shape[0]
    obs = obs + 0.5 * torch.randn((k, 2), generator=g, device=DEV, dtype=F64)
    wrong = torch.rand(k, generator=g, device=DEV) < 0.01
    anywhere = torch.rand((k, 2), generator=g, device=DEV, dtype=F64) * torch.tensor([1920.0, 1440.0], device=DEV)
    obs = torch.where(wrong[:, None], anywhere, obs)
    wn = math.radians(0.5) * torch.randn((C, 3), generator=g, device=DEV, dtype=F64)
    R0 = Rt @ _exp_so3(wn)
    c0 = ct + 0.02 * torch.randn((C, 3), generator=g, device=DEV, dtype=F64)
    P0 = pts + 0.02 * torch.randn(pts.shape, generator=g, device=DEV, dtype=F64)
    axis = int(np.argmax(np.abs(centre[1] - centre[0])))
    R0[0], c0[0] = Rt[0], ct[0]
    c0[1, axis] = ct[1, axis]
    return dict(obs_cam=o[:, 1].cpu().numpy().astype(np.uint32), obs_pt=o[:, 0].cpu().numpy().astype(np.uint32),
                obs_uv=obs.cpu().numpy(), fx=f, fy=f, cx=cx, cy=cy, gauge_axis=axis, R0=R0.cpu().numpy(),
                c0=c0.cpu().numpy(), P0=P0.cpu().numpy())


def _exp_so3(w):
    th = w.norm(dim=1).clamp(min=1e-150)[:, None, None]
    z = torch.zeros_like(w[:, 0])
    K = torch.stack([z, -w[:, 2], w[:, 1], w[:, 2], z, -w[:, 0], -w[:, 1], w[:, 0], z], 1).reshape(-1, 3, 3)
    return torch.eye(3, dtype=w.dtype, device=w.device) + torch.sin(th) / th * K + (1 - torch.cos(th)) / th ** 2 * (K @ K)


def _capture(case, seed):
    """Grey views [V][H][W] of a scene ray-cast along a hand-held arc, their
    cameras, and sparse surface points."""
    g = _gen(seed)
    r = np.random.default_rng(seed)
    scene = _Scene(seed)
    V, W, H = case["views"], case["w"], case["h"]
    a0 = 2 * math.pi * r.uniform()
    cams = [_ring(W, H, a0 + i * 0.09 + r.uniform(-0.01, 0.01), 0.8 + r.uniform(-0.05, 0.05),
                  4.5 + r.uniform(-0.1, 0.1)) for i in range(V)]
    noise = torch.rand((64, 64, 64), generator=g, device=DEV)
    grey = torch.empty((V, H, W), dtype=torch.uint8, device=DEV)
    ys, xs = torch.meshgrid(torch.arange(H, device=DEV, dtype=torch.float32),
                            torch.arange(W, device=DEV, dtype=torch.float32), indexing="ij")
    for v, cam in enumerate(cams):
        vm = torch.as_tensor(cam["viewmat"], device=DEV)
        R, t = vm[:, :3], vm[:, 3]
        o = -R.T @ t
        d = torch.stack([(xs.reshape(-1) - cam["cx"]) / cam["fx"], (ys.reshape(-1) - cam["cy"]) / cam["fy"],
                         torch.ones(H * W, device=DEV)], 1) @ R
        best = torch.full((H * W,), math.inf, device=DEV)
        sid = torch.full((H * W,), -1, dtype=torch.int64, device=DEV)
        aa = (d * d).sum(1)
        for s in range(20):
            oc = o - scene.centres[s]
            b = d @ oc
            disc = b * b - aa * (oc @ oc - scene.radii[s] ** 2)
            z = (-b - torch.sqrt(disc.clamp(min=0))) / aa
            hit = (disc >= 0) & (z >= 0.2) & (z < best)
            best, sid = torch.where(hit, z, best), torch.where(hit, s, sid)
        for k, (po, ua, va, nn, ul, vl) in enumerate(scene.planes):
            po, ua, va, nn = (torch.tensor(x, dtype=torch.float32, device=DEV) for x in (po, ua, va, nn))
            z = ((po - o) @ nn) / (d @ nn)
            q = o + z[:, None] * d - po
            u, w_ = q @ ua, q @ va
            hit = (z >= 0.2) & (z < best) & (u >= 0) & (u <= ul) & (w_ >= 0) & (w_ <= vl)
            best, sid = torch.where(hit, z, best), torch.where(hit, 20 + k, sid)
        ok = sid >= 0
        p = o + torch.where(ok, best, 1.0)[:, None] * d
        lum = scene.colour(sid.clamp(min=0), p) @ torch.tensor([0.299, 0.587, 0.114], device=DEV)
        for cell, amp in ((0.012, 0.12), (0.04, 0.08)):
            i = torch.remainder(torch.floor(p / cell).to(torch.int64), 64)
            lum = lum + amp * (2 * noise[i[:, 0], i[:, 1], i[:, 2]] - 1)
        grey[v] = torch.where(ok, torch.floor(255 * lum.clamp(0, 1) + 0.5), 0.0).to(torch.uint8).reshape(H, W)
    pts = scene.sample(20000, g)[0].to(F64).contiguous()
    targets = [int(round(x)) for x in np.linspace(0, V - 1, case["targets"])]
    return cams, grey, pts, targets


# ------------------------------------------------------------------ the calls

def prepare(case, seed):
    k = case["kind"]
    if k == "train":
        tr = Trainer(_gaussians(case["n"], case["sh"], seed), case["sh"], case["w"], case["h"], cached=case["cached"],
                     lam=case["lam"], extent=4.5)
        tr.lr = 1e-3 * tr.lr  # late in the schedule, so that the model stays what it is over many passes
        cam = _view(case, seed)
        tr.prepare(cam)
        return dict(case=case, tr=tr, cam=cam, target=_image(case["w"], case["h"], seed + 1))
    if k == "render":
        P = _gaussians(case["n"], case["sh"], seed)
        r = Rasterizer(case["n"], case["sh"], case["w"], case["h"], cached=False)
        cam = _view(case, seed)
        r.forward_checked(P, cam)
        return dict(case=case, r=r, P=P, cam=cam)
    if k == "batch":
        cams = _batch_views(case, seed)
        targets = [_image(c["width"], c["height"], seed + 1 + v) for v, c in enumerate(cams)]
        b = BatchedStep(_gaussians(case["n"], case["sh"], seed), case["sh"], cams, targets, cached=case["cached"],
                        extent=4.5)
        b.lr = 1e-3 * b.lr
        b.prepare()
        return dict(case=case, b=b)
    if k in ("seed", "learned"):
        pts, col = _cloud(case["m"], seed)
        return dict(case=case, pts=pts, col=col, w=seed_mlp.load_weights(device=DEV) if k == "learned" else None)
    if k == "seednet":
        t = seed_mlp.SeedNetTrainer(_net_weights(seed), lr=1e-5, max_rows=case["m"])
        return dict(case=case, t=t, batch=_net_batch(case["m"], seed))
    if k == "ba":
        tr = _tracks(case, seed)
        return dict(case=case, pb=ba.BAProblem.from_tracks(tr), st=ba.state(tr["R0"], tr["c0"], tr["P0"]))
    cams, grey, pts, targets = _capture(case, seed)
    mv = MVS(cams, case["w"], case["h"], MVSParams(n_planes=case["planes"]), max_targets=case["targets"])
    return dict(case=case, mv=mv, grey=grey, pts=pts, targets=torch.tensor(targets, dtype=torch.int32, device=DEV),
                points=torch.zeros((3, case["targets"] * case["w"] * case["h"]), device=DEV))


def run(s):
    k = s["case"]["kind"]
    if k == "train":
        tr = s["tr"]
        loss = tr.step(s["cam"], s["target"], check=s["case"]["check"])
        return dict(loss=loss, image=tr.rast.image, grads=tr.grads, params=tr.params, m=tr.m, v=tr.v)
    if k == "render":
        return s["r"].forward(s["P"], s["cam"])
    if k == "batch":
        b = s["b"]
        b.step()
        return dict(losses=b.losses, image=b.image, grads=b.grads, params=b.params, m=b.m, v=b.v)
    if k == "seed":
        return seed_pca(s["pts"], s["col"])
    if k == "learned":
        return seed_mlp.seed_learned(s["pts"], s["col"], s["w"])
    if k == "seednet":
        t = s["t"]
        loss = t.step(*s["batch"])
        return dict(loss=loss, w=t.w, g=t.g, m=t.m, v=t.v)
    if k == "ba":
        pb, st = s["pb"], s["st"]
        if s["case"]["iters"]:
            st, hist, _ = ba.lm(pb, st, iters=s["case"]["iters"])
            return dict(state=st, cost=hist)
        dpose, dpoint = ba.step(pb, st, 1e-3)
        new = ba.apply(pb, st, dpose, dpoint)
        return dict(dpose=dpose, dpoint=dpoint, state=new, cost=ba.cost(pb, new))
    mv = s["mv"]
    mv.prepare(s["grey"], s["pts"])
    depth = mv.depth_maps(s["targets"])
    count = mv.fuse(s["targets"], s["points"])
    return dict(cost=mv.cost, depth=depth, conf=mv.conf, count=count, points=s["points"])


# ------------------------------------------------------------------ the least work

# Splats composited per pixel and tile pairs per Gaussian and view, as these scenes have them.
_SPLATS, _PAIRS = 40, 4


def work(case):
    k = case["kind"]
    if k in ("train", "render", "batch"):
        F = param_rows(case["sh"])
        px = sum(a * b for a, b in MIXED_SIZES[case["first"]:case["first"] + case["views"]]) if k == "batch" \
            else case["w"] * case["h"]
        views = case.get("views", 1)
        flops = px * _SPLATS * 25 + case["n"] * views * 400
        if k == "render":
            return dict(bytes=4 * F * case["n"] + 12 * px, flops=flops)
        # parameters and both moments read and written, gradients written; image written, target read
        return dict(bytes=4 * F * case["n"] * 7 + 24 * px, flops=flops + px * (_SPLATS * 60 + 700) + case["n"] * views * 900)
    if k in ("seed", "learned"):
        # coordinates and colours in, 14 rows out; 16 neighbours' distances and a 3x3 eigenproblem each
        return dict(bytes=case["m"] * (24 + 56), flops=case["m"] * (16 * 40 + 1500 + (26000 if k == "learned" else 0)))
    if k == "seednet":
        return dict(bytes=case["m"] * (256 + 64 + 32) + 13000 * 4 * 7, flops=case["m"] * (6 * 13000 + 800))
    if k == "ba":
        obs = min(8, case["cams"]) * case["points"]
        it = max(1, case["iters"])
        n6 = 6 * case["cams"]
        return dict(bytes=it * (obs * 24 + case["points"] * 24 * 3 + case["cams"] * 96 * 3),
                    flops=it * (obs * (500 + 4.5 * 2 * 108) + n6 ** 3 / 3))
    px = case["w"] * case["h"]
    cells = px * case["targets"] * case["planes"]
    # grey views in, cost volume and depth maps out; the volume is aggregated along four paths
    return dict(bytes=px * case["views"] + cells + px * case["targets"] * 8, flops=cells * (25 + 4 * 8))


# ------------------------------------------------------------------ float64

_SH = ((0.28209479177387814,), (0.4886025119029199,),
       (1.0925484305920792, 0.31539156525252005, 0.5462742152960396),
       (0.5900435899266435, 2.890611442640554, 0.4570457994644658, 0.3731763325901154, 1.445305721320277))


def _basis(deg, d):
    x, y, z = d.unbind(1)
    Y = [torch.full_like(x, _SH[0][0])]
    if deg >= 1:
        c = _SH[1][0]
        Y += [-c * y, c * z, -c * x]
    if deg >= 2:
        a, b, c = _SH[2]
        Y += [a * x * y, -a * y * z, b * (3 * z * z - 1), -a * x * z, c * (x * x - y * y)]
    if deg >= 3:
        a, b, c, e, f = _SH[3]
        Y += [-a * y * (3 * x * x - y * y), b * x * y * z, -c * y * (5 * z * z - 1), e * z * (5 * z * z - 3),
              -c * x * (5 * z * z - 1), f * z * (x * x - y * y), -a * x * (x * x - 3 * y * y)]
    return torch.stack(Y, 1)


def _project64(P, deg, cam):
    """Differentiable 2D records (n, 9) = u, v, A, B, C, opacity, rgb, with
    the depth, the tile rectangle (16 x 16 tiles) and who is visible."""
    n = P.shape[1]
    vm = torch.as_tensor(np.asarray(cam["viewmat"], np.float64), device=DEV)
    Rc, tc = vm[:, :3], vm[:, 3]
    fx, fy, cx, cy, W, H = (cam[k] for k in ("fx", "fy", "cx", "cy", "width", "height"))
    mu = P[0:3].T
    x, y, z = (mu @ Rc.T + tc).unbind(1)
    R = _rotation_of(torch.nn.functional.normalize(P[6:10].T, dim=1))
    M = R * torch.exp(P[3:6].T)[:, None, :]
    lx, ly = 1.3 * W / (2 * fx), 1.3 * H / (2 * fy)
    tx, ty = torch.clamp(x / z, -lx, lx), torch.clamp(y / z, -ly, ly)
    o = torch.zeros_like(z)
    J = torch.stack([fx / z, o, -fx * tx / z, o, fy / z, -fy * ty / z], 1).reshape(n, 2, 3)
    T = (J @ Rc) @ M
    S = T @ T.transpose(1, 2)
    a, b, c = S[:, 0, 0] + 0.3, S[:, 0, 1], S[:, 1, 1] + 0.3
    det = a * c - b * b
    u, v = fx * x / z + cx, fy * y / z + cy
    d = torch.nn.functional.normalize(mu + Rc.T @ tc, dim=1)
    rgb = torch.clamp((_basis(deg, d)[:, :, None] * P[11:].T.reshape(n, -1, 3)).sum(1) + 0.5, min=0)
    rec = torch.cat([torch.stack([u, v, c / det, -b / det, a / det, torch.sigmoid(P[10])], 1), rgb], 1)
    with torch.no_grad():
        mid = 0.5 * (a + c)
        r = torch.ceil(3 * torch.sqrt(mid + torch.sqrt(torch.clamp(mid * mid - det, min=0.1))))
        TX, TY = (W + 15) // 16, (H + 15) // 16
        rect = torch.stack([torch.floor((u - r) / 16).clamp(0, TX), torch.floor((u + r) / 16).clamp(-1, TX - 1),
                            torch.floor((v - r) / 16).clamp(0, TY), torch.floor((v + r) / 16).clamp(-1, TY - 1)], 1)
        ok = (z > 0.2) & (det > 0) & torch.isfinite(u) & torch.isfinite(v)
        rect = torch.where(ok[:, None], rect, torch.tensor([0.0, -1.0, 0.0, -1.0], dtype=F64, device=DEV)).to(torch.int64)
        ok = ok & (rect[:, 0] <= rect[:, 1]) & (rect[:, 2] <= rect[:, 3])
    return rec, z.detach(), rect, ok


def _lists(z, rect, ok, TX, n_tiles):
    """Splat ids of every tile front to back, and each tile's start."""
    ids = ok.nonzero()[:, 0]
    ids = ids[torch.sort(z[ids].float(), stable=True)[1]]
    r = rect[ids]
    w = r[:, 1] - r[:, 0] + 1
    cnt = w * (r[:, 3] - r[:, 2] + 1)
    who = torch.repeat_interleave(torch.arange(ids.numel(), device=DEV), cnt)
    loc = torch.arange(who.numel(), device=DEV) - (torch.cumsum(cnt, 0) - cnt)[who]
    tile = (r[who, 2] + loc // w[who]) * TX + r[who, 0] + loc % w[who]
    tile, order = torch.sort(tile, stable=True)
    start = torch.searchsorted(tile, torch.arange(n_tiles + 1, device=DEV))
    return ids[who[order]], start


def _composite64(rec, ids, start, W, H, dl=None, most=20_000_000):
    """Image of one view; with dl also dL/d(records)."""
    TX, TY = (W + 15) // 16, (H + 15) // 16
    image = torch.zeros((3, TY * 16, TX * 16), dtype=F64, device=DEV)
    grad = None if dl is None else torch.zeros_like(rec)
    if dl is not None:
        pad = torch.zeros_like(image)
        pad[:, :H, :W] = dl
    lens = start[1:] - start[:-1]
    order = torch.sort(lens, descending=True)[1]
    lens_h = lens[order].tolist()
    lane = torch.arange(256, device=DEV)
    at = 0
    while at < len(lens_h) and lens_h[at] > 0:
        L = lens_h[at]
        k = max(1, min(len(lens_h) - at, most // (256 * L)))
        t = order[at:at + k]
        at += k
        j = torch.arange(L, device=DEV)
        live = j[None] < lens[t][:, None]
        idx = ids[(start[t][:, None] + j[None]).clamp(max=ids.numel() - 1)]
        py, px = (t // TX)[:, None] * 16 + lane // 16, (t % TX)[:, None] * 16 + lane % 16
        inside = (px < W) & (py < H)
        S = rec[idx].detach().requires_grad_(dl is not None)
        with torch.set_grad_enabled(dl is not None):
            dx = S[:, None, :, 0] - (px.to(F64) + 0.5)[:, :, None]
            dy = S[:, None, :, 1] - (py.to(F64) + 0.5)[:, :, None]
            power = -0.5 * (S[:, None, :, 2] * dx * dx + S[:, None, :, 4] * dy * dy) - S[:, None, :, 3] * dx * dy
            al = torch.clamp(S[:, None, :, 5] * torch.exp(torch.clamp(power, max=0)), max=0.99)
            use = (power <= 0) & (al >= 1.0 / 255.0) & live[:, None] & inside[:, :, None]
            al = torch.where(use, al, 0.0)
            with torch.no_grad():
                going = torch.cumprod(1 - al, 2) >= 1e-4
            al = torch.where(going, al, 0.0)
            q = torch.cumprod(1 - al, 2)
            wgt = al * torch.cat([torch.ones_like(q[:, :, :1]), q[:, :, :-1]], 2)
            c = wgt @ S[:, :, 6:9]
            if dl is not None:
                g = torch.stack([pad[ch][py, px] for ch in range(3)], -1)
                (gs,) = torch.autograd.grad((c * g).sum(), S)
                grad.index_add_(0, idx.reshape(-1), (gs * live[:, :, None]).reshape(-1, rec.shape[1]))
        for ch in range(3):
            image[ch][py, px] = c[:, :, ch].detach()
    return image[:, :H, :W], grad


def _loss64(x, y, lam):
    """L1 / D-SSIM loss and its gradient by x."""
    x = x.clone().requires_grad_(True)
    loss = (x - y).abs().mean()
    if lam > 0:
        d = torch.arange(11, dtype=F64) - 5
        win = torch.exp(-d * d / 4.5)
        win = (win / win.sum()).tolist()
        H, W = x.shape[1:]

        def blur(a):
            p = torch.nn.functional.pad(a, (5, 5, 0, 0))
            a = sum(win[i] * p[:, :, i:i + W] for i in range(11))
            p = torch.nn.functional.pad(a, (0, 0, 5, 5))
            return sum(win[i] * p[:, i:i + H] for i in range(11))
        mx, my = blur(x), blur(y)
        vx, vy, cxy = blur(x * x) - mx * mx, blur(y * y) - my * my, blur(x * y) - mx * my
        ssim = (2 * mx * my + 1e-4) * (2 * cxy + 9e-4) / ((mx * mx + my * my + 1e-4) * (vx + vy + 9e-4))
        loss = (1 - lam) * loss + lam * (1 - ssim.mean())
    (g,) = torch.autograd.grad(loss, x)
    return loss.detach(), g


def _view64(P32, deg, cam, target=None, lam=0.0):
    """(image, loss, dL/d(parameters)) of one view; the image alone without a target."""
    W, H = cam["width"], cam["height"]
    TX, TY = (W + 15) // 16, (H + 15) // 16
    P = P32.to(F64).requires_grad_(target is not None)
    rec, z, rect, ok = _project64(P, deg, cam)
    ids, start = _lists(z, rect, ok, TX, TX * TY)
    img, _ = _composite64(rec.detach(), ids, start, W, H)
    if target is None:
        return img, None, None
    loss, dl = _loss64(img, target.to(F64), lam)
    _, g2 = _composite64(rec.detach(), ids, start, W, H, dl)
    g2 = torch.where(ok[:, None], g2, 0.0)
    (g,) = torch.autograd.grad(rec, P, torch.where(ok[:, None], g2, torch.zeros_like(g2)))
    return img, loss, torch.nan_to_num(g)


def _adam64(p, g, lr, b1, b2, eps):
    """The first Adam step; lr a number or one rate per row."""
    b1, b2 = float(np.float32(b1)), float(np.float32(b2))
    m, v = (1 - b1) * g, (1 - b2) * g * g
    return p.to(F64) - lr * (m / (1 - b1)) / (torch.sqrt(v / (1 - b2)) + eps), m, v


def _neighbours64(pts):
    """Squared distances and indices of every point's 16 nearest others."""
    p = pts.T.to(F64)
    m = p.shape[0]
    d2, nb = [], []
    step = max(1, 300_000_000 // m)
    for s in range(0, m, step):
        q = p[s:s + step]
        d = (q[:, 0, None] - p[None, :, 0]) ** 2 + (q[:, 1, None] - p[None, :, 1]) ** 2 + \
            (q[:, 2, None] - p[None, :, 2]) ** 2
        d[torch.arange(q.shape[0], device=DEV), torch.arange(s, s + q.shape[0], device=DEV)] = math.inf
        v, i = torch.topk(d, 16, dim=1, largest=False)
        d2.append(v)
        nb.append(i)
    return torch.cat(d2), torch.cat(nb), p


def _eigen64(A):
    """Eigenvalues (diagonal) and vectors (columns) of symmetric 3x3 matrices by cyclic Jacobi rotations."""
    A = A.clone()
    V = torch.eye(3, dtype=F64, device=DEV).expand_as(A).clone()
    for _ in range(10):
        for p, q in ((0, 1), (0, 2), (1, 2)):
            off = A[:, p, q]
            th = (A[:, q, q] - A[:, p, p]) / (2 * off)
            t = torch.where(th >= 0, 1.0, -1.0) / (th.abs() + torch.sqrt(th * th + 1))
            t = torch.where(off.abs() > 1e-300, t, 0.0)
            c = 1 / torch.sqrt(t * t + 1)
            G = torch.eye(3, dtype=F64, device=DEV).expand_as(A).clone()
            G[:, p, p], G[:, q, q], G[:, p, q], G[:, q, p] = c, c, t * c, -t * c
            A = G.transpose(1, 2) @ A @ G
            V = V @ G
    return torch.diagonal(A, dim1=1, dim2=2), V


def _quaternion64(R):
    """Unit quaternions (w, x, y, z), the branch by the largest of the trace and the diagonal."""
    d = torch.diagonal(R, dim1=1, dim2=2)
    tr = d.sum(1)
    r = lambda a, b: R[:, a, b]  # noqa: E731
    w = torch.stack([1 + tr, r(2, 1) - r(1, 2), r(0, 2) - r(2, 0), r(1, 0) - r(0, 1)], 1)
    x = torch.stack([r(2, 1) - r(1, 2), 1 + d[:, 0] - d[:, 1] - d[:, 2], r(0, 1) + r(1, 0), r(0, 2) + r(2, 0)], 1)
    y = torch.stack([r(0, 2) - r(2, 0), r(0, 1) + r(1, 0), 1 - d[:, 0] + d[:, 1] - d[:, 2], r(1, 2) + r(2, 1)], 1)
    z = torch.stack([r(1, 0) - r(0, 1), r(0, 2) + r(2, 0), r(1, 2) + r(2, 1), 1 - d[:, 0] - d[:, 1] + d[:, 2]], 1)
    best = torch.argmax(torch.cat([tr[:, None], d], 1), 1)
    q = torch.stack([w, x, y, z], 1)[torch.arange(R.shape[0], device=DEV), best]
    return torch.nn.functional.normalize(q, dim=1)


def _disc64(pts, col):
    d2, nb, p = _neighbours64(pts)
    P = p[nb]
    D = P - P.mean(1, keepdim=True)
    C = D.transpose(1, 2) @ D / 16
    val, V = _eigen64(C)
    n = torch.nn.functional.normalize(V[torch.arange(V.shape[0], device=DEV), :, val.argmin(1)], dim=1)
    st = torch.sqrt(d2[:, :3]).mean(1)
    sg = torch.where(n[:, 2] >= 0, 1.0, -1.0)
    a = -1 / (sg + n[:, 2])
    b = n[:, 0] * n[:, 1] * a
    R = torch.stack([1 + sg * n[:, 0] ** 2 * a, b, n[:, 0], sg * b, sg + n[:, 1] ** 2 * a, n[:, 1],
                     -sg * n[:, 0], -n[:, 1], n[:, 2]], 1).reshape(-1, 3, 3)
    out = torch.empty((14, p.shape[0]), dtype=F64, device=DEV)
    out[0:3] = p.T
    out[3] = out[4] = torch.log(st)
    out[5] = torch.log(0.1 * st)
    out[6:10] = _quaternion64(R).T
    out[10] = math.log(0.1 / 0.9)
    out[11:14] = (col.to(F64) - 0.5) / _SH[0][0]
    return out, st, P - p[:, None], C, val, V


def _layers(w):
    w = w.to(F64)
    out, at = [], 0
    for o, i in ((64, 64), (64, 64), (64, 64), (8, 64)):
        out.append((w[at:at + o * i].reshape(o, i), w[at + o * i:at + o * i + o]))
        at += o * i + o
    return out


def _net64(w, x):
    h = x.to(F64)
    L = _layers(w)
    for W, b in L[:3]:
        h = torch.nn.functional.gelu(h @ W.T + b)
    return h @ L[3][0].T + L[3][1]


def _learned64(pts, col, w):
    pca, st, off, C, val, V = _disc64(pts, col)
    m = pts.shape[1]
    order = torch.argsort(val, dim=1, descending=True)
    e = [torch.nn.functional.normalize(V[torch.arange(m, device=DEV), :, order[:, c]], dim=1) for c in range(2)]
    e = [v * torch.where(((off * v[:, None]).sum(2) ** 3).sum(1) < 0, -1.0, 1.0)[:, None] for v in e]
    e.append(torch.cross(e[0], e[1], dim=1))
    R = torch.stack(e, 2)
    x = torch.zeros((m, 64), dtype=F64, device=DEV)
    x[:, :48] = ((off @ R) / st[:, None, None]).reshape(m, 48)
    x[:, 48:57] = (R.transpose(1, 2) @ C @ R / (st * st)[:, None, None]).reshape(m, 9)
    y = _net64(w, x)
    qn = y[:, 3:7].norm(dim=1, keepdim=True)
    qo = y[:, 3:7] / qn
    s = torch.stack([torch.log(st), torch.log(st), torch.log(0.1 * st)], 1) + y[:, :3]
    Ro = _rotation_of(qo)
    c = Ro[torch.arange(m, device=DEV), 2, s.argmin(1)].abs()
    back = (y[:, :3].abs().amax(1) > 2) | (c < 0.5) | (qn[:, 0] < 1e-6)
    a, b = _quaternion64(R), qo
    q = torch.stack([a[:, 0] * b[:, 0] - a[:, 1] * b[:, 1] - a[:, 2] * b[:, 2] - a[:, 3] * b[:, 3],
                     a[:, 0] * b[:, 1] + b[:, 0] * a[:, 1] + a[:, 2] * b[:, 3] - a[:, 3] * b[:, 2],
                     a[:, 0] * b[:, 2] + b[:, 0] * a[:, 2] + a[:, 3] * b[:, 1] - a[:, 1] * b[:, 3],
                     a[:, 0] * b[:, 3] + b[:, 0] * a[:, 3] + a[:, 1] * b[:, 2] - a[:, 2] * b[:, 1]])
    out = pca.clone()
    out[3:6], out[6:10], out[10] = s.T, q, math.log(0.1 / 0.9) + y[:, 7]
    return torch.where(back[None], pca, out)


def _net_step64(w32, batch, lr):
    x, base, t = (a.to(F64) for a in batch)
    m = x.shape[0]
    w = w32.to(F64).requires_grad_(True)
    y = _net64(w, x)
    R = base[:, :9].reshape(m, 3, 3) @ _rotation_of(torch.nn.functional.normalize(y[:, 3:7], dim=1))
    L = R @ torch.diag_embed(2 * (base[:, 9:12] + y[:, :3])) @ R.transpose(1, 2)
    M = torch.stack([t[:, 0], t[:, 3], t[:, 4], t[:, 3], t[:, 1], t[:, 5], t[:, 4], t[:, 5], t[:, 2]], 1).reshape(m, 3, 3)
    loss = (((L - M) ** 2).sum((1, 2)) + (math.log(1 / 9) + y[:, 7] - t[:, 6]) ** 2).mean()
    (g,) = torch.autograd.grad(loss, w)
    p, am, av = _adam64(w32, g, lr, 0.9, 0.999, 1e-8)
    return dict(loss=loss.detach().reshape(1), w=p, g=g, m=am, v=av)


class _Adjust64:
    """Residuals and damped normal equations of a track set."""

    def __init__(self, tr, delta=2.0):
        t = lambda a: torch.as_tensor(a, device=DEV)  # noqa: E731
        self.cam, self.pt = t(tr["obs_cam"].astype(np.int64)), t(tr["obs_pt"].astype(np.int64))
        self.uv, self.f, self.cc = t(tr["obs_uv"]), tr["fx"], t(np.array([tr["cx"], tr["cy"]]))
        self.delta, self.axis = delta, tr["gauge_axis"]
        self.state = (t(tr["R0"]), t(tr["c0"]), t(tr["P0"]))
        self.C, self.M = tr["R0"].shape[0], tr["P0"].shape[0]
        start = torch.searchsorted(self.pt, torch.arange(self.M, device=DEV))
        self.slot = torch.arange(self.pt.numel(), device=DEV) - start[self.pt]

    def residual(self, st):
        R, c, P = st
        d = P[self.pt] - c[self.cam]
        x = (R[self.cam] @ d[:, :, None])[:, :, 0]
        r = self.f * x[:, :2] / x[:, 2:] + self.cc - self.uv
        return r, x, d

    def cost(self, st):
        n = self.residual(st)[0].norm(dim=1)
        return torch.where(n <= self.delta, n * n, 2 * self.delta * n - self.delta ** 2).sum().reshape(1)

    def step(self, st, lam):
        r, x, d = self.residual(st)
        n = r.norm(dim=1)
        w = torch.where(n <= self.delta, 1.0, self.delta / n)
        iz, z = 1 / x[:, 2], torch.zeros_like(n)
        A = torch.stack([self.f * iz, z, -self.f * x[:, 0] * iz * iz, z, self.f * iz, -self.f * x[:, 1] * iz * iz],
                        1).reshape(-1, 2, 3)
        Jp = A @ st[0][self.cam]
        X = torch.stack([z, -d[:, 2], d[:, 1], d[:, 2], z, -d[:, 0], -d[:, 1], d[:, 0], z], 1).reshape(-1, 3, 3)
        Jt = torch.cat([-(Jp @ X), -Jp], 2)
        wt = w[:, None, None]
        Hpp = torch.zeros((self.M, 3, 3), dtype=F64, device=DEV).index_add_(0, self.pt, wt * Jp.transpose(1, 2) @ Jp)
        bp = torch.zeros((self.M, 3), dtype=F64, device=DEV).index_add_(
            0, self.pt, -(w[:, None] * (Jp.transpose(1, 2) @ r[:, :, None])[:, :, 0]))
        Htt = torch.zeros((self.C, 6, 6), dtype=F64, device=DEV).index_add_(0, self.cam, wt * Jt.transpose(1, 2) @ Jt)
        bt = torch.zeros((self.C, 6), dtype=F64, device=DEV).index_add_(
            0, self.cam, -(w[:, None] * (Jt.transpose(1, 2) @ r[:, :, None])[:, :, 0]))
        Hpp = Hpp + lam * torch.diag_embed(torch.diagonal(Hpp, dim1=1, dim2=2))
        Htt = Htt + lam * torch.diag_embed(torch.diagonal(Htt, dim1=1, dim2=2))
        inv = torch.linalg.inv(Hpp)
        B = wt * Jt.transpose(1, 2) @ Jp
        T = B @ inv[self.pt]
        g = bt.index_add(0, self.cam, -(T @ bp[self.pt][:, :, None])[:, :, 0])
        S = torch.zeros((self.C * self.C, 36), dtype=F64, device=DEV)
        S[torch.arange(self.C, device=DEV) * (self.C + 1)] = Htt.reshape(-1, 36)
        # every pair of observations of a point: observation o with the one in slot k of its point
        k_max = int(self.slot.max()) + 1
        table = torch.full((self.M, k_max), -1, dtype=torch.int64, device=DEV)
        table[self.pt, self.slot] = torch.arange(self.pt.numel(), device=DEV)
        for k in range(k_max):
            o2 = table[self.pt, k]
            on = o2 >= 0
            o2 = o2[on]
            S.index_add_(0, self.cam[on] * self.C + self.cam[o2], -(T[on] @ B[o2].transpose(1, 2)).reshape(-1, 36))
        S = S.reshape(self.C, self.C, 6, 6).permute(0, 2, 1, 3).reshape(6 * self.C, 6 * self.C)
        free = torch.tensor([i for i in range(6, 6 * self.C) if i != 9 + self.axis])
        dt = torch.zeros(6 * self.C, dtype=F64)
        dt[free] = torch.linalg.solve(S.cpu()[free][:, free], g.reshape(-1).cpu()[free])
        dt = dt.to(DEV).reshape(self.C, 6)
        back = bp.index_add(0, self.pt, -(B.transpose(1, 2) @ dt[self.cam][:, :, None])[:, :, 0])
        return dt, (inv @ back[:, :, None])[:, :, 0]

    def apply(self, st, dt, dp):
        return (st[0] @ _exp_so3(dt[:, :3]), st[1] + dt[:, 3:], st[2] + dp)


def _adjust64(case, tr):
    a = _Adjust64(tr)
    st = a.state
    flat = lambda s: (s[0].reshape(-1, 9), s[1], s[2])  # noqa: E731
    if not case["iters"]:
        dt, dp = a.step(st, 1e-3)
        new = a.apply(st, dt, dp)
        return dict(dpose=dt, dpoint=dp, state=flat(new), cost=a.cost(new))
    lam, hist = 1e-3, [float(a.cost(st))]
    for _ in range(case["iters"]):
        new = a.apply(st, *a.step(st, lam))
        f = float(a.cost(new))
        if f < hist[-1]:
            st, lam = new, lam / 10
        else:
            lam *= 10
        hist.append(min(f, hist[-1]))
    return dict(state=flat(st), cost=hist)


def _depth_range64(cam, pts, W, H):
    vm = np.asarray(cam["viewmat"], np.float64)
    x = pts.cpu().numpy() @ vm[:, :3].T + vm[:, 3]
    z = x[:, 2]
    u, v = cam["fx"] * x[:, 0] / z + cam["cx"], cam["fy"] * x[:, 1] / z + cam["cy"]
    z = np.sort(z[(z > 0) & (u >= -0.5) & (u < W - 0.5) & (v >= -0.5) & (v < H - 0.5)])
    if not z.size:
        return 0.0, 0.0
    q = []
    for p in (0.05, 0.95):
        h = (z.size - 1) * p
        i = int(math.floor(h))
        j = min(i + 1, z.size - 1)
        q.append(z[i] + (z[j] - z[i]) * (h - i))
    return 0.5 * q[0], 1.5 * q[1]


def _census(grey):
    g = torch.nn.functional.pad(grey[:, None].float(), (3, 3, 3, 3), mode="replicate")[:, 0]
    H, W = grey.shape[1:]
    c, out, b = grey.float(), torch.zeros(grey.shape, dtype=torch.int64, device=DEV), 0
    for dy in range(7):
        for dx in range(7):
            if (dy, dx) != (3, 3):
                out |= (g[:, dy:dy + H, dx:dx + W] < c).to(torch.int64) << b
                b += 1
    return out


def _popcount(v):
    n = torch.zeros(v.shape, dtype=torch.int16, device=DEV)
    table = torch.tensor([bin(i).count("1") for i in range(4096)], dtype=torch.int16, device=DEV)
    for s in range(0, 48, 12):
        n += table[(v >> s) & 4095]
    return n


def _stereo64(case, cams, grey, pts, targets):
    W, H, D = case["w"], case["h"], case["planes"]
    census = _census(grey)
    vm = [np.asarray(c["viewmat"], np.float64) for c in cams]
    centre = [-m[:, :3].T @ m[:, 3] for m in vm]
    cost = torch.empty((len(targets), H, W, D), dtype=torch.int16, device=DEV)
    invs = []
    ys, xs = torch.meshgrid(torch.arange(H, device=DEV, dtype=F64), torch.arange(W, device=DEV, dtype=F64), indexing="ij")
    for n, t in enumerate(targets):
        score = []
        for c in range(len(cams)):
            base = float(np.linalg.norm(centre[c] - centre[t]))
            al = math.acos(max(-1.0, min(1.0, float(vm[t][2, :3] @ vm[c][2, :3]))))
            score.append(-1.0 if c == t else math.exp(-(base - 0.5) ** 2 / (2 * 0.25 ** 2)) * max(al / math.radians(5), 1.0))
        r = int(np.argmax(score))
        lo, hi = _depth_range64(cams[t], pts, W, H)
        far = 1 / hi
        step = (1 / lo - far) / (D - 1)
        invs.append((far, step))
        # the sweep is defined in float32 from rounded pose, planes and rays
        M = (vm[r][:, :3] @ vm[t][:, :3].T)
        mt = (vm[r][:, 3] - M @ vm[t][:, 3]).astype(np.float32).tolist()
        M = M.astype(np.float32).tolist()
        a = ((xs - cams[t]["cx"]) / cams[t]["fx"]).float()
        b = ((ys - cams[t]["cy"]) / cams[t]["fy"]).float()
        f, cx, cy = cams[r]["fx"], cams[r]["cx"], cams[r]["cy"]
        for k in range(D):
            d = float(np.float32(1 / (far + k * step)))
            X, Y = d * a, d * b
            x, y, z = (M[i][0] * X + M[i][1] * Y + float(np.float32(M[i][2]) * np.float32(d)) + mt[i] for i in range(3))
            u, v = torch.floor(f * (x / z) + cx + 0.5), torch.floor(f * (y / z) + cy + 0.5)
            ok = (z > 0) & (u >= 0) & (u <= W - 1) & (v >= 0) & (v <= H - 1)
            at = torch.where(ok, v * W + u, 0.0).to(torch.int64) if W * H < (1 << 24) else \
                torch.where(ok, v, 0.0).to(torch.int64) * W + torch.where(ok, u, 0.0).to(torch.int64)
            ham = _popcount(census[t] ^ census[r].reshape(-1)[at])
            cost[n, :, :, k] = torch.where(ok, ham, torch.tensor(48, dtype=torch.int16, device=DEV))
    total = torch.zeros_like(cost)
    for axis in (2, 1):
        for order in (range(cost.shape[axis]), range(cost.shape[axis] - 1, -1, -1)):
            L = None
            for i in order:
                c = cost.select(axis, i)
                if L is None:
                    L = c.clone()
                else:
                    m = L.amin(2, keepdim=True)
                    best = torch.minimum(L, m + 32)
                    best[:, :, 1:] = torch.minimum(best[:, :, 1:], L[:, :, :-1] + 4)
                    best[:, :, :-1] = torch.minimum(best[:, :, :-1], L[:, :, 1:] + 4)
                    L = c + best - m
                total.select(axis, i).add_(L)
    s1, kw = total.min(3)
    planes = torch.arange(D, device=DEV)
    depth = torch.empty(s1.shape, dtype=F64, device=DEV)
    conf = torch.empty_like(depth)
    points = torch.zeros((3, s1.numel()), dtype=F64, device=DEV)
    at = 0
    for n, t in enumerate(targets):
        far_off = (planes - kw[n][..., None]).abs() >= 2
        s2 = torch.where(far_off, total[n], torch.tensor(32767, dtype=torch.int16, device=DEV)).amin(2).to(F64)
        s = s1[n].to(F64)
        below = total[n].gather(2, (kw[n] - 1).clamp(min=0)[..., None])[..., 0].to(F64)
        above = total[n].gather(2, (kw[n] + 1).clamp(max=D - 1)[..., None])[..., 0].to(F64)
        keep = (kw[n] > 0) & (kw[n] < D - 1) & (s2 > 0) & (s <= 0.6 * s2)
        den = below - 2 * s + above
        delta = torch.where(den > 0, (below - above) / (2 * den), 0.0)
        depth[n] = torch.where(keep, 1 / (invs[n][0] + (kw[n] + delta) * invs[n][1]), 0.0)
        conf[n] = torch.where(s2 > 0, 1 - s / s2, 0.0)
        m = torch.as_tensor(vm[t], device=DEV)
        z = depth[n][keep]
        X = torch.stack([z * (xs[keep] - cams[t]["cx"]) / cams[t]["fx"], z * (ys[keep] - cams[t]["cy"]) / cams[t]["fy"], z])
        points[:, at:at + z.numel()] = m[:, :3].T @ (X - m[:, 3:])
        at += z.numel()
    return dict(cost=None, depth=depth, conf=conf, count=None, points=points)


def exact(case, seed):
    k = case["kind"]
    if k == "train":
        P = _gaussians(case["n"], case["sh"], seed)
        img, loss, g = _view64(P, case["sh"], _view(case, seed), _image(case["w"], case["h"], seed + 1), case["lam"])
        lr = torch.as_tensor(1e-3 * learning_rates(case["sh"], 4.5).astype(np.float64), device=DEV)[:, None]
        p, m, v = _adam64(P, g, lr, 0.9, 0.999, 1e-15)
        return dict(loss=loss.reshape(1), image=img, grads=g, params=p, m=m, v=v)
    if k == "render":
        return _view64(_gaussians(case["n"], case["sh"], seed), case["sh"], _view(case, seed))[0]
    if k == "batch":
        P = _gaussians(case["n"], case["sh"], seed)
        losses, images, grads = [], [], 0.0
        for v, cam in enumerate(_batch_views(case, seed)):
            img, loss, g = _view64(P, case["sh"], cam, _image(cam["width"], cam["height"], seed + 1 + v), 0.2)
            losses.append(loss)
            images.append(img.reshape(-1))
            grads = grads + g
        lr = torch.as_tensor(1e-3 * learning_rates(case["sh"], 4.5).astype(np.float64), device=DEV)[:, None]
        p, m, v = _adam64(P, grads, lr, 0.9, 0.999, 1e-15)
        return dict(losses=torch.stack(losses), image=torch.cat(images), grads=grads, params=p, m=m, v=v)
    if k == "seed":
        return _disc64(*_cloud(case["m"], seed))[0]
    if k == "learned":
        return _learned64(*_cloud(case["m"], seed), seed_mlp.load_weights(device=DEV)), None
    if k == "seednet":
        return _net_step64(_net_weights(seed), _net_batch(case["m"], seed), 1e-5)
    if k == "ba":
        return _adjust64(case, _tracks(case, seed))
    return _stereo64(case, *_capture(case, seed))
