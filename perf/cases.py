"""Performance cases: the calls that a relocalization program makes.

Every case is a dict of plain values with a "kind":

  render        forward maps of P poses (Renderer.render / render_into)
  refine        one pose-refinement step: render, residual and pose gradient
  train         render and the gradients of every Gaussian parameter
  match         coarse-to-fine matching of query and rendered feature maps
  solve         the RANSAC pose solve from 2D-3D correspondences
  significance  scoring of the Gaussians against a batch of training views

Inputs are seeded and drawn on the device: Gaussians on a heightfield with box
buildings seen from a downward-looking camera, N(0, 1) feature maps, pixel
correspondences with noise and outliers.  exact() evaluates the same
definitions in 64 bits with plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2507_15683_amd as hg

DEV = "cuda"
F64 = torch.float64
LAYERS = 15  # Gaussians blended per pixel at the scenes' density of about 1 per square metre


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # a preview render of a small scene through the checked call: latency and launches
        dict(name="render_small", kind="render", n=20_000, extent=200.0, sh=0, D=0, W=256, H=192, P=1, alt=120.0,
             spatial=False, checked=True, bf16=False, parts=0),
        # the dense stage's render of one query view: colour, depth and 32-channel features at full resolution
        dict(name="render_1080p", kind="render", n=1_000_000, extent=1000.0, sh=3, D=32, W=1920, H=1080, P=1,
             alt=200.0, spatial=True, checked=False, bf16=False, parts=0),
        # a few candidate views of odd size with bfloat16 feature maps (the matcher's input type)
        dict(name="render_odd_bf16", kind="render", n=300_000, extent=550.0, sh=2, D=16, W=333, H=217, P=6,
             alt=150.0, spatial=True, checked=False, bf16=True, parts=0),
        # one candidate pose refined at the coarse level: the shortest step of the refinement loop
        dict(name="refine_one", kind="refine", n=1_000_000, extent=1000.0, sh=3, D=32, W=480, H=270, P=1, alt=200.0,
             spatial=True, parts=0),
        # sixteen query poses at the coarse level of a partitioned scene
        dict(name="refine_16_parts", kind="refine", n=2_000_000, extent=2000.0, sh=0, D=32, W=480, H=270, P=16,
             alt=200.0, spatial=True, parts=16),
        # sixty-four candidate poses of one query at half resolution: the batched refinement step
        dict(name="refine_64", kind="refine", n=1_000_000, extent=1000.0, sh=3, D=32, W=960, H=540, P=64, alt=200.0,
             spatial=True, parts=0),
        # fine-tuning the scene on one view: gradients of all Gaussian parameters and the pose
        dict(name="train_vga", kind="train", n=200_000, extent=447.0, sh=0, D=32, W=640, H=480, P=1, alt=120.0,
             spatial=True, parts=0),
        # matching of a 1920x1080 query with a rendered view (coarse maps at 1/8)
        dict(name="match_1080p", kind="match", D=32, Hc=135, Wc=240, fine=True),
        # matching at the coarse refinement level, an odd number of positions
        dict(name="match_odd", kind="match", D=32, Hc=33, Wc=59, fine=True),
        # pose from every fine match of a 1920x1080 view
        dict(name="solve_640k", kind="solve", m=640_000, hyps=1024, outliers=0.5),
        # pose from the matches of a small view
        dict(name="solve_small", kind="solve", m=5_001, hyps=256, outliers=0.3),
        # one batch of training views of the landmark scoring
        dict(name="significance_64", kind="significance", n=1_000_000, extent=1000.0, sh=3, D=32, W=960, H=540, P=64,
             alt=200.0, spatial=True, parts=0, layout="planar"),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    """One more case of the listed ranges."""
    kind = rng.choice(["render", "refine", "train", "match", "solve", "significance"])
    if kind == "match":
        Hc = int(_log(rng, 9, 135))
        return dict(kind=kind, D=rng.choice([8, 16, 32, 64]), Hc=Hc, Wc=int(Hc * rng.uniform(1.2, 1.7)) + 1,
                    fine=rng.random() < 0.8)
    if kind == "solve":
        return dict(kind=kind, m=int(_log(rng, 500, 640_000)), hyps=int(_log(rng, 64, 1024)),
                    outliers=round(rng.uniform(0.2, 0.5), 3))
    W = int(_log(rng, 640 if kind == "train" else 240, 1920))  # scenes are tuned at the training images' size
    H = int(W * rng.uniform(0.5, 0.8))
    n = int(_log(rng, 20_000, 1_000_000))
    most = max(1, min(64, 16_000_000 // (W * H)))
    c = dict(kind=kind, n=n, extent=round(math.sqrt(n), 1), sh=rng.choice([0, 1, 2, 3]),
             D=rng.choice([0, 8, 16, 32, 32, 64]), W=W, H=H, P=min(most, int(_log(rng, 1, 64.99))),
             alt=round(rng.uniform(100.0, 300.0), 1), spatial=rng.random() < 0.75, parts=rng.choice([0, 0, 4, 9]))
    if kind == "render":
        c.update(checked=rng.random() < 0.5, bf16=c["D"] > 0 and rng.random() < 0.4)
    elif kind == "train":
        c.update(P=min(c["P"], 4), alt=round(rng.uniform(100.0, 160.0), 1))
    elif kind == "significance":
        c["D"] = c["D"] or 32
        c["layout"] = rng.choice(["planar", "interleaved"])
    return c


# ------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + 17)


def _terrain(x, y):
    return 8.0 * torch.sin(x / 23.0) * torch.cos(y / 31.0)


class _HostScene:
    pass


def _points(case, g):
    """Means on the heightfield (90 %) and on the walls and roofs of boxes of 50 points each (10 %)."""
    n, ext = case["n"], case["extent"]
    u = lambda m, lo, hi: torch.rand(m, generator=g, device=DEV, dtype=F64) * (hi - lo) + lo  # noqa: E731
    nb = n // 500
    nt = n - 50 * nb
    x, y = u(nt, -ext / 2, ext / 2), u(nt, -ext / 2, ext / 2)
    z = _terrain(x, y) + 0.5 * torch.randn(nt, generator=g, device=DEV, dtype=F64)
    parts = [torch.stack([x, y, z], 1)]
    if nb:
        rep = lambda t: t.repeat_interleave(50)  # noqa: E731
        m = 50 * nb
        cx, cy = u(nb, -ext / 2, ext / 2), u(nb, -ext / 2, ext / 2)
        sx, sy, hz, yaw = rep(u(nb, 8, 30)), rep(u(nb, 8, 30)), rep(u(nb, 5, 40)), rep(u(nb, 0, math.pi / 2))
        base, cx, cy = rep(_terrain(cx, cy)), rep(cx), rep(cy)
        face = torch.randint(0, 5, (m,), generator=g, device=DEV)
        a, b, h = u(m, -0.5, 0.5), u(m, -0.5, 0.5), u(m, 0, 1)
        side = torch.where((face == 0) | (face == 2), -0.5, 0.5).to(F64)
        lx = torch.where((face == 0) | (face == 1) | (face == 4), a * sx, side * sx)
        ly = torch.where((face == 2) | (face == 3), a * sy, torch.where(face == 4, b * sy, (face.to(F64) - 0.5) * sy))
        lz = torch.where(face == 4, hz, h * hz)
        c, s = torch.cos(yaw), torch.sin(yaw)
        parts.append(torch.stack([cx + c * lx - s * ly, cy + s * lx + c * ly, base + lz], 1))
    return torch.cat(parts).float()


def _scene(case, seed):
    """The case's scene as a GaussianScene: partitions are square cells, Gaussians in Morton order when spatial."""
    g = _gen(seed)
    n, D, K = case["n"], case["D"], (case["sh"] + 1) ** 2
    means = _points(case, g)
    offsets = None
    if case["parts"]:
        side = int(round(math.sqrt(case["parts"])))
        cell = ((means[:, :2] / case["extent"] + 0.5) * side).long().clamp(0, side - 1)
        cell = cell[:, 1] * side + cell[:, 0]
        means = means[torch.sort(cell, stable=True).indices]
        offsets = torch.zeros(side * side + 1, dtype=torch.int64, device=DEV)
        offsets[1:] = torch.cumsum(torch.bincount(cell, minlength=side * side), 0)
    if case["spatial"]:
        perm = hg.spatial_order(means.cpu().numpy(), None if offsets is None else offsets.cpu().numpy())
        means = means[torch.from_numpy(perm).to(DEV)]
    rn = lambda *s: torch.randn(*s, generator=g, device=DEV)  # noqa: E731
    sh = 0.2 * rn(n, K, 3)
    sh[:, 0] = (torch.rand(n, 3, generator=g, device=DEV) * 2 - 1) * math.sqrt(math.pi)
    quats = rn(n, 4)
    feat = None
    if D:
        feat = rn(n, D)
        feat = (feat / feat.norm(dim=1, keepdim=True)).bfloat16()
    sc = hg.GaussianScene(means.contiguous(), 0.3 * rn(n, 3) - 0.5, quats / quats.norm(dim=1, keepdim=True),
                          torch.sigmoid(rn(n)), sh, case["sh"], feat)
    if offsets is not None:
        host = _HostScene()
        host.means, host.log_scales, host.quats, host.opacities, host.sh = (
            t.cpu().numpy() for t in (sc.means, sc.log_scales, sc.quats, sc.opacities, sc.sh))
        host.sh_degree, host.feat, host.part_offsets = case["sh"], None, offsets.cpu().numpy()
        sc.part_offsets = offsets
        sc.part_bounds = torch.from_numpy(hg.host_partition_bounds(host)).to(DEV)
    return sc


def _rot(v):
    x, y, z = v
    return torch.linalg.matrix_exp(torch.tensor([[0, -z, y], [z, 0, -x], [-y, x, 0]], dtype=F64))


def _poses(case, seed, count=None):
    """World-to-camera poses (count x 12): one downward view, the others moved by N(0, 5 m) and N(0, 3 degrees)."""
    r = np.random.default_rng(int(seed) * 31 + 5)
    span = 0.2 * case["extent"]
    ang, d = math.radians(r.uniform(0.0, 20.0)), r.uniform(0, 2 * math.pi)
    cx, cy = r.uniform(-span, span, 2)
    C = np.array([cx, cy, 8.0 * math.sin(cx / 23.0) * math.cos(cy / 31.0) + case["alt"]])
    R0 = _rot((0.0, 0.0, r.uniform(0, 2 * math.pi))) @ _rot((ang * math.cos(d), ang * math.sin(d), 0.0))
    R0 = R0 @ torch.diag(torch.tensor([1.0, -1.0, -1.0], dtype=F64))
    out = []
    for k in range(count or case["P"]):
        Rk = (_rot(np.deg2rad(r.normal(0, 3.0, 3))) if k else torch.eye(3, dtype=F64)) @ R0
        Ck = torch.from_numpy(C + (r.normal(0, 5.0, 3) if k else 0.0))
        out.append(torch.cat([Rk.T, -(Rk.T @ Ck)[:, None]], 1).reshape(12))
    return torch.stack(out).float().to(DEV)


def _camera(case):
    f = case["W"] / 1.28
    return hg.Intrinsics(f, f, case["W"] / 2.0, case["H"] / 2.0, case["W"], case["H"])


def _match_maps(case, seed):
    """Query and rendered maps: the rendered one is the query's moved by a few pixels with N(0, 0.3) noise."""
    g = _gen(seed)
    D, Hf, Wf = case["D"], 8 * case["Hc"], 8 * case["Wc"]
    q = torch.randn(D, Hf, Wf, generator=g, device=DEV)
    r = torch.roll(q, (-6, 11), (1, 2)) + 0.3 * torch.randn(D, Hf, Wf, generator=g, device=DEV)
    pool = lambda f: f.reshape(D, case["Hc"], 8, case["Wc"], 8).mean(dim=(2, 4)).bfloat16().contiguous()  # noqa: E731
    return pool(q), pool(r), q.bfloat16(), r.bfloat16()


def _correspondences(case, seed):
    r = np.random.default_rng(int(seed) * 131 + 3)
    m, h = case["m"], case["hyps"]
    K = hg.Intrinsics(1500.0, 1500.0, 960.0, 540.0, 1920, 1080)
    geo = dict(extent=100.0, alt=200.0, P=1)
    T = _poses(geo, seed)[0].double().cpu().numpy().reshape(3, 4)
    uv = r.uniform((0, 0), (K.width, K.height), (m, 2))
    d = r.uniform(150, 260, m)
    Xc = np.stack([(uv[:, 0] - K.cx) / K.fx * d, (uv[:, 1] - K.cy) / K.fy * d, d], 1)
    X = (Xc - T[:, 3]) @ T[:, :3]
    p = uv + r.normal(0, 0.7, (m, 2))
    bad = r.random(m) < case["outliers"]
    p[bad] = r.uniform((0, 0), (K.width, K.height), (int(bad.sum()), 2))
    prior = T.copy()
    prior[:, :3] = _rot(np.deg2rad(r.normal(0, 0.7, 3))).numpy() @ T[:, :3]
    prior[:, 3] = prior[:, :3] @ (T[:, :3].T @ T[:, 3]) + r.normal(0, 1.2, 3)
    samples = np.sort(r.integers(0, m - 2, (h, 3)), axis=1) + np.arange(3)  # three different points
    t = lambda a, dt=np.float32: torch.from_numpy(np.ascontiguousarray(a.astype(dt))).to(DEV)  # noqa: E731
    return K, t(p), t(X), t(prior.reshape(12)), t(samples, np.int32)


# ------------------------------------------------------------------ prepare and run
def prepare(case, seed):
    kind = case["kind"]
    s = dict(kind=kind, r=hg.Renderer())
    if kind == "match":
        s["maps"] = _match_maps(case, seed)
        N = case["Hc"] * case["Wc"]
        F = N * 64 if case["fine"] else 0
        # results past the last correspondence keep what the buffers held
        s["out"] = dict(n_coarse=torch.zeros(1, dtype=torch.int32, device=DEV))
        for k, m in (("coarse", N), ("fine", F)):
            for f, dt in (("query", torch.int32), ("render", torch.int32), ("p", torch.float32)):
                s["out"][f"{k}_{f}"] = torch.zeros(m, dtype=dt, device=DEV)
        if not case["fine"]:
            s["maps"] = s["maps"][:2] + (None, None)
        return s
    if kind == "solve":
        s["K"], s["p2d"], s["x3d"], s["pose0"], s["samples"] = _correspondences(case, seed)
        return s
    r = s["r"]
    s["scene"], s["poses"], s["K"] = _scene(case, seed), _poses(case, seed), _camera(case)
    if kind == "significance":
        g = _gen(seed + 1)
        P, D, H, W = case["P"], case["D"], case["H"], case["W"]
        shape = (P, D, H, W) if case["layout"] == "planar" else (P, H, W, D)
        s["maps"] = torch.randn(shape, generator=g, device=DEV)
        s["layout"] = case["layout"]
        r.render(s["scene"], s["poses"], s["K"])  # sizes the workspace for these views
        s["sum"] = torch.zeros(case["n"], device=DEV)
        s["count"] = torch.zeros(case["n"], dtype=torch.int32, device=DEV)
        s["opts"] = r.opts(tile=16)
        return s
    bf16 = bool(case.get("bf16"))
    s["checked"] = bool(case.get("checked"))
    s["out"] = r.alloc_outputs(s["scene"], case["P"], s["K"], bf16)
    s["opts"] = r.opts(feat_bf16=bf16)
    r.render(s["scene"], s["poses"], s["K"], feat_bf16=bf16, out=s["out"])  # sizes the workspace
    if kind == "refine":
        # the query view, one target for all candidate poses, a little off the first of them
        q = _target(case, seed, s["scene"], s["K"])
        s["t_rgb"], s["t_feat"] = q["rgb"], q["feat"]
        s["loss"] = torch.empty(case["P"], device=DEV)
        s["grads"] = r.alloc_grads(s["scene"], case["P"], ("pose",))
    elif kind == "train":
        s["go"] = _grad_out(case, seed)
        s["want"] = ("pose", "means", "opacities", "log_scales", "quats", "sh") + (("feat",) if case["D"] else ())
        s["grads"] = r.alloc_grads(s["scene"], case["P"], s["want"])
    return s


def _target(case, seed, scene, K):
    pose = _poses(case, seed, 1).double().cpu()
    T = torch.cat([pose.reshape(3, 4), torch.tensor([[0, 0, 0, 1.0]], dtype=F64)])
    d = torch.zeros(4, 4, dtype=F64)
    d[:3, :3] = torch.tensor([[0, -0.004, 0.006], [0.004, 0, -0.005], [-0.006, 0.005, 0]], dtype=F64)
    d[:3, 3] = torch.tensor([0.8, -0.5, 0.4], dtype=F64)
    pose = (torch.linalg.matrix_exp(d) @ T)[:3].reshape(1, 12).float().to(DEV)
    return hg.Renderer().render(scene, pose, K)


def _grad_out(case, seed):
    g = _gen(seed + 2)
    P, D, H, W = case["P"], case["D"], case["H"], case["W"]
    go = dict(rgb=(P, 3, H, W), depth=(P, H, W), alpha=(P, H, W), feat=(P, D, H, W))
    scale = 1.0 / (H * W)
    return {k: torch.randn(s, generator=g, device=DEV) * scale for k, s in go.items() if D or k != "feat"}


def run(s):
    r, kind = s["r"], s["kind"]
    if kind == "match":
        return r.match(*s["maps"], out=s["out"])
    if kind == "solve":
        return r.pnp(s["p2d"], s["x3d"], s["K"], s["pose0"], s["samples"])
    if kind == "significance":
        s["sum"].zero_()
        s["count"].zero_()
        r.significance_into(s["scene"], s["poses"], s["K"], s["maps"], s["sum"], s["count"], s["opts"],
                            layout=s["layout"])
        return dict(score_sum=s["sum"], vis_count=s["count"], score=hg.significance_final(s["sum"], s["count"]))
    if s["checked"]:
        return r.render(s["scene"], s["poses"], s["K"], out=s["out"])
    r.render_into(s["scene"], s["poses"], s["K"], s["out"], s["opts"])
    if kind == "refine":
        loss, grads = r.residual_backward(s["t_rgb"], s["t_feat"], loss=s["loss"], grads=s["grads"])
        return dict(s["out"], loss=loss, pose=grads["pose"])
    if kind == "train":
        grads = r.backward(s["go"], want=s["want"], grads=s["grads"])
        return dict(s["out"], grads=grads)
    return s["out"]


# ------------------------------------------------------------------ necessary work
def work(case):
    kind = case["kind"]
    if kind == "match":
        N, D = case["Hc"] * case["Wc"], case["D"]
        fine = 64 * N if case["fine"] else 0
        # both passes of the softmaxes need the cosines, which are not kept
        return dict(bytes=4 * D * (N + fine) + 12 * (N + fine), flops=2.0 * N * N * D + 2.0 * fine * 64 * D)
    if kind == "solve":
        m, h = case["m"], case["hyps"]
        return dict(bytes=21 * m + 16 * h, flops=m * h * 26.0 + 11 * m * 130.0)
    n, D, P, px = case["n"], case["D"], case["P"], case["W"] * case["H"]
    ground = (1.28 * case["alt"]) ** 2 * case["H"] / case["W"]
    seen = min(1.0, ground / case["extent"] ** 2)
    vis = seen * n
    scene = 28 * n + vis * (16 + 12 * (case["sh"] + 1) ** 2 + 2 * D)
    fb = 2 if case.get("bf16") else 4
    maps = P * px * (20 + fb * D)
    pair = 20 + 2 * (D + 4)
    if kind == "render":
        return dict(bytes=scene + maps, flops=P * px * LAYERS * float(pair))
    if kind == "refine":
        return dict(bytes=scene + maps + px * (12 + 4 * D), flops=P * px * LAYERS * float(3 * pair))
    if kind == "train":
        grads = n * 4 * (11 + 3 * (case["sh"] + 1) ** 2 + D)
        return dict(bytes=scene + 2 * maps + grads, flops=P * px * LAYERS * float(3 * pair))
    # significance: a pair's map vector, the scene, sums and counts
    return dict(bytes=scene + P * vis * 4 * D + 20 * n, flops=P * px * LAYERS * 20.0 + P * vis * 4.0 * D)


# ------------------------------------------------------------------ 64-bit values
def _sh_basis(deg, d):
    """Real spherical harmonics (Condon-Shortley phase, index l^2 + l + m)."""
    x, y, z = d.unbind(-1)
    Y = [torch.full_like(x, 0.28209479177387814)]
    if deg >= 1:
        c = 0.48860251190291987
        Y += [-c * y, c * z, -c * x]
    if deg >= 2:
        a, b, c = 1.0925484305920792, 0.31539156525252005, 0.5462742152960396
        Y += [a * x * y, -a * y * z, b * (2 * z * z - x * x - y * y), -a * x * z, c * (x * x - y * y)]
    if deg >= 3:
        a, b, c = 0.5900435899266435, 2.890611442640554, 0.4570457994644658
        q = 4 * z * z - x * x - y * y
        Y += [-a * y * (3 * x * x - y * y), b * x * y * z, -c * y * q,
              0.3731763325901154 * z * (2 * z * z - 3 * x * x - 3 * y * y), -c * x * q,
              0.5 * b * z * (x * x - y * y), -a * x * (x * x - 3 * y * y)]
    return torch.stack(Y, -1)


def _project(p, T, K, deg):
    """Per Gaussian: mean (u, v), conic, z, colour, k2 = 2 ln(255 o) and support half-widths, in 64 bits."""
    R, t = T[:, :3], T[:, 3]
    Xc = p["means"] @ R.T + t
    z = Xc[:, 2]
    xz, yz = Xc[:, 0] / z, Xc[:, 1] / z
    lx, ly = 1.3 * 0.5 * K.width / K.fx, 1.3 * 0.5 * K.height / K.fy
    zero = torch.zeros_like(z)
    J = torch.stack([torch.stack([K.fx / z, zero, -K.fx * xz.clamp(-lx, lx) / z], -1),
                     torch.stack([zero, K.fy / z, -K.fy * yz.clamp(-ly, ly) / z], -1)], 1)
    w, x, y, q = (p["quats"] / p["quats"].norm(dim=1, keepdim=True)).unbind(-1)
    Rq = torch.stack([1 - 2 * (y * y + q * q), 2 * (x * y - w * q), 2 * (x * q + w * y),
                      2 * (x * y + w * q), 1 - 2 * (x * x + q * q), 2 * (y * q - w * x),
                      2 * (x * q - w * y), 2 * (y * q + w * x), 1 - 2 * (x * x + y * y)], -1).reshape(-1, 3, 3)
    M = (J @ R) @ (Rq * torch.exp(p["log_scales"])[:, None, :])
    S = M @ M.transpose(1, 2).contiguous() + 0.3 * torch.eye(2, dtype=F64, device=DEV)
    det = S[:, 0, 0] * S[:, 1, 1] - S[:, 0, 1] ** 2
    conic = torch.stack([S[:, 1, 1] / det, -S[:, 0, 1] / det, S[:, 0, 0] / det], -1)
    d = p["means"] + (R.T @ t)
    Y = _sh_basis(deg, d / d.norm(dim=1, keepdim=True))
    colour = torch.relu((Y[..., None] * p["sh"]).sum(1) + 0.5)
    k2 = 2 * torch.log(255 * p["opacities"].detach())
    return dict(u=K.fx * xz + K.cx, v=K.fy * yz + K.cy, conic=conic, z=z, colour=colour, k2=k2,
                rx=torch.sqrt(k2 * S[:, 0, 0].detach()), ry=torch.sqrt(k2 * S[:, 1, 1].detach()))


def _tiles(f, K, tile=16):
    """(tile, depth)-ordered entries: per entry its tile and Gaussian; every tile its support rectangle touches."""
    ntx, nty = -(-K.width // tile), -(-K.height // tile)
    lo = lambda c, r: torch.floor((c - r - 1) / tile).long()  # noqa: E731
    hi = lambda c, r: torch.floor((c + r + 1) / tile).long()  # noqa: E731
    u, v = f["u"].detach(), f["v"].detach()
    x0, x1 = lo(u, f["rx"]).clamp(min=0), hi(u, f["rx"]).clamp(max=ntx - 1)
    y0, y1 = lo(v, f["ry"]).clamp(min=0), hi(v, f["ry"]).clamp(max=nty - 1)
    w, h = (x1 - x0 + 1).clamp(min=0), (y1 - y0 + 1).clamp(min=0)
    order = torch.sort(f["z"].detach(), stable=True).indices
    cnt = (w * h)[order]
    j = order.repeat_interleave(cnt)
    k = torch.arange(j.numel(), device=DEV) - (torch.cumsum(cnt, 0) - cnt).repeat_interleave(cnt)
    t = (y0[j] + k // w[j]) * ntx + x0[j] + k % w[j]
    s = torch.sort(t, stable=True)
    return s.values, j[s.indices], ntx, ntx * nty


def _visible(full, T, K):
    """Indices of the Gaussians that may reach the image."""
    with torch.no_grad():
        R, t = T[:, :3], T[:, 3]
        z = full["means"] @ R[2] + t[2]
        ok = torch.nonzero((z > 0.2) & (full["opacities"] >= 1 / 255)).squeeze(1)
        sub = {k: v[ok] for k, v in full.items() if k in ("means", "quats", "log_scales", "opacities")}
        sub["sh"] = torch.zeros(ok.numel(), 1, 3, dtype=F64, device=DEV)
        f = _project(sub, T, K, 0)
        keep = ((f["u"] + f["rx"] > -1) & (f["u"] - f["rx"] < K.width + 1) &
                (f["v"] + f["ry"] > -1) & (f["v"] - f["ry"] < K.height + 1))
    return ok[keep]


def _blend(p, f, K, D, entries, chunk=30_000_000):
    """Yields (pixels, maps, hit) per group of tiles: maps = (rgb, depth, alpha, feat), hit the entries' Gaussians
    and whether any pixel blends them."""
    tile = 16
    te, ge, ntx, nt = entries
    if not ge.numel():
        return
    count = torch.bincount(te, minlength=nt)
    start = torch.cumsum(count, 0) - count
    by = torch.sort(count, descending=True).indices
    sizes = count[by].tolist()
    a = 0
    while a < nt:
        L = max(1, sizes[a])
        b = min(nt, a + max(1, chunk // (L * tile * tile)))
        ts = by[a:b]
        a = b
        slot = torch.arange(L, device=DEV)
        live = slot[None] < count[ts][:, None]
        idx = torch.where(live, start[ts][:, None] + slot[None], 0)
        g = ge[idx]
        i = torch.arange(tile * tile, device=DEV)
        px = (ts % ntx)[:, None] * tile + i % tile
        py = (ts // ntx)[:, None] * tile + i // tile
        inside = (px < K.width) & (py < K.height)
        pix = torch.where(inside, py * K.width + px, -1)
        dx = (px + 0.5).to(F64)[:, :, None] - f["u"][g][:, None, :]
        dy = (py + 0.5).to(F64)[:, :, None] - f["v"][g][:, None, :]
        c = f["conic"][g][:, None]
        power = -0.5 * (c[..., 0] * dx * dx + c[..., 2] * dy * dy) - c[..., 1] * dx * dy
        alpha = torch.clamp(p["opacities"][g][:, None] * torch.exp(power), max=0.99)
        with torch.no_grad():
            gate = (alpha >= 1 / 255) & (power <= 0) & live[:, None]
            keep = gate & (torch.cumprod(torch.where(gate, 1 - alpha, 1.0), 2) >= 1e-4)
        alpha = torch.where(keep, alpha, 0.0)
        Tn = torch.cumprod(1 - alpha, 2)
        w = alpha * torch.cat([torch.ones_like(Tn[..., :1]), Tn[..., :-1]], 2)
        A = 1 - Tn[..., -1]
        rgb = w @ f["colour"][g].contiguous()
        zs = (w * f["z"][g][:, None]).sum(2)
        depth = torch.where(A > 0, zs / torch.where(A > 0, A, 1.0), 0.0)
        feat = w @ p["feat"][g].contiguous() if D else None
        yield pix, inside, (rgb, depth, A, feat), (g, keep.any(1))


def _full(scene, grad=False):
    p = dict(means=scene.means, quats=scene.quats, log_scales=scene.log_scales, opacities=scene.opacities, sh=scene.sh)
    if scene.feat is not None:
        p["feat"] = scene.feat.float()
    return {k: v.double().requires_grad_(grad) for k, v in p.items()}


def _exp_left(xi, T):
    h = torch.zeros(4, 4, dtype=F64, device=DEV)
    E = [torch.zeros(4, 4, dtype=F64, device=DEV) for _ in range(6)]
    for k in range(3):
        E[k][k, 3] = 1
    for k, (i, j) in enumerate(((2, 1), (0, 2), (1, 0))):
        E[3 + k][i, j], E[3 + k][j, i] = 1, -1
    for k in range(6):
        h = h + xi[k] * E[k]
    T4 = torch.cat([T, torch.tensor([[0, 0, 0, 1.0]], dtype=F64, device=DEV)])
    return (torch.linalg.matrix_exp(h) @ T4)[:3]


def _exact_maps(case, seed):
    scene, poses, K = _scene(case, seed), _poses(case, seed), _camera(case)
    kind, P, D, W, H = case["kind"], case["P"], case["D"], case["W"], case["H"]
    train, refine = kind == "train", kind == "refine"
    full = _full(scene, train)
    bf16 = bool(case.get("bf16"))
    out = dict(rgb=torch.zeros(P, 3, H * W, dtype=F64, device=DEV), depth=torch.zeros(P, H * W, dtype=F64, device=DEV),
               alpha=torch.zeros(P, H * W, dtype=F64, device=DEV),
               feat=torch.zeros(P, D, H * W, dtype=F64, device=DEV) if D else None)
    if refine:
        q = _target(case, seed, scene, K)
        t_rgb, t_feat = q["rgb"][0].reshape(3, -1).T, q["feat"][0].reshape(D, -1).T if D else None
        loss, gpose = torch.zeros(P, dtype=F64, device=DEV), torch.zeros(P, 6, dtype=F64, device=DEV)
    if train:
        go = {k: v.double() for k, v in _grad_out(case, seed).items()}
        gpose = torch.zeros(P, 6, dtype=F64, device=DEV)
    for k in range(P):
        T0 = poses[k].double().reshape(3, 4)
        xi = torch.zeros(6, dtype=F64, device=DEV, requires_grad=train or refine)
        T = _exp_left(xi, T0) if train or refine else T0
        vis = _visible(full, T0, K)
        with torch.set_grad_enabled(train or refine):
            p = {n: v[vis] for n, v in full.items()}
            f = _project(p, T, K, case["sh"])
            names = [n for n in ("u", "v", "conic", "z", "colour")]
            cut = {n: f[n].detach().requires_grad_(train or refine) for n in names}
            cutp = {n: p[n].detach().requires_grad_(train) for n in ("opacities", "feat") if n in p}
            for pix, inside, (rgb, depth, A, feat), _ in _blend(cutp, cut, K, D, _tiles(f, K)):
                at = pix[inside]
                out["rgb"][k][:, at] = rgb.detach()[inside].T
                out["depth"][k][at] = depth.detach()[inside]
                out["alpha"][k][at] = A.detach()[inside]
                if D:
                    out["feat"][k][:, at] = feat.detach()[inside].T
                if refine:
                    l = (rgb[inside] - t_rgb[at].double()).abs().sum()
                    if D:
                        F, Ft = feat[inside], t_feat[at].double()
                        n2 = torch.linalg.vector_norm(F, dim=1) * torch.linalg.vector_norm(Ft, dim=1) + 1e-8
                        l = l + (1 - (F * Ft).sum(1) / n2).sum()
                    l = l / (H * W)
                    loss[k] += l.detach()
                    l.backward()
                elif train:
                    l = (rgb[inside] * go["rgb"][k].reshape(3, -1)[:, at].T).sum()
                    l = l + (depth[inside] * go["depth"][k].reshape(-1)[at]).sum()
                    l = l + (A[inside] * go["alpha"][k].reshape(-1)[at]).sum()
                    if D:
                        l = l + (feat[inside] * go["feat"][k].reshape(D, -1)[:, at].T).sum()
                    l.backward()
            if train or refine:
                pairs = [(f[n], cut[n].grad) for n in names] + [(p[n], cutp[n].grad) for n in cutp if train]
                pairs = [(a, b) for a, b in pairs if b is not None and a.requires_grad]
                if pairs:
                    torch.autograd.backward([a for a, _ in pairs], [b for _, b in pairs])
                if xi.grad is not None:
                    gpose[k] = xi.grad
    res = dict(rgb=out["rgb"].reshape(P, 3, H, W), depth=out["depth"].reshape(P, H, W),
               alpha=out["alpha"].reshape(P, H, W), feat=out["feat"].reshape(P, D, H, W) if D else None)
    if refine:
        res.update(loss=loss, pose=gpose)
    if train:
        res["grads"] = dict(pose=gpose, **{k: v.grad if v.grad is not None else torch.zeros_like(v)
                                           for k, v in full.items()})
    return res


def _exact_significance(case, seed):
    s = prepare(case, seed)
    scene, poses, K = s["scene"], s["poses"], s["K"]
    full, n, D = _full(scene), case["n"], case["D"]
    total = torch.zeros(n, dtype=F64, device=DEV)
    count = torch.zeros(n, dtype=F64, device=DEV)
    with torch.no_grad():
        for k in range(case["P"]):
            T = poses[k].double().reshape(3, 4)
            vis = _visible(full, T, K)
            p = {m: v[vis] for m, v in full.items()}
            f = _project(p, T, K, case["sh"])
            seen = torch.zeros(vis.numel(), dtype=torch.bool, device=DEV)
            for _, _, _, (g, hit) in _blend(dict(opacities=p["opacities"]), f, K, 0, _tiles(f, K)):
                seen[g[hit]] = True
            u, v = f["u"], f["v"]
            seen &= (u >= 0) & (u < K.width) & (v >= 0) & (v < K.height)
            j = torch.nonzero(seen).squeeze(1)
            cx, cy = u[j].floor().long().clamp(max=K.width - 1), v[j].floor().long().clamp(max=K.height - 1)
            m = s["maps"][k]
            m = (m[:, cy, cx].T if case["layout"] == "planar" else m[cy, cx]).double()
            F = p["feat"][j]
            total[vis[j]] += (F * m).sum(1) / (F.norm(dim=1) * m.norm(dim=1) + 1e-8)
            count[vis[j]] += 1
    return dict(score_sum=total, vis_count=None, score=total / count.clamp(min=1))


def _exact_match(case, seed):
    q_c, r_c, q_f, r_f = _match_maps(case, seed)
    D, N, Wc, tau = case["D"], case["Hc"] * case["Wc"], case["Wc"], 0.1
    Q, R = q_c.double().reshape(D, N).T.contiguous(), r_c.double().reshape(D, N).T.contiguous()
    nq, nr = Q.norm(dim=1), R.norm(dim=1)
    cos = lambda b: (Q[b] @ R.T.contiguous()) / (nq[b][:, None] * nr + 1e-8) / tau  # noqa: E731
    rows = [slice(a, min(N, a + 4096)) for a in range(0, N, 4096)]
    a, b = torch.empty(N, dtype=F64, device=DEV), torch.full((N,), -math.inf, dtype=F64, device=DEV)
    for k in rows:
        S = cos(k)
        a[k] = torch.logsumexp(S, 1)
        b = torch.logaddexp(b, torch.logsumexp(S, 0))
    best, arg = torch.full((N,), -math.inf, dtype=F64, device=DEV), torch.zeros(N, dtype=torch.long, device=DEV)
    ra, rp = torch.empty(N, dtype=torch.long, device=DEV), torch.empty(N, dtype=F64, device=DEV)
    for k in rows:
        L = 2 * cos(k) - a[k][:, None] - b
        rp[k], ra[k] = L.max(1)
        v, i = L.max(0)
        arg = torch.where(v > best, i + k.start, arg)
        best = torch.maximum(best, v)
    i = torch.nonzero(arg[ra] == torch.arange(N, device=DEV)).squeeze(1)
    j, cnt = ra[i], i.numel()
    p = torch.zeros(N, dtype=F64, device=DEV)
    p[:cnt] = torch.exp(rp[i])
    res = dict(coarse_p=p, fine_p=torch.zeros(0, dtype=F64, device=DEV))
    if case["fine"]:
        win = lambda m: m.reshape(D, case["Hc"], 8, Wc, 8).permute(1, 3, 2, 4, 0).reshape(N, 64, D)  # noqa: E731
        fp = torch.zeros(N, 64, dtype=F64, device=DEV)
        qf, rf = win(q_f), win(r_f)
        for c in range(0, cnt, 4096):
            x, y = qf[i[c:c + 4096]].double(), rf[j[c:c + 4096]].double()
            S = (x @ y.transpose(1, 2).contiguous()) / (x.norm(dim=2)[:, :, None] * y.norm(dim=2)[:, None] + 1e-8) / tau
            L = 2 * S - torch.logsumexp(S, 2, keepdim=True) - torch.logsumexp(S, 1, keepdim=True)
            v, m = L.max(2)
            mutual = L.argmax(1).gather(1, m) == torch.arange(64, device=DEV)
            fp[c:c + v.shape[0]] = torch.where(mutual, torch.exp(v), 0.0)
        res["fine_p"] = fp.reshape(-1)
    return res


def _exact_solve(case, seed, tau=2.0):
    K, p2d, x3d, pose0, samples = _correspondences(case, seed)
    p, X = p2d.double(), x3d.double()

    def rows(T, X, p):
        Xc = X @ T[..., :3].transpose(-1, -2).contiguous() + T[..., None, :, 3]
        x, y, z = Xc.unbind(-1)
        r = torch.stack([K.fx * x / z + K.cx, K.fy * y / z + K.cy], -1) - p
        o = torch.zeros_like(z)
        a, a2, b, b2 = K.fx / z, -K.fx * x / z ** 2, K.fy / z, -K.fy * y / z ** 2
        J = torch.stack([torch.stack([a, o, a2, a2 * y, a * z - a2 * x, -a * y], -1),
                         torch.stack([o, b, b2, -b * z + b2 * y, -b2 * x, b * x], -1)], -2)
        return r, J, z

    def hat(d):
        h = torch.zeros(d.shape[:-1] + (4, 4), dtype=F64, device=DEV)
        h[..., 0, 1], h[..., 0, 2], h[..., 1, 2] = -d[..., 5], d[..., 4], -d[..., 3]
        h[..., 1, 0], h[..., 2, 0], h[..., 2, 1] = d[..., 5], -d[..., 4], d[..., 3]
        h[..., :3, 3] = d[..., :3]
        return h

    def step(T, r, J, w):
        A = (J * w[..., None, None]).flatten(-3, -2).transpose(-1, -2).contiguous() @ J.flatten(-3, -2).contiguous()
        g = (J * (r * w[..., None])[..., None]).sum((-3, -2))
        d = -torch.linalg.solve_ex(A, g).result
        T4 = torch.zeros(T.shape[:-2] + (4, 4), dtype=F64, device=DEV)
        T4[..., :3, :], T4[..., 3, 3] = T, 1
        return (torch.linalg.matrix_exp(hat(d)) @ T4)[..., :3, :]

    best, refined = -1, pose0.double().reshape(3, 4)
    s = samples.long()
    T = refined.expand(s.shape[0], 3, 4)
    full_p = p
    p = full_p[s]
    for _ in range(10):
        r, J, _z = rows(T, X[s], p)
        T = step(T, r, J, torch.ones_like(_z))
    p = full_p
    for k in range(s.shape[0]):
        r, _J, z = rows(T[k], X, p)
        c = int(((r.square().sum(-1) < tau * tau) & (z > 0)).sum())
        if c > best and bool(torch.isfinite(T[k]).all()):
            best, refined = c, T[k]
    for _ in range(10):
        r, J, z = rows(refined, X, p)
        refined = step(refined, r, J, ((r.square().sum(-1) < tau * tau) & (z > 0)).to(F64))
    return dict(pose=refined.reshape(12), best=None, counts=None, n_inliers=None, inliers=None, hyp_poses=None)


def exact(case, seed):
    kind = case["kind"]
    if kind == "match":
        return _exact_match(case, seed)
    if kind == "solve":
        return _exact_solve(case, seed)
    if kind == "significance":
        return _exact_significance(case, seed)
    return _exact_maps(case, seed)
