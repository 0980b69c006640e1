"""GPU backward against a dense 64-bit evaluation with autograd on the CPU
(every pixel against every Gaussian, no tiles and no lists), over lists of
several staging rounds; the summation error of the mean gradient; infinite
features and output gradients; one shared target over several pose blocks; a
captured step at another tile size than the workspace was sized at."""
import math

import numpy as np
import pytest

import synth
from gpu_util import log, to_np

pytestmark = pytest.mark.gpu
REL = 1e-3  # of the norm: the bar of the gradient checks against the oracle


@pytest.fixture(scope="module")
def hg():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2507_15683_amd as hg
    return hg


def _t(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _rel(a, b):
    a, b = np.asarray(a, np.float64).ravel(), np.asarray(b, np.float64).ravel()
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30))


def _leaves(sc, D):
    import torch
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).double().requires_grad_(True)  # noqa: E731
    p = dict(means=d(sc.means), opacities=d(sc.opacities), log_scales=d(sc.log_scales), quats=d(sc.quats), sh=d(sc.sh))
    if D:
        p["feat"] = d((sc.feat.astype(np.uint32) << 16).view(np.float32))
    p["pose"] = torch.zeros(6, dtype=torch.float64, requires_grad=True)
    return p


def _maps64(p, pose, cam, bg=(0.0, 0.0, 0.0)):
    """rgb, depth, alpha and feature maps of one view (degree-0 colour), differentiable in every leaf."""
    import torch
    F64 = torch.float64
    xi = p["pose"]
    hat = torch.zeros(4, 4, dtype=F64)
    for k, (i, j) in enumerate(((2, 1), (0, 2), (1, 0))):
        e, r = torch.zeros(4, 4, dtype=F64), torch.zeros(4, 4, dtype=F64)
        e[k, 3] = 1
        r[i, j], r[j, i] = 1, -1
        hat = hat + xi[k] * e + xi[3 + k] * r
    T0 = torch.cat([torch.from_numpy(np.asarray(pose, np.float64)).reshape(3, 4), torch.tensor([[0, 0, 0, 1.0]], dtype=F64)])
    T = (torch.linalg.matrix_exp(hat) @ T0)[:3]
    R, t = T[:, :3], T[:, 3]
    X = p["means"] @ R.T + t
    z = X[:, 2]
    xz, yz = X[:, 0] / z, X[:, 1] / z
    lx, ly = 1.3 * 0.5 * cam.width / cam.fx, 1.3 * 0.5 * cam.height / cam.fy
    o = torch.zeros_like(z)
    J = torch.stack([torch.stack([cam.fx / z, o, -cam.fx * xz.clamp(-lx, lx) / z], -1),
                     torch.stack([o, cam.fy / z, -cam.fy * yz.clamp(-ly, ly) / z], -1)], 1)
    w, x, y, q = (p["quats"] / p["quats"].norm(dim=1, keepdim=True)).unbind(-1)
    Rq = torch.stack([1 - 2 * (y * y + q * q), 2 * (x * y - w * q), 2 * (x * q + w * y),
                      2 * (x * y + w * q), 1 - 2 * (x * x + q * q), 2 * (y * q - w * x),
                      2 * (x * q - w * y), 2 * (y * q + w * x), 1 - 2 * (x * x + y * y)], -1).reshape(-1, 3, 3)
    M = (J @ R) @ (Rq * torch.exp(p["log_scales"])[:, None, :])
    S = M @ M.transpose(1, 2) + 0.3 * torch.eye(2, dtype=F64)
    det = S[:, 0, 0] * S[:, 1, 1] - S[:, 0, 1] ** 2
    a, b, c = S[:, 1, 1] / det, -S[:, 0, 1] / det, S[:, 0, 0] / det
    colour = torch.relu(0.28209479177387814 * p["sh"][:, 0] + 0.5)
    order = torch.sort(z.detach(), stable=True).indices
    order = order[z.detach()[order] > 0.2]
    py, px = torch.meshgrid(torch.arange(cam.height) + 0.5, torch.arange(cam.width) + 0.5, indexing="ij")
    dx = px.reshape(-1, 1).double() - (cam.fx * xz + cam.cx)[order]
    dy = py.reshape(-1, 1).double() - (cam.fy * yz + cam.cy)[order]
    power = -0.5 * (a[order] * dx * dx + c[order] * dy * dy) - b[order] * dx * dy
    alpha = torch.clamp(p["opacities"][order] * torch.exp(power), max=0.99)
    with torch.no_grad():
        gate = (alpha >= 1 / 255) & (power <= 0)
        keep = gate & (torch.cumprod(torch.where(gate, 1 - alpha, 1.0), 1) >= 1e-4)
    alpha = torch.where(keep, alpha, 0.0)
    Tn = torch.cumprod(1 - alpha, 1)
    wt = alpha * torch.cat([torch.ones_like(Tn[:, :1]), Tn[:, :-1]], 1)
    A = 1 - Tn[:, -1]
    img = lambda m: m.T.reshape(-1, cam.height, cam.width)  # noqa: E731
    rgb = wt @ colour[order] + Tn[:, -1:] * torch.tensor(bg, dtype=F64)
    depth = torch.where(A > 0, (wt * z[order]).sum(1) / torch.where(A > 0, A, 1.0), 0.0)
    out = dict(rgb=img(rgb), depth=img(depth[:, None])[0], alpha=img(A[:, None])[0], feat=None)
    if "feat" in p:
        out["feat"] = img(wt @ p["feat"][order])
    return out


def _long_scene(D, seed):
    sc, P, cam = synth.tiny_scene(1500, seed, width=45, height=37, feat_dim=D, sh_degree=0)
    sc = sc.copy()
    sc.opacities[:] *= 0.15  # long walks: many splats blend before a pixel stops
    return sc, P, cam


@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("D", [0, 8, 16, 32, 64])
def test_gradients_over_long_lists(hg, D, tile):
    """Random output gradients of every map, a background: all Gaussian
    gradients (the features' among them) and the pose's."""
    import torch
    sc, P, cam = _long_scene(D, 201 + D)
    bg = (0.3, 0.1, 0.6)
    log(f"case: gradients against 64 bits D={D} tile={tile}")
    r = hg.Renderer()
    out = r.render(hg.GaussianScene.from_numpy(sc), _t(P), hg.Intrinsics.of(cam), tile=tile, bg=bg)
    assert r.stats()["max_tile_list"] > 130  # several rounds of 64
    gen = torch.Generator().manual_seed(D + tile)
    go = {k: torch.randn(v.shape, generator=gen) for k, v in out.items() if v is not None}
    want = ("pose", "means", "opacities", "log_scales", "quats", "sh") + (("feat",) if D else ())
    got = r.backward({k: v.cuda() for k, v in go.items()}, want=want)
    p = _leaves(sc, D)
    ref = _maps64(p, P[0], cam, bg)
    sum((ref[k] * go[k][0].double()).sum() for k in go).backward()
    for k in want:
        rel = _rel(to_np(got[k]), p[k].grad.numpy())
        log(k, rel)
        assert rel < REL, (k, rel)


@pytest.mark.parametrize("D,tile", [(0, 16), (8, 8), (16, 16), (32, 8), (32, 16), (32, 32), (64, 8), (64, 16)])
def test_residual_gradients_over_long_lists(hg, D, tile):
    """The refinement residual's loss, pose gradient alone and with the means'."""
    import torch
    sc, P, cam = _long_scene(D, 301 + D)
    scene, K = hg.GaussianScene.from_numpy(sc), hg.Intrinsics.of(cam)
    log(f"case: residual against 64 bits D={D} tile={tile}")
    tgt = hg.Renderer().render(scene, _t(synth.perturb_poses(P[0], 1, 7, 1.0, 2.0)), K)
    r = hg.Renderer()
    r.render(scene, _t(P), K, tile=tile)
    assert r.stats()["max_tile_list"] > 130
    loss, g1 = r.residual_backward(tgt["rgb"], tgt["feat"])
    loss, g1 = to_np(loss).copy(), to_np(g1["pose"]).copy()
    _, g2 = r.residual_backward(tgt["rgb"], tgt["feat"], want=("pose", "means", "opacities"))
    p = _leaves(sc, D)
    ref = _maps64(p, P[0], cam)
    npx = cam.width * cam.height
    L = (ref["rgb"] - tgt["rgb"][0].cpu().double()).abs().sum() / npx
    if D:
        F, G = ref["feat"], tgt["feat"][0].cpu().double()
        n = torch.linalg.vector_norm(F, dim=0) * torch.linalg.vector_norm(G, dim=0) + 1e-8
        L = L + (1 - (F * G).sum(0) / n).sum() / npx
    L.backward()
    assert abs(loss[0] - float(L)) < 1e-5 * abs(float(L))
    assert _rel(g1, p["pose"].grad.numpy()) < REL
    for k in ("pose", "means", "opacities"):
        assert _rel(to_np(g2[k]), p[k].grad.numpy()) < REL, k


@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("length,turn", [(60.0, 0.6), (60.0, 2.2), (90.0, 0.9), (90.0, 1.1)])
def test_mean_gradient_of_needles(hg, length, turn, tile):
    """One tilted needle whose mean is the image centre, a corner between
    pixels: the pixels p and its mirror image through the mean have the same
    alpha to the bit and opposite terms dL/dpower (a dx + b dy), so the mean's
    gradient along x and y is 0 and what comes out is the error of the sum.

    Bound: a term passes at most 8 additions in its row, 3 across the rows and 4
    across the waves, and carries 2 roundings of its own, each at most 2^-24 of
    the terms of its tile; the tiles' sums, nearly 0 each, add less than one
    more: 18 x 2^-24 of the sum of |terms|."""
    import torch
    W = H = 1024
    f, z, o, thin = 100.0, 10.0, 0.8, 0.05
    q = np.array([[math.cos(turn / 2), 0, 0, math.sin(turn / 2)]], np.float32)
    ls = np.log(np.array([[length, thin, thin]]) * z / f).astype(np.float32)
    sc = synth.Scene(means=np.array([[0, 0, z]], np.float32), log_scales=ls, quats=q,
                     opacities=np.array([o], np.float32), sh=np.ones((1, 1, 3), np.float32), sh_degree=0)
    K = hg.Intrinsics(f, f, W / 2.0, H / 2.0, W, H)
    pose = _t(np.array([[1, 0, 0, 0, 0, 1, 0, 0, 0, 0, 1, 0]], np.float32))
    log(f"case: needle {length} px at {turn} rad, tile {tile}")
    r = hg.Renderer()
    out = r.render(hg.GaussianScene.from_numpy(sc), pose, K, tile=tile)
    g = to_np(r.backward(dict(rgb=torch.ones_like(out["rgb"])), want=("means",))["means"])[0]
    c, s = math.cos(turn), math.sin(turn)
    R = np.array([[c, -s], [s, c]])
    a, b, _, d = np.linalg.inv(R @ np.diag([length ** 2, thin ** 2]) @ R.T + 0.3 * np.eye(2)).ravel()
    dx, dy = np.meshgrid(np.arange(W) + 0.5 - W / 2, np.arange(H) + 0.5 - H / 2)
    alpha = o * np.exp(-0.5 * (a * dx * dx + d * dy * dy) - b * dx * dy)
    dpow = np.where(alpha >= 1 / 255, alpha, 0) * 3 * (0.28209479177387814 + 0.5)
    for k, term in enumerate((a * dx + b * dy, b * dx + d * dy)):
        scale = np.abs(dpow * term).sum() * f / z
        log("error of the sum, in 2^-24 of the terms:", abs(g[k]) / scale * 2 ** 24)
        assert abs(g[k]) <= 18 * 2.0 ** -24 * scale, k


@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("D", [8, 16, 32, 64])
def test_infinite_feature_or_gradient_gives_infinities(hg, D, tile):
    """Three concentric splats, dL/dfeat = 1.  h is the pixel gradient times
    the feature, so an infinite feature of the middle splat makes its opacity
    gradient +infinity, that of the splat before it -infinity (its suffix sum)
    and leaves the one behind finite; an infinite pixel gradient and positive
    features make that of the last splat +infinity."""
    import torch
    n = 3
    feat = np.full((n, D), 0x3F80, np.uint16)  # 1.0
    sc = synth.Scene(means=np.array([[0, 0, 9], [0, 0, 10], [0, 0, 11]], np.float32),
                     log_scales=np.full((n, 3), -1.0, np.float32), quats=np.tile(np.float32([1, 0, 0, 0]), (n, 1)),
                     opacities=np.full(n, 0.5, np.float32), sh=np.ones((n, 1, 3), np.float32), sh_degree=0, feat=feat)
    K = hg.Intrinsics(100.0, 100.0, 20.0, 18.0, 40, 36)
    pose = _t(np.array([[1, 0, 0, 0, 0, 1, 0, 0, 0, 0, 1, 0]], np.float32))
    r = hg.Renderer()
    for piece in range(D // 8):
        log(f"case: infinite feature D={D} tile={tile} piece {piece}")
        sc.feat[:] = 0x3F80
        sc.feat[1, 8 * piece + 5] = 0x7F80
        out = r.render(hg.GaussianScene.from_numpy(sc), pose, K, tile=tile)
        g = to_np(r.backward(dict(feat=torch.ones_like(out["feat"])), want=("opacities",))["opacities"])
        assert g[0] == -math.inf and g[1] == math.inf and math.isfinite(g[2]), g
        sc.feat[:] = 0x3F80
        out = r.render(hg.GaussianScene.from_numpy(sc), pose, K, tile=tile)
        go = torch.ones_like(out["feat"])
        go[0, 8 * piece + 2] = math.inf
        g = to_np(r.backward(dict(feat=go), want=("opacities",))["opacities"])
        assert g[2] == math.inf, g


def test_shared_target_over_several_pose_blocks(hg):
    """One target for 11 poses -- a full block of 8 and a ragged one, 35 tiles
    in runs of 16, 16 and 3 -- gives what the same target per pose gives: the
    loss bitwise, the gradients to float-atomic rounding."""
    sc, P, cam = synth.tiny_scene(700, 150, width=97, height=71, feat_dim=32, sh_degree=1)
    Ps = synth.perturb_poses(P[0], 11, 151, 1.0, 2.0)
    scene, K = hg.GaussianScene.from_numpy(sc), hg.Intrinsics.of(cam)
    log("case: shared target over 11 poses")
    q = hg.Renderer().render(scene, _t(P), K)
    rep = {k: q[k].expand(11, -1, -1, -1).contiguous() for k in ("rgb", "feat")}
    r = hg.Renderer()
    r.render(scene, _t(Ps), K)
    la, ga = r.residual_backward(q["rgb"], q["feat"])
    la, pa = to_np(la).copy(), to_np(ga["pose"]).copy()
    lb, gb = r.residual_backward(rep["rgb"], rep["feat"])
    assert np.array_equal(la, to_np(lb))
    for k in range(11):
        assert _rel(to_np(gb["pose"])[k], pa[k]) < 1e-6, k


def test_captured_step_at_a_larger_tile_than_sized(hg):
    """A workspace sized by an eager step at tile 16 holds a captured one at
    tile 32, where an odd size has more quadrants than it had tiles of 16 (540
    against 510); every replay gives the eager step's loss and pose gradient."""
    import torch
    sc, P, cam = synth.tiny_scene(600, 160, width=480, height=270, feat_dim=8, sh_degree=0)
    scene, K = hg.GaussianScene.from_numpy(sc), hg.Intrinsics.of(cam)
    log("case: captured step at tile 32 after an eager one at tile 16")
    tgt = hg.Renderer().render(scene, _t(synth.perturb_poses(P[0], 1, 161, 1.0, 2.0)), K)
    poses, opts = _t(P), hg.Renderer().opts(tile=32)
    e = hg.Renderer()
    e.render(scene, poses, K, tile=32)
    loss, g = e.residual_backward(tgt["rgb"], tgt["feat"])
    want = to_np(loss).copy(), to_np(g["pose"]).copy()
    r, s = hg.Renderer(), torch.cuda.Stream()
    out = r.render(scene, poses, K, tile=16)
    loss, g = r.residual_backward(tgt["rgb"], tgt["feat"])
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        r.graph_begin(s)
        try:
            r.render_into(scene, poses, K, out, opts, s)
            r.residual_backward(tgt["rgb"], tgt["feat"], loss=loss, grads=g, stream=s)
        finally:
            r.graph_end()
        for _ in range(3):
            loss.zero_()
            g["pose"].zero_()
            r.graph_launch(1, s)
            s.synchronize()
            assert np.array_equal(to_np(loss), want[0])
            assert _rel(to_np(g["pose"]), want[1]) < 1e-6
