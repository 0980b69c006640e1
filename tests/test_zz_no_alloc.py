"""The allocation-free render (hgsr_render_noalloc, workspace in the
library's static per-device array) against hgsr_render through the C ABI:
bitwise equal images on consecutive calls (the 1080p / 1M-Gaussian view, then
a smaller scene and image), capacity errors, and the overflow flag."""
import ctypes

import numpy as np
import pytest

import synth
from gpu_util import log, to_np

pytestmark = pytest.mark.gpu

SCRATCH_BYTES = 128 << 20


@pytest.fixture(scope="module")
def hg():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2507_15683_amd as hg
    return hg


def _poses(P):
    import torch
    return torch.from_numpy(np.ascontiguousarray(P, dtype=np.float32).reshape(-1, 12)).cuda()


def _noalloc(hg, scene, poses, K, opts, out, records=0, keys=0):
    """One hgsr_render_noalloc call; returns (status, overflow flags)."""
    import torch
    from paper_2507_15683_amd import _lib
    lib = _lib.load()
    flags = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    g = scene.c()
    o = _lib.Outputs(out["rgb"].data_ptr(), out["depth"].data_ptr(), out["alpha"].data_ptr(),
                     out["feat"].data_ptr() if out["feat"] is not None else None)
    kc = K.c()
    st = lib.hgsr_render_noalloc(ctypes.byref(g), poses.data_ptr(), poses.shape[0], ctypes.byref(kc),
                                 ctypes.byref(opts), ctypes.byref(o), records, keys, flags.data_ptr(), None)
    torch.cuda.synchronize()
    return st, int(flags.item()) if st == 0 else None


def _same(a, b, label):
    for k in ("rgb", "depth", "alpha", "feat"):
        if a[k] is None:
            assert b[k] is None
            continue
        x, y = to_np(a[k]), to_np(b[k])
        assert np.array_equal(x, y), (label, k, float(np.abs(x - y).max()))
    log(label, "bitwise equal to hgsr_render")


def _case(hg, sc, P, cam, label, tile=16, records=0, keys=0, feat_bf16=False):
    scene = hg.GaussianScene.from_numpy(sc)
    poses = _poses(P)
    K = hg.Intrinsics.of(cam)
    r = hg.Renderer()
    ref = r.render(scene, poses, K, tile=tile, feat_bf16=feat_bf16)
    opts = r.opts(tile=tile, feat_bf16=feat_bf16)
    out = r.alloc_outputs(scene, poses.shape[0], K, feat_bf16)
    for k in ("rgb", "depth", "alpha"):
        out[k].fill_(float("nan"))
    log(f"case: {label}: hgsr_render_noalloc, {poses.shape[0]} pose(s) {cam.width}x{cam.height}, "
        f"{scene.n} Gaussians, tile {tile}, capacities {records}/{keys}")
    st, flags = _noalloc(hg, scene, poses, K, opts, out, records, keys)
    assert st == 0, hg._lib.load().hgsr_last_error()
    assert flags == 0, flags
    _same(ref, out, label)
    r.close()


def test_two_calls_in_a_row_match_hgsr_render(hg):
    sc, P, cam = synth.aerial_1m_1080p(0)
    _case(hg, sc, P, cam, "1M Gaussians, 1920x1080")
    sc2, P2, cam2 = synth.tiny_scene(300, 7, width=80, height=56, sh_degree=2, feat_dim=16)
    P2 = np.concatenate([P2, synth.perturb_poses(P2[0], 2, 7, 1.0, 2.0)], axis=0)
    _case(hg, sc2, P2, cam2, "300 Gaussians, 3 poses of 80x56 (smaller, after the large call)", tile=8)


def test_explicit_capacities_and_bf16_features(hg):
    sc, P, cam = synth.terrain_20k_view(1)
    sc = synth.terrain_scene(20_000, 200.0, 1001, sh_degree=1, feat_dim=32)
    _case(hg, sc, P, cam, "20k Gaussians, 256x192, explicit capacities", records=40_000, keys=200_000,
          feat_bf16=True)


def test_capacity_rejected_with_message(hg):
    import torch
    sc, P, cam = synth.terrain_20k_view(0)
    scene = hg.GaussianScene.from_numpy(sc)
    K = hg.Intrinsics(1500.0, 1500.0, 960.0, 540.0, 1920, 1080)
    poses = _poses(np.repeat(P, 16, axis=0))
    r = hg.Renderer()
    opts = r.opts()
    # outputs are never written: the call fails before it enqueues anything
    out = dict(rgb=torch.empty(1, device="cuda"), depth=torch.empty(1, device="cuda"),
               alpha=torch.empty(1, device="cuda"), feat=None)
    log("case: 16 poses of 1920x1080 exceed the static scratch")
    st, _ = _noalloc(hg, scene, poses, K, opts, out)
    msg = hg._lib.load().hgsr_last_error().decode()
    log("status", st, msg)
    assert st == 3 and "static scratch" in msg
    log("case: explicit capacities beyond the scratch")
    st, _ = _noalloc(hg, scene, poses[:1], K, opts, out, records=1 << 20, keys=1 << 24)
    msg = hg._lib.load().hgsr_last_error().decode()
    assert st == 3 and str(SCRATCH_BYTES) in msg, msg
    log("case: only one capacity given")
    st, _ = _noalloc(hg, scene, poses[:1], K, opts, out, records=1000, keys=0)
    assert st == 1
    r.close()


def test_overflow_flag_then_clean_call(hg):
    sc, P, cam = synth.terrain_20k_view(2)
    scene = hg.GaussianScene.from_numpy(sc)
    poses = _poses(P)
    K = hg.Intrinsics.of(cam)
    r = hg.Renderer()
    ref = r.render(scene, poses, K)
    opts = r.opts()
    out = r.alloc_outputs(scene, 1, K)
    log("case: capacities of 64 records and 64 keys raise the overflow flags")
    st, flags = _noalloc(hg, scene, poses, K, opts, out, records=64, keys=64)
    assert st == 0 and flags != 0 and (flags & ~3) == 0, flags
    log("case: the next call with default capacities is complete and exact")
    st, flags = _noalloc(hg, scene, poses, K, opts, out)
    assert st == 0 and flags == 0
    _same(ref, out, "after an overflowing call")
    r.close()


def test_larger_tiles_need_less_scratch(hg):
    """The bytes a render needs, as its refusal states them: 20 per tile (two
    counters, a range, a loss share) beside what the tile size does not change,
    up to the scan's block sums (4 bytes per 4096 tiles) and 256-byte rounding
    of 20 buffers; so what fits the scratch at tile 32 does not depend on how
    the blend splits a tile."""
    import re
    import torch
    sc, P, _ = synth.terrain_20k_view(0)
    scene, r = hg.GaussianScene.from_numpy(sc), hg.Renderer()
    side = 4096
    K = hg.Intrinsics(3000.0, 3000.0, side / 2, side / 2, side, side)
    out = dict(rgb=torch.empty(1, device="cuda"), depth=torch.empty(1, device="cuda"),
               alpha=torch.empty(1, device="cuda"), feat=None)
    need = {}
    for tile in (16, 32):
        log(f"case: refused at tile {tile}")  # nothing is enqueued
        st, _ = _noalloc(hg, scene, _poses(P), K, r.opts(tile=tile), out, records=1 << 20, keys=1 << 22)
        assert st == 3
        need[tile] = int(re.search(r"needs (\d+) bytes", hg._lib.load().hgsr_last_error().decode()).group(1))
    tiles = {t: (side // t) ** 2 for t in need}
    diff = need[16] - need[32] - 20 * (tiles[16] - tiles[32])
    log("beyond 20 bytes per tile:", diff)
    assert abs(diff) <= 4 * (tiles[16] // 4096) + 20 * 256
    r.close()
