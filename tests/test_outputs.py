"""Output buffers that a caller supplies to a render: the library is told the
type that the feature buffer holds, and buffers too small for what the kernels
write are refused before it is called.  Host only: the library's entry is
replaced by one that records its arguments."""
import types

import pytest
import torch

import paper_2507_15683_amd as hg

P, D, W, H = 3, 16, 43, 21
K = hg.Intrinsics(30.0, 30.0, 21.5, 10.5, W, H)
STREAM = types.SimpleNamespace(cuda_stream=0)


class _Scene:
    n, feat_dim, sh_degree, device = 5, D, 0, torch.device("cpu")

    def c(self):
        return hg._lib.Gaussians()


@pytest.fixture
def rendered():
    """A Renderer over a recording library, and the options of its calls."""
    calls = []

    def render(ctx, g, poses, n, kc, opts, out, stream):
        calls.append(opts._obj.feat_out_bf16)
        return 0

    def autotune(ctx, g, poses, n, kc, opts, out, *rest):
        calls.append(opts._obj.feat_out_bf16)
        return 0

    r = object.__new__(hg.Renderer)
    r.ctx, r._keep = None, None
    r.lib = types.SimpleNamespace(hgsr_render=render, hgsr_autotune=autotune)
    return r, calls


def _render(r, out, **kw):
    return r.render(_Scene(), torch.zeros(P, 12), K, out=out, check_overflow=False, stream=STREAM, **kw)


@pytest.mark.parametrize("flag", [False, True])
@pytest.mark.parametrize("bf16", [False, True])
def test_feature_type_follows_the_buffer(rendered, bf16, flag):
    r, calls = rendered
    out = r.alloc_outputs(_Scene(), P, K, bf16)
    assert _render(r, out, feat_bf16=flag) is out
    assert calls == [int(bf16 or flag)]


def test_without_buffers_the_flag_decides(rendered):
    r, calls = rendered
    for flag in (False, True):
        out = _render(r, None, feat_bf16=flag)
        assert out["feat"].dtype == (torch.bfloat16 if flag else torch.float32)
    assert calls == [0, 1]


def test_fp32_features_into_a_bfloat16_buffer_are_refused(rendered):
    r, calls = rendered
    out = r.alloc_outputs(_Scene(), P, K, True)
    with pytest.raises(ValueError, match="feat"):
        r.render_into(_Scene(), torch.zeros(P, 12), K, out, r.opts(feat_bf16=False), STREAM)
    assert calls == []
    r.render_into(_Scene(), torch.zeros(P, 12), K, out, r.opts(feat_bf16=True), STREAM)
    assert calls == [1]


@pytest.mark.parametrize("name", ["rgb", "depth", "alpha", "feat"])
def test_short_buffers_are_refused(rendered, name):
    r, calls = rendered
    out = r.alloc_outputs(_Scene(), P, K)
    whole = out[name]
    for short in (torch.empty(whole.numel() - 1), torch.empty(whole.numel())[1:], whole[:1, ..., :1].clone().expand_as(whole)):
        with pytest.raises(ValueError, match=name):
            _render(r, dict(out, **{name: short}))
    assert calls == []
    _render(r, dict(out, **{name: torch.empty(whole.numel() + 7)[7:]}))
    assert calls == [0]


def test_no_feature_buffer_and_no_features(rendered):
    r, calls = rendered
    out = r.alloc_outputs(_Scene(), P, K)
    _render(r, dict(out, feat=None))
    assert calls == [0]


def test_autotune_buffers(rendered):
    r, calls = rendered
    tune = lambda out: r.autotune(_Scene(), torch.zeros(P, 12), K, out, stream=STREAM)  # noqa: E731
    for bf16 in (False, True):
        tune(r.alloc_outputs(_Scene(), P, K, bf16))
    assert calls == [0, 1]
    with pytest.raises(ValueError, match="depth"):
        tune(dict(r.alloc_outputs(_Scene(), P, K), depth=torch.empty(P * H * W - 1)))
    assert calls == [0, 1]
