"""The channel-minor form of the matrix-core kernel (PCONV_FLAG_NHWC: x [N][H][W][C], y [N][Ho][Wo][F]) against the
oracle: every tile shape and channel splits, tiles that run from one image into the next, a ragged last tile, both
strides and paddings, widths that make the 64-position pieces of the staging straddle rows, a library that leaves taps
unused; and what the form refuses."""
import numpy as np
import pytest

import oracle
import paper_2001_07710_amd as pc
from workloads import layers as L

from gpu_util import TOL, GpuLayer, rel_err

pytestmark = pytest.mark.gpu


def say(*a):
    print("[case]", *a, flush=True)


def run_nhwc(layer, x_nchw, relu, **tuning):
    import torch
    s = layer.spec
    N = x_nchw.shape[0]
    dx = torch.from_numpy(np.ascontiguousarray(x_nchw.transpose(0, 2, 3, 1))).cuda()
    n_out = N * s.F * s.Ho * s.Wo
    buf = torch.full((n_out + 8192,), -777.0, dtype=torch.float16, device="cuda")
    dy = buf[4096:4096 + n_out]
    flags = pc.FLAG_NHWC | (pc.FLAG_RELU if relu else 0)
    st = torch.cuda.current_stream().cuda_stream
    if tuning:
        pc.conv3x3_tuned(dx, dy, layer.packed, layer.d_bias, N, s.H, s.W, s.stride, s.pad, flags, st, **tuning)
    else:
        pc.conv3x3(dx, dy, layer.packed, layer.d_bias, N, s.H, s.W, s.stride, s.pad, flags, st)
    torch.cuda.synchronize()
    out = buf.cpu().numpy()
    assert np.all(out[:4096] == -777.0) and np.all(out[4096 + n_out:] == -777.0), "write outside the output buffer"
    return out[4096:4096 + n_out].reshape(N, s.Ho, s.Wo, s.F).transpose(0, 3, 1, 2)


SHAPES = [  # N, C, F, H, W, stride, pad
    (3, 40, 72, 13, 28, 1, 1),      # 13 rows: tiles cross images; F ragged against 32 and 128
    (2, 32, 136, 9, 12, 1, 1),      # two filter tiles of 128, the second nearly empty
    (5, 16, 64, 7, 7, 1, 1),        # several images per tile
    (33, 24, 40, 7, 7, 1, 1),       # more images than one tile holds
    (2, 24, 32, 14, 14, 1, 1),
    (2, 32, 16, 15, 18, 2, 1),      # stride 2, odd height
    (3, 8, 8, 16, 16, 2, 0),        # stride 2, no padding
    (1, 8, 16, 5, 130, 1, 0),       # no padding, a row wider than a 128-pixel operand group
    (2, 64, 8, 8, 8, 1, 0),
    (1, 8, 8, 1, 1, 1, 1),          # a single pixel
    (2, 8, 64, 30, 224, 1, 1),      # a first layer (channels padded to eight) at full width
    (2, 48, 96, 20, 56, 2, 1),
    (4, 128, 128, 28, 28, 1, 1),
]


@pytest.mark.parametrize("case", SHAPES, ids=[f"n{c[0]}c{c[1]}f{c[2]}h{c[3]}w{c[4]}s{c[5]}p{c[6]}" for c in SHAPES])
def test_channel_minor_form(case):
    N, C, F, H, W, stride, pad = case
    spec = L.LayerSpec(cfg=50, idx=SHAPES.index(case), name="nhwc", N=N, C=C, F=F, H=H, W=W, stride=stride, pad=pad,
                       dtype="f16", K=8, keep=0.4)
    layer = GpuLayer(spec)
    x = L.gen_activations(spec)
    ref = layer.oracle(x, True)
    forms = [{}] + [dict(mfma_shape=s, channel_splits=k) for s in (1, 2, 3, 4) for k in (1, 2)]
    ran = 0
    for t in forms:
        say(case, t)
        try:
            got = run_nhwc(layer, x, True, **t)
        except pc.PconvError as e:
            assert e.code == pc.EUNSUPPORTED and t, (case, t, e.code)
            say("  unsupported")
            continue
        ran += 1
        err = rel_err(got, ref)
        assert err <= TOL["f16"], (case, t, err)
    assert ran >= 3
    assert rel_err(run_nhwc(layer, x, False), layer.oracle(x, False)) <= TOL["f16"]
    layer.free()


# Nine taps and two blocks of channels or more: the kernel walks its tiles as one sequence of K steps with three buffers of
# activations.  Five tiles or more for some workgroups, so that every buffer is written again; a last half block of channels;
# one and two loads of pixels a lane and block; the last column is the shapes that run the row in sequence (test_host_logic.py
# holds the table to it).  Then the shapes above whose library, another one, uses every tap.
SEQUENCE = [  # N, C, F, H, W, stride, pad, shapes
    (145, 24, 16, 57, 56, 1, 1, (1, 2, 3)),     # tiles cross rows and images
    (566, 40, 8, 29, 28, 1, 1, (1, 2, 3)),      # three blocks
    (73, 40, 8, 29, 150, 1, 1, (2, 3)),         # 64 x 448: two loads of pixels
    (70, 40, 8, 29, 204, 2, 1, (1, 3)),         # stride 2, a window of twice the pixels
    (206, 40, 8, 20, 192, 2, 1, (2,)),
    (19, 24, 8, 224, 224, 2, 1, (1,)),
    (2345, 32, 40, 14, 14, 1, 1, (2, 3)),       # several images a tile, filters that end inside a wave's 32
    (206, 24, 8, 20, 220, 1, 0, (2, 3)),        # no padding
] + [c for c in SHAPES if c[1] > 16]


@pytest.mark.parametrize("case", SEQUENCE, ids=lambda c: f"n{c[0]}c{c[1]}h{c[3]}w{c[4]}s{c[5]}p{c[6]}")
def test_many_tiles_in_sequence(case):
    N, C, F, H, W, stride, pad = case[:7]
    spec = L.LayerSpec(cfg=23, idx=80 + SEQUENCE.index(case), name="nhwc sequence", N=N, C=C, F=F, H=H, W=W, stride=stride,
                       pad=pad, dtype="f16", K=8, keep=0.4)
    layer = GpuLayer(spec)
    assert np.all(np.bitwise_or.reduce(layer.lib) == 0x1FF)
    x = L.gen_activations(spec)
    ref = layer.oracle(x, True)
    for shape in (1, 2, 3):
        say(case, shape)
        assert rel_err(run_nhwc(layer, x, True, mfma_shape=shape), ref) <= TOL["f16"]
    layer.free()


def test_unused_taps_and_equality_with_the_channel_major_form():
    # a library whose masks all lie in the upper two kernel rows: three tap slots are never staged
    spec = L.LayerSpec(cfg=50, idx=40, name="nhwc", N=3, C=32, F=64, H=12, W=20, dtype="f16", K=4, keep=0.5,
                       lib_kind="fixed4")
    spec = L.LayerSpec(**{**spec.__dict__, "K": 2})
    layer = GpuLayer(spec)
    x = L.gen_activations(spec)
    got = run_nhwc(layer, x, False)
    assert rel_err(got, layer.oracle(x, False)) <= TOL["f16"]
    # both forms multiply the same operands in the same order: equal bit for bit
    assert np.array_equal(got, layer.run(x, False))
    layer.free()


@pytest.mark.parametrize("case", [  # N, C, F, H, W, stride, pad, every tap used
    (3, 24, 40, 9, 12, 1, 1, True),       # two blocks of channels, the second half full
    (2, 8, 32, 10, 20, 1, 1, True),       # half a block
    (2, 40, 72, 15, 18, 2, 1, True),
    (3, 24, 16, 9, 12, 1, 0, False),
    (700, 24, 8, 14, 14, 1, 1, False),    # several tiles a workgroup
    (700, 24, 8, 14, 14, 1, 1, True),
], ids=lambda c: f"n{c[0]}c{c[1]}h{c[3]}w{c[4]}s{c[5]}p{c[6]}{'' if c[7] else 'u'}")
def test_infinities_stay_in_their_windows(case):
    """A last block of eight channels: in memory the next pixel's first channels lie where its other eight would, and an
    infinity there must not reach outputs whose window holds the pixel before only (at the ends of rows and images too)."""
    N, C, F, H, W, stride, pad, full = case
    spec = L.LayerSpec(cfg=23, idx=90, name="nhwc", N=N, C=C, F=F, H=H, W=W, stride=stride, pad=pad, dtype="f16", K=8,
                       keep=0.4)
    if not full:
        spec = L.LayerSpec(**{**spec.__dict__, "K": 2, "lib_kind": "fixed4"})
    layer = GpuLayer(spec)
    assert np.all(np.bitwise_or.reduce(layer.lib) == 0x1FF) == full
    clean = L.gen_activations(spec)
    ref = layer.oracle(clean)
    x, inside = clean.copy(), np.zeros((N, spec.Ho, spec.Wo), bool)
    for n, iy, ix, c in ((0, 4, 6, 0), (0, 7, 0, 7), (N - 1, 0, 0, 3), (N - 2, H - 1, 3, 1)):
        x[n, c, iy, ix] = np.inf
        oy, ox = np.arange(spec.Ho) * stride - pad, np.arange(spec.Wo) * stride - pad
        inside[n] |= ((oy <= iy) & (iy <= oy + 2))[:, None] & ((ox <= ix) & (ix <= ox + 2))[None, :]
    outside = np.broadcast_to(~inside[:, None], ref.shape)
    ran = 0
    for t in [{}] + [dict(mfma_shape=s, channel_splits=k) for s in (1, 2, 3, 4) for k in (1, 2)]:
        say(case, t)
        try:
            want = run_nhwc(layer, clean, False, **t)
        except pc.PconvError as e:
            assert e.code == pc.EUNSUPPORTED and t, (case, t, e.code)
            continue
        ran += 1
        assert rel_err(want, ref) <= TOL["f16"]
        got = run_nhwc(layer, x, False, **t)
        assert not np.isfinite(got).all()
        assert np.array_equal(got[outside], want[outside]), (case, t)
    assert ran >= 4
    layer.free()


def test_what_the_form_refuses():
    import torch
    one = torch.zeros(4096, dtype=torch.float16, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    def refused(spec, **kw):
        layer = GpuLayer(spec)
        with pytest.raises(pc.PconvError) as e:
            pc.conv3x3(one, one[2048:], layer.packed, None, 1, 4, 4, 1, 1, pc.FLAG_NHWC, st)
        assert e.value.code == pc.EUNSUPPORTED
        layer.free()
    refused(L.LayerSpec(cfg=50, idx=60, name="nhwc", N=1, C=12, F=16, H=4, W=4, dtype="f16", K=8, keep=0.5))   # C % 8
    refused(L.LayerSpec(cfg=50, idx=61, name="nhwc", N=1, C=16, F=12, H=4, W=4, dtype="f16", K=8, keep=0.5))   # F % 8
    refused(L.LayerSpec(cfg=50, idx=62, name="nhwc", N=1, C=16, F=16, H=4, W=4, dtype="f32", K=8, keep=0.5))   # fp32
    layer = GpuLayer(L.LayerSpec(cfg=50, idx=63, name="nhwc", N=1, C=16, F=16, H=4, W=4, dtype="f16", K=8, keep=0.5))
    with pytest.raises(pc.PconvError) as e:                                          # a pointer that is not 16-byte aligned
        pc.conv3x3(one[1:], one[2048:], layer.packed, None, 1, 4, 4, 1, 1, pc.FLAG_NHWC, st)
    assert e.value.code == pc.EUNSUPPORTED
    layer.free()
    torch.cuda.synchronize()


@pytest.mark.parametrize("name", ["conv1_2", "conv3_2", "conv5_1"])
def test_channel_minor_form_at_benchmark_shapes(name):
    # config 4 at batch 64 (K = 8, keep 0.28), as bench.py --nhwc launches it: the first and the last image whole,
    # and 65,536 outputs sampled over the batch
    spec = [s for s in L.config4(8, 0.28, 64) if s.name == name][0]
    say("nhwc full", name)
    layer = GpuLayer(spec)
    base = L.gen_activations(spec, images=[0, 1, 2, 3])
    x = np.concatenate([base] * (spec.N // 4), axis=0)
    x[spec.N - 1] = L.gen_image(spec, spec.N - 1)
    got = run_nhwc(layer, x, spec.relu)
    ref_first, ref_last = layer.oracle(x[:1]), layer.oracle(x[spec.N - 1:])
    tol = TOL["f16"]
    assert rel_err(got[0], ref_first[0]) <= tol and rel_err(got[spec.N - 1], ref_last[0]) <= tol
    rng = np.random.default_rng(77 + spec.idx)
    coords = np.stack([rng.integers(0, spec.N, 65536), rng.integers(0, spec.F, 65536), rng.integers(0, spec.Ho, 65536),
                       rng.integers(0, spec.Wo, 65536)], axis=1).astype(np.int32)
    ref_pts = layer.oracle_at(x, coords)
    pts = got[coords[:, 0], coords[:, 1], coords[:, 2], coords[:, 3]].astype(np.float64)
    rms = float(np.sqrt(np.mean(ref_first ** 2)))
    assert np.max(np.abs(pts - ref_pts) / np.maximum(np.abs(ref_pts), rms)) <= tol
    layer.free()


@pytest.mark.parametrize("shape", [2, 4])
def test_equal_images_give_equal_outputs(shape):
    """Every image of the batch is the same, so are its outputs, bit for bit: a store whose data registers are written
    again before it has read them shows as an image that differs.  Six taps and 64 filters: two workgroups fit a compute
    unit and keep the path of the stores busy."""
    spec = L.LayerSpec(cfg=50, idx=70, name="nhwc", N=1, C=16, F=64, H=28, W=28, dtype="f16", K=2, keep=0.5, lib_kind="fixed4")
    layer = GpuLayer(spec)
    one = L.gen_activations(spec)
    x = np.concatenate([one] * 96, axis=0)
    ref = layer.oracle(one, True)
    for _ in range(3):
        y = run_nhwc(layer, x, True, mfma_shape=shape)
        assert np.array_equal(y, np.broadcast_to(y[:1], y.shape))
        assert rel_err(y[0], ref[0]) <= TOL["f16"]
    layer.free()
