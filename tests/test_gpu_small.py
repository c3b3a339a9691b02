"""The matrix-core kernel for layers of few tiles (mfma_shape 5, 6, 7; channel_splits = waves that share a tile) against
the oracle: every shape with one to eight waves, sizes around its tiles (32 or 64 filters, 32 or 64 pixels), channel
counts around its blocks and its steps of four blocks, rows that allow loads of four, two and one pixels, both strides
and paddings, both layouts, channel lists, 1x1 layers."""
import numpy as np
import pytest

import oracle
import paper_2001_07710_amd as pc
from workloads import layers as L

from gpu_util import TOL, GpuLayer, rel_err
from test_gpu_nhwc import run_nhwc

pytestmark = pytest.mark.gpu
M = pc.KERNEL_MFMA


def say(*a):
    print("[case]", *a, flush=True)


SHAPES = [  # N, C, F, H, W, stride, pad
    (1, 16, 32, 4, 8, 1, 1), (1, 3, 1, 1, 1, 1, 1), (2, 17, 33, 5, 9, 1, 1), (1, 136, 65, 8, 64, 1, 1),
    (3, 40, 31, 7, 7, 1, 1), (1, 200, 64, 9, 33, 1, 0), (2, 24, 40, 13, 12, 2, 1), (1, 72, 96, 16, 28, 2, 1),
    (2, 64, 24, 11, 30, 2, 0), (1, 8, 70, 3, 225, 1, 1), (1, 32, 16, 40, 56, 1, 1)]


@pytest.mark.parametrize("case", SHAPES, ids=["n%dc%df%dh%dw%ds%dp%d" % c for c in SHAPES])
def test_every_shape_and_number_of_waves(case):
    N, C, F, H, W, stride, pad = case
    spec = L.LayerSpec(cfg=36, idx=SHAPES.index(case), name="small", N=N, C=C, F=F, H=H, W=W, stride=stride, pad=pad,
                       dtype="f16", K=12, keep=0.4)
    layer = GpuLayer(spec)
    x = L.gen_activations(spec)
    for relu in (False, True):
        ref = layer.oracle(x, relu)
        for shape in (5, 6, 7):
            for waves in (0, 1, 2, 4, 8):
                say(case, shape, waves, relu)
                try:
                    got = layer.run(x, relu, kernel=M, mfma_shape=shape, channel_splits=waves)
                except pc.PconvError as e:
                    # (a patch that does not fit the loads or the LDS of so many waves; the automatic number always does)
                    assert e.code == pc.EUNSUPPORTED and (waves == 8 or waves > (C + 15) // 16)
                    continue
                assert rel_err(got, ref) <= TOL["f16"], (case, shape, waves)
        assert rel_err(layer.run(x, relu), ref) <= TOL["f16"]
    for xs, ys in ((1, 0), (2, 3), (0, 2)):              # narrower loads, narrower stores
        say(case, "x shifted by", xs, "y by", ys)
        assert rel_err(layer.run(x, True, x_shift=xs, y_shift=ys, kernel=M, mfma_shape=6), layer.oracle(x, True)) <= TOL["f16"]
    layer.free()


@pytest.mark.parametrize("case", [(1, 16, 32, 4, 8, 1), (2, 24, 40, 7, 9, 1), (3, 136, 72, 14, 14, 1), (2, 64, 16, 9, 15, 2),
                                  (1, 8, 96, 20, 56, 1)])
def test_channel_minor_layout(case):
    N, C, F, H, W, stride = case
    spec = L.LayerSpec(cfg=37, idx=C + F, name="smallnhwc", N=N, C=C, F=F, H=H, W=W, stride=stride, dtype="f16", K=8, keep=0.6)
    layer = GpuLayer(spec)
    x = L.gen_activations(spec)
    ref = layer.oracle(x, True)
    for shape in (5, 6, 7):
        for waves in (0, 1, 4):
            if waves > (C + 15) // 16:
                continue
            say("nhwc", case, shape, waves)
            assert rel_err(run_nhwc(layer, x, True, kernel=M, mfma_shape=shape, channel_splits=waves), ref) <= TOL["f16"]
    assert rel_err(run_nhwc(layer, x, True), ref) <= TOL["f16"]
    layer.free()


def test_channel_lists_and_few_taps():
    spec = L.LayerSpec(cfg=38, idx=1, name="smalllists", N=2, C=200, F=128, H=9, W=12, dtype="f16", K=8, keep=0.1)
    w, _ = L.gen_clustered_weights(spec, 4, 0.2)
    order = None
    layer = GpuLayer(spec, w=w)
    order = pc.filter_similarity_order(layer.mask, 64)
    layer = GpuLayer(spec, w=w[order])
    listed, blocks = pc.packed_mfma_blocks(layer.packed, 64)
    assert listed < blocks                               # (the layer has channel lists)
    x = L.gen_activations(spec)
    ref = layer.oracle(x, False)
    for shape in (5, 6, 7):
        say("lists", shape)
        assert rel_err(layer.run(x, False, kernel=M, mfma_shape=shape), ref) <= TOL["f16"]
    layer.free()
    # one pattern: four of the nine taps occur
    spec = L.LayerSpec(cfg=38, idx=2, name="fourtaps", N=2, C=48, F=40, H=9, W=12, dtype="f16", K=1, keep=0.5, lib_kind="all126")
    layer = GpuLayer(spec)
    x = L.gen_activations(spec)
    for shape in (5, 6, 7):
        say("four taps", shape)
        assert rel_err(layer.run(x, False, kernel=M, mfma_shape=shape), layer.oracle(x, False)) <= TOL["f16"]
    layer.free()


@pytest.mark.parametrize("case", [(1, 16, 32, 1, 1, 1), (2, 40, 33, 7, 7, 1), (1, 72, 130, 14, 14, 1), (2, 200, 64, 10, 9, 2),
                                  (3, 64, 24, 8, 16, 2), (1, 528, 40, 6, 10, 1)])
@pytest.mark.parametrize("nhwc", [False, True])
def test_1x1_layers(case, nhwc):
    import torch
    N, C, F, H, W, stride = case
    if nhwc and F % 8:
        F = 40
    r = np.random.default_rng(C + F + H)
    G = -(-C // 9)
    w = (r.standard_normal((F, C)) * np.sqrt(2.0 / C)).astype(np.float16)
    lib = np.array(L.drawn_library(4, 8), dtype=np.uint16)
    pid = r.integers(0, 8, (F, G)).astype(np.uint8)
    mask = (r.random((F, G)) < 0.6).astype(np.uint8)
    p = pc.pack_1x1(w, lib, pid, mask)
    x = np.maximum(r.standard_normal((N, C, H, W)), 0).astype(np.float16)
    b = (r.standard_normal(F) * 0.1).astype(np.float32)
    ref = oracle.conv1x1(x, w, pid, mask, lib, b, stride)
    Ho, Wo = ref.shape[2:]
    dx = torch.from_numpy(np.ascontiguousarray(x.transpose(0, 2, 3, 1)) if nhwc else x).cuda()
    st = torch.cuda.current_stream().cuda_stream
    for shape in (0, 5, 6, 7):
        for waves in (0, 1, 2) if shape else (0,):
            if waves > (C + 63) // 64:
                continue
            say("1x1", case, nhwc, shape, waves)
            dy = torch.full((N * F * Ho * Wo + 64,), -7.0, dtype=torch.float16, device="cuda")
            pc.conv3x3_tuned(dx, dy, p, torch.from_numpy(b).cuda(), N, H, W, stride, 1, pc.FLAG_NHWC if nhwc else 0, st,
                             kernel=M if shape else 0, mfma_shape=shape, channel_splits=waves)
            torch.cuda.synchronize()
            out = dy.cpu().numpy()
            assert np.all(out[N * F * Ho * Wo:] == -7.0)
            got = out[:N * F * Ho * Wo]
            got = got.reshape(N, Ho, Wo, F).transpose(0, 3, 1, 2) if nhwc else got.reshape(N, F, Ho, Wo)
            assert rel_err(got, ref) <= TOL["f16"], (case, shape, waves)
    p.free()


def test_the_choice_is_the_same_on_every_call():
    """The handle keeps what the automatic choice came to; results are bit-equal from call to call, on a call that finds its
    size kept and on one that does not because more sizes than the handle keeps have come by in between."""
    spec = L.LayerSpec(cfg=39, idx=1, name="choice", N=1, C=64, F=48, H=14, W=14, dtype="f16", K=8, keep=0.3)
    layer = GpuLayer(spec)
    x = L.gen_activations(spec)
    first = layer.run(x, True)
    for round_ in range(2):
        assert np.array_equal(layer.run(x, True).view(np.uint16), first.view(np.uint16))      # (kept)
        for h in range(3, 73):                               # (70 sizes, the handle keeps 64)
            sub = L.shrink(spec, H=h, W=h + 1)
            layer.spec = sub
            xs = L.gen_activations(sub)
            a = layer.run(xs, True)
            assert np.array_equal(layer.run(xs, True).view(np.uint16), a.view(np.uint16))     # (kept)
            if h < 24:
                assert rel_err(a, layer.oracle(xs, True)) <= TOL["f16"]
        layer.spec = spec
        assert np.array_equal(layer.run(x, True).view(np.uint16), first.view(np.uint16))      # (found again)
    layer.free()


@pytest.mark.parametrize("outcome,N,C,F,H,W,pad", [("few", 1, 64, 48, 14, 14, 1), ("few", 2, 256, 40, 9, 11, 0), ("tile", 8, 256, 256, 56, 56, 1),
                                                   ("vector", 1, 227, 16, 224, 224, 0)])
def test_a_kept_choice_runs_the_launch_it_was_made_for(outcome, N, C, F, H, W, pad):
    """Every outcome of the choice, made and then found again, with other layouts and alignments of the same size in between."""
    import torch
    say("kept choice", outcome, N, C, F, H, W)
    r = np.random.default_rng(C)
    lib = np.array([0x1B, 0x36, 0xB1, 0x72], dtype=np.uint16)           # (eight taps)
    p = pc.pack((r.standard_normal((F, C, 3, 3)) * np.sqrt(2.0 / (9 * C))).astype(np.float16), lib,
                r.integers(0, 4, (F, C)).astype(np.uint8), (r.random((F, C)) < (0.1 if outcome == "vector" else 0.2)).astype(np.uint8))
    kernel, shape = pc.conv3x3_choice(p, N, H, W, 1, pad)
    assert {"few": kernel == M and shape >= 5, "tile": kernel == M and shape < 5, "vector": kernel != M}[outcome]
    Ho, Wo = H + 2 * pad - 2, W + 2 * pad - 2
    g = torch.Generator(device="cuda").manual_seed(C)
    x = torch.randn((N, C, H, W), generator=g, device="cuda").half()
    bias = torch.randn((F,), generator=g, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    want = torch.empty((N, F, Ho, Wo), dtype=torch.float16, device="cuda")
    pc.conv3x3_tuned(x, want, p, bias, N, H, W, 1, pad, 0, st, kernel=pc.KERNEL_GENERIC)
    want = want.cpu().numpy()

    def run(x_shift=0, y_shift=0, nhwc=False):
        xs = x.permute(0, 2, 3, 1).contiguous() if nhwc else x
        xb = torch.zeros(xs.numel() + x_shift, dtype=torch.float16, device="cuda")
        xb[x_shift:] = xs.reshape(-1)
        yb = torch.full((N * F * Ho * Wo + y_shift + 64,), -777.0, dtype=torch.float16, device="cuda")
        pc.conv3x3(xb[x_shift:], yb[y_shift:], p, bias, N, H, W, 1, pad, pc.FLAG_NHWC if nhwc else 0, st)
        torch.cuda.synchronize()
        y = yb.cpu().numpy()
        n = N * F * Ho * Wo
        assert np.all(y[:y_shift] == -777.0) and np.all(y[y_shift + n:] == -777.0)
        y = y[y_shift:y_shift + n]
        y = y.reshape(N, Ho, Wo, F).transpose(0, 3, 1, 2) if nhwc else y.reshape(N, F, Ho, Wo)
        assert rel_err(y, want) <= TOL["f16"]
        return np.ascontiguousarray(y).view(np.uint16)

    forms = [dict(), dict(x_shift=1), dict(x_shift=2, y_shift=1), dict(y_shift=2), dict(x_shift=4, y_shift=4)]
    if C % 8 == 0 and pad == 1:
        forms.append(dict(nhwc=True))
    made = [run(**f) for f in forms]
    for round_ in range(2):
        for f, m in zip(forms, made):
            assert np.array_equal(run(**f), m), f
    p.free()


@pytest.mark.parametrize("case", [(512, 40, 7, 7), (500, 33, 7, 9), (700, 24, 5, 5)])
def test_many_channels_on_a_small_map_by_the_automatic_choice(case):
    C, F, H, W = case
    spec = L.LayerSpec(cfg=39, idx=C, name="smalldeep", N=1, C=C, F=F, H=H, W=W, dtype="f16", K=8, keep=0.3)
    layer = GpuLayer(spec)
    x = L.gen_activations(spec)
    say("deep", case)
    kernel, shape = pc.conv3x3_choice(layer.packed, 1, H, W, 1, 1)
    assert kernel == M and shape >= 5
    assert rel_err(layer.run(x, True), layer.oracle(x, True)) <= TOL["f16"]
    layer.free()


@pytest.mark.parametrize("case", [  # N, C, F, H, W, stride, K, keep
    (1, 7, 224, 224, 224, 1, 12, 0.35), (4, 8, 224, 224, 224, 1, 8, 0.35), (6, 9, 480, 144, 144, 1, 8, 0.3),
    (17, 6, 93, 50, 76, 1, 8, 0.28), (4, 16, 46, 224, 224, 1, 8, 0.28), (31, 4, 160, 99, 64, 2, 12, 0.15),
    (24, 18, 191, 42, 35, 2, 4, 0.15), (53, 4, 336, 56, 56, 2, 12, 0.2), (3, 32, 48, 60, 55, 2, 4, 0.2)])
def test_layers_of_few_channels_and_many_tiles_stay_on_the_matrix_cores(case):
    """A layer whose tile kernel is expected to beat the vector kernels is not given to them because a third kernel is
    there to compare with; at stride 2 the non-allocating entry takes such a layer on its first call."""
    import torch
    N, C, F, H, W, stride, K, keep = case
    spec = L.LayerSpec(cfg=40, idx=C + F, name="fewchannels", N=N, C=C, F=F, H=H, W=W, stride=stride, dtype="f16", K=K, keep=keep)
    layer = GpuLayer(spec)
    say("few channels", case)
    kernel, _ = pc.conv3x3_choice(layer.packed, N, H, W, stride, 1)
    assert kernel == M
    x = torch.zeros((N, C, H, W), dtype=torch.float16, device="cuda")
    y = torch.full((N, F, spec.Ho, spec.Wo), -7.0, dtype=torch.float16, device="cuda")
    pc.conv3x3_noalloc(x, y, layer.packed, layer.d_bias, N, H, W, stride, 1, 0, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert bool((y == layer.d_bias.half()[None, :, None, None]).all())      # zero input: the bias alone
    layer.free()


@pytest.mark.parametrize("case", [(2, 1844, 96, 224, 224, 0.35), (1, 1104, 219, 224, 224, 0.5), (17, 1680, 768, 32, 32, 0.3),
                                  (1, 419, 208, 224, 224, 0.28), (11, 1082, 114, 32, 32, 0.28)])
def test_1x1_layers_whose_planes_crowd_the_cache_are_priced_as_such(case):
    """Planes a multiple of 2 KB apart: small tiles, which read them over and over, are not what such a layer gets."""
    N, C, F, H, W, keep = case
    say("crowded planes", case)
    r = np.random.default_rng(C + F)
    G = -(-C // 9)
    p = pc.pack_1x1(r.standard_normal((F, C)).astype(np.float16), np.array(L.drawn_library(4, 8), dtype=np.uint16),
                    r.integers(0, 8, (F, G)).astype(np.uint8), (r.random((F, G)) < keep).astype(np.uint8))
    kernel, shape = pc.conv3x3_choice(p, N, H, W, 1, 1)                 # (a 1x1 layer is a 3x3 one of centre taps)
    assert kernel == M and shape not in (5, 6) and (shape != 7 or H == 32)
    p.free()


@pytest.mark.parametrize("case", [  # N, C, F, H, W
    (2, 160, 512, 127, 127), (4, 96, 96, 158, 158), (25, 226, 208, 43, 57), (32, 149, 144, 45, 61), (1, 96, 448, 167, 150),
    (2, 128, 384, 121, 121)])
def test_rows_that_only_narrow_loads_divide_are_priced_as_such(case):
    """Nine taps, rows of an odd number of pixels or of pairs: small tiles took 67, 33, 103, 75, 36 and 47 us on these layers,
    128 x 224 tiles 111, 50, 152, 100, 52 and 65 (and the other large tiles more)."""
    N, C, F, H, W = case
    say("narrow rows", case)
    r = np.random.default_rng(C + F)
    lib = L.drawn_library(23, 8)
    assert np.bitwise_or.reduce(lib) == 0x1FF
    p = pc.pack((r.standard_normal((F, C, 3, 3)) * 0.05).astype(np.float16), lib, r.integers(0, 8, (F, C)).astype(np.uint8),
                (r.random((F, C)) < 0.28).astype(np.uint8))
    kernel, shape = pc.conv3x3_choice(p, N, H, W, 1, 1)
    assert kernel == M and shape >= 5
    p.free()
