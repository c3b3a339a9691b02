"""The work that a user of libpconv has it do, as measurable cases: one pass each through the public entry points of
paper_2001_07710_amd, over the ranges of sizes, storage types, layouts and directions the library is used with.

Kinds of work
  conv      one pruned 3x3 layer, forward (inference): fp32 or fp16 storage, channel-major or channel-minor tensors,
            either stride and padding, uniform or clustered connectivity
  conv1x1   one pruned 1x1 layer, forward
  chain     the thirteen 3x3 layers of VGG-16 with the five max-pools between them, one after the other
  backward  input gradient and masked weight gradient of one layer whose weights are packed already
  train     one weight update's worth of work of one layer: packing of the new weights and of the transposed layer,
            forward, input gradient, weight gradient
  select    one iteration of the pruning framework over the kernels of a network: proximal step with multiplier
            update, pattern assignment, argmax projection, connectivity selection
"""
import math

import numpy as np
import torch

import paper_2001_07710_amd as pc

#: (input channels, filters, map size in 224ths, max-pool behind) of VGG-16's layers, channels in units of 64
VGG16 = [(0, 1, 224, False), (1, 1, 224, True), (1, 2, 112, False), (2, 2, 112, True), (2, 4, 56, False),
         (4, 4, 56, False), (4, 4, 56, True), (4, 8, 28, False), (8, 8, 28, False), (8, 8, 28, True),
         (8, 8, 14, False), (8, 8, 14, False), (8, 8, 14, True)]
#: kernels kept per layer: all in the first, fewer with depth
VGG16_KEEP = [1.0, 0.35, 0.35, 0.35, 0.28, 0.28, 0.28, 0.2, 0.2, 0.2, 0.2, 0.2, 0.2]

CENTRE_MASKS = np.array([m for m in range(512) if bin(m).count("1") == 4 and (m >> 4) & 1], dtype=np.uint16)


def _conv(name, dtype, N, C, F, H, W, stride=1, pad=1, K=8, keep=0.28, relu=True, layout="nchw", clusters=0):
    c = {"kind": "conv", "dtype": dtype, "layout": layout, "N": N, "C": C, "F": F, "H": H, "W": W, "stride": stride,
         "pad": pad, "K": K, "keep": keep, "relu": relu, "clusters": clusters}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest layer anyone calls: a launch and its latency
        _conv("tiny_f32", "f32", 1, 16, 16, 32, 32, K=4, keep=0.5, relu=False),
        # real-time inference on single images, the paper's own use: the whole network in fp32
        {"name": "vgg16_chain_f32", "kind": "chain", "dtype": "f32", "N": 1, "side": 224, "width": 64},
        # one image through a deep bottleneck layer: few tiles, many channels
        _conv("res256_14_n1_f16", "f16", 1, 256, 256, 14, 14, keep=0.3),
        # a batch through a bottleneck layer that halves the map
        _conv("res128_56_s2_n32_f16", "f16", 32, 128, 128, 56, 56, stride=2, keep=0.3),
        # throughput serving: the layer with the most outputs, and the typical middle layer
        _conv("vgg64_224_n64_f16", "f16", 64, 64, 64, 224, 224),
        _conv("vgg256_56_n64_f16", "f16", 64, 256, 256, 56, 56),
        # the same kind of serving from a program whose tensors are channel-minor
        _conv("vgg128_112_n64_nhwc", "f16", 64, 128, 128, 112, 112, layout="nhwc"),
        # sizes that no tile divides: a crop, odd channel counts, no padding
        _conv("ragged_f16", "f16", 5, 100, 72, 37, 61, pad=0, K=12, keep=0.4),
        # the 1x1 layers around the bottleneck's 3x3
        {"name": "conv1x1_1024_256_14_n32", "kind": "conv1x1", "dtype": "f16", "layout": "nchw", "N": 32, "C": 1024,
         "F": 256, "H": 14, "W": 14, "stride": 1, "keep": 0.3},
        # fine-tuning: gradients of a layer at the batch of the throughput case
        {"name": "backward_vgg128_112_n64", "kind": "backward", "N": 64, "C": 128, "F": 128, "H": 112, "W": 112,
         "K": 8, "keep": 0.28},
        # fine-tuning with the weights just updated: everything a step asks of the library for one layer
        {"name": "train_res256_14_n32", "kind": "train", "N": 32, "C": 256, "F": 256, "H": 14, "W": 14, "K": 8,
         "keep": 0.3},
        # pruning: selection over all 3x3 kernels of VGG-16
        {"name": "select_vgg16", "kind": "select", "dtype": "f32", "n": 1634496, "K": 8, "keep": 0.28},
    ]


# -------------------------------------------------------------------------------------------- more of the same ranges

def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo, hi, of=1):
    """A count spread over its logarithm; two thirds of the time a multiple of 16, as networks have them."""
    n = _log(rng, lo, hi)
    of = max(of, 16 if rng.random() < 0.67 and n >= 16 else 1)
    return max(of, (n + of // 2) // of * of)


def _map(rng):
    """Height and width of a map: two thirds of the time one of the square maps of the usual networks."""
    if rng.random() < 0.67:
        s = rng.choice([7, 14, 28, 32, 56, 112, 224])
        return s, s
    h = _log(rng, 7, 224)
    return h, max(7, min(224, int(round(h * rng.uniform(0.6, 1.7)))))


def _dense_macs(c):
    s = c.get("stride", 1)
    return c["N"] * c["C"] * c["F"] * (c["H"] / s) * (c["W"] / s) * (1 if c["kind"] == "conv1x1" else 9)


def _elements(c):
    return c["N"] * c["H"] * c["W"] * max(c["C"], c["F"])


def draw(rng):
    kind = rng.choice(["conv_f32", "conv_f16", "conv_f16", "conv_f16", "conv_nhwc", "conv1x1", "backward", "train",
                       "chain", "select"])
    while True:
        K, keep = rng.choice([4, 8, 12]), rng.choice([0.15, 0.2, 0.28, 0.3, 0.35, 0.5])
        H, W = _map(rng)
        if kind == "conv_f32":
            c = _conv("", "f32", rng.choice([1, 1, 1, _log(rng, 2, 16)]), _channels(rng, 3, 512),
                      _channels(rng, 16, 512), H, W, rng.choice([1, 1, 1, 2]), rng.choice([1, 1, 1, 0]), K, keep,
                      rng.random() < 0.7)
            most = 16e9
        elif kind == "conv_f16":
            c = _conv("", "f16", rng.choice([1, _log(rng, 1, 64)]), _channels(rng, 3, 512), _channels(rng, 16, 512), H,
                      W, rng.choice([1, 1, 1, 2]), rng.choice([1, 1, 1, 0]), K, keep, rng.random() < 0.7,
                      clusters=rng.choice([0, 0, 0, 0, 4]))
            most = 1.2e11
        elif kind == "conv_nhwc":
            c = _conv("", "f16", _log(rng, 1, 64), _channels(rng, 8, 512, of=8), _channels(rng, 16, 512, of=8), H, W,
                      rng.choice([1, 1, 1, 2]), 1, K, max(keep, 0.28), rng.random() < 0.7, layout="nhwc")
            most = 1.2e11
        elif kind == "conv1x1":
            nhwc = rng.random() < 0.3
            c = {"kind": "conv1x1", "dtype": "f16", "layout": "nhwc" if nhwc else "nchw", "N": _log(rng, 1, 64),
                 "C": _channels(rng, 32, 2048, of=8 if nhwc else 1), "F": _channels(rng, 32, 2048, of=8 if nhwc else 1),
                 "H": H, "W": W, "stride": rng.choice([1, 1, 1, 2]), "keep": max(keep, 0.28)}
            most = 3e10
        elif kind in ("backward", "train"):
            c = {"kind": kind, "N": _log(rng, 1, 64), "C": _channels(rng, 16, 512), "F": _channels(rng, 16, 512),
                 "H": H, "W": W, "K": K, "keep": keep}
            most = 1.2e11 if kind == "backward" else 4e10
        elif kind == "chain":
            return {"kind": "chain", "dtype": rng.choice(["f32", "f32", "f16"]), "N": 1,
                    "side": 32 * rng.randint(1, 7), "width": 16 * rng.randint(1, 4)}
        else:
            return {"kind": "select", "dtype": rng.choice(["f32", "f16"]), "n": _log(rng, 256, 1634496), "K": K,
                    "keep": keep}
        if _dense_macs(c) <= most and _elements(c) <= 2.1e8:
            return c


# ------------------------------------------------------------------------------------------------------------ inputs

def _library(rng, K):
    return np.sort(rng.permutation(CENTRE_MASKS)[:K])


def _weights(rng, F, C, dtype, clusters=0, keep=1.0):
    """He-initialised; with clusters, filters of one cluster have their large kernels on the same channels."""
    w = rng.standard_normal((F, C, 3, 3), dtype=np.float32) * np.float32(math.sqrt(2.0 / (9.0 * C)))
    if clusters:
        group = rng.permutation(F) * clusters // F
        for g in range(clusters):
            outside = rng.permutation(C)[max(1, round(1.25 * keep * C)):]
            w[np.ix_(np.nonzero(group == g)[0], outside)] *= np.float32(0.05)
    return w.astype(np.float16) if dtype == "f16" else w


def _prune(w, lib, keep):
    w32 = w.astype(np.float32)
    pid = pc.assign_patterns(w32, lib)
    return pid, pc.select_connectivity(w32, lib, pid, keep)


def _torch_type(dtype):
    return torch.float16 if dtype == "f16" else torch.float32


def _normal(gen, shape, dtype, relu=False, scale=1.0):
    t = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float16 if dtype == "f16" else torch.float32)
    if relu:
        t.clamp_min_(0)
    return t.mul_(scale) if scale != 1.0 else t


def _out(c, n, pad=1, ext=3):
    return (n + 2 * pad - ext) // c.get("stride", 1) + 1


def _prepare_conv(c, rng, gen):
    w, lib = _weights(rng, c["F"], c["C"], c["dtype"], c["clusters"], c["keep"]), _library(rng, c["K"])
    pid, mask = _prune(w, lib, c["keep"] if c["C"] > 3 else 1.0)
    if c["clusters"]:      # similar filters side by side: the next layer's channels absorb the order
        order = pc.filter_similarity_order(mask, 128)
        w, pid, mask = w[order], pid[order], mask[order]
    Ho, Wo = _out(c, c["H"], c["pad"]), _out(c, c["W"], c["pad"])
    nhwc = c["layout"] == "nhwc"
    xs, ys = ((c["N"], c["H"], c["W"], c["C"]), (c["N"], Ho, Wo, c["F"])) if nhwc else (
        (c["N"], c["C"], c["H"], c["W"]), (c["N"], c["F"], Ho, Wo))
    return {"packed": pc.pack(w, lib, pid, mask), "x": _normal(gen, xs, c["dtype"], relu=True),
            "y": torch.empty(ys, device="cuda", dtype=_torch_type(c["dtype"])),
            "bias": _normal(gen, (c["F"],), "f32", scale=0.1),
            "flags": (pc.FLAG_RELU if c["relu"] else 0) | (pc.FLAG_NHWC if nhwc else 0)}


def _prepare_conv1x1(c, rng, gen):
    F, C, lib = c["F"], c["C"], _library(rng, 8)
    w = rng.standard_normal((F, C), dtype=np.float32) * np.float32(math.sqrt(2.0 / C))
    groups = -(-C // 9)
    wide = np.zeros((F, groups * 9), np.float32)
    wide[:, :C] = w
    pid, mask = _prune(wide.reshape(F, groups, 3, 3), lib, c["keep"])
    Ho, Wo = _out(c, c["H"], 0, 1), _out(c, c["W"], 0, 1)
    nhwc = c["layout"] == "nhwc"
    xs, ys = ((c["N"], c["H"], c["W"], C), (c["N"], Ho, Wo, F)) if nhwc else ((c["N"], C, c["H"], c["W"]),
                                                                             (c["N"], F, Ho, Wo))
    return {"packed": pc.pack_1x1(w.astype(np.float16 if c["dtype"] == "f16" else np.float32), lib, pid, mask),
            "x": _normal(gen, xs, c["dtype"], relu=True), "bias": _normal(gen, (F,), "f32", scale=0.1),
            "y": torch.empty(ys, device="cuda", dtype=_torch_type(c["dtype"])),
            "flags": pc.FLAG_RELU | (pc.FLAG_NHWC if nhwc else 0)}


def _chain_layers(c):
    """(C, F, side, pool behind, keep) of the chain's layers; a map that has shrunk to one row is pooled no further."""
    out = []
    for (ci, fi, part, pool), keep in zip(VGG16, VGG16_KEEP):
        side = max(1, c["side"] * part // 224)
        out.append((ci * c["width"] or 3, fi * c["width"], side, pool and side > 1, keep))
    return out


def _prepare_chain(c, rng, gen):
    lib, layers, t = _library(rng, 8), [], _torch_type(c["dtype"])
    for C, F, side, pool, keep in _chain_layers(c):
        w = _weights(rng, F, C, c["dtype"])
        pid, mask = _prune(w, lib, keep)
        # (kept weights rescaled so that the activations keep their size through thirteen pruned layers)
        w = (w.astype(np.float32) * math.sqrt(9.0 / (4.0 * keep) * 0.6)).astype(w.dtype)
        layers.append({"packed": pc.pack(w, lib, pid, mask), "bias": _normal(gen, (F,), "f32", scale=0.1),
                       "side": side, "y": torch.empty((c["N"], F, side, side), device="cuda", dtype=t),
                       "pooled": torch.empty((c["N"], F, side // 2, side // 2), device="cuda", dtype=t) if pool else None})
    return {"layers": layers, "x": _normal(gen, (c["N"], 3, c["side"], c["side"]), c["dtype"])}


def _prepare_grad(c, rng, gen):
    w, lib = _weights(rng, c["F"], c["C"], "f16"), _library(rng, c["K"])
    pid, mask = _prune(w, lib, c["keep"])
    packed = pc.pack(w, lib, pid, mask)
    N, C, F, H, W = (c[k] for k in ("N", "C", "F", "H", "W"))
    size = pc.conv3x3_grad_weight_workspace(packed, N, H, W)
    s = {"x": _normal(gen, (N, C, H, W), "f16", relu=True), "dy": _normal(gen, (N, F, H, W), "f16", scale=0.1),
         "dx": torch.empty((N, C, H, W), device="cuda", dtype=torch.float16), "size": size,
         "dw": torch.empty((packed.n_kept, 4), device="cuda", dtype=torch.float32),
         "work": torch.empty(max(1, size), device="cuda", dtype=torch.uint8)}
    if c["kind"] == "backward":
        return dict(s, packed=packed, turned=pc.packed_transpose(packed))
    packed.free()
    return dict(s, w=w, lib=lib, pid=pid, mask=mask, bias=_normal(gen, (F,), "f32", scale=0.1),
                y=torch.empty((N, F, H, W), device="cuda", dtype=torch.float16))


def _prepare_select(c, rng, gen):
    n, K = c["n"], c["K"]
    size = pc.select_connectivity_device_workspace(n)
    return {"z": _normal(gen, (n, K), "f32", scale=0.3).add_(1.0 / K), "mu": _normal(gen, (n, K), "f32", scale=0.1),
            "w": _normal(gen, (n, 9), c["dtype"], scale=0.05), "lib": _library(rng, K),
            "u": torch.empty((n, K), device="cuda"), "mu_out": torch.empty((n, K), device="cuda"),
            "hard": torch.empty(n, device="cuda", dtype=torch.int32),
            "pid": torch.empty(n, device="cuda", dtype=torch.int32),
            "mask": torch.empty(n, device="cuda", dtype=torch.uint8),
            "work": torch.empty(size, device="cuda", dtype=torch.uint8), "size": size}


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    kind = case["kind"]
    make = {"conv": _prepare_conv, "conv1x1": _prepare_conv1x1, "chain": _prepare_chain, "backward": _prepare_grad,
            "train": _prepare_grad, "select": _prepare_select}[kind]
    return dict(make(case, rng, gen), case=case, stream=torch.cuda.current_stream().cuda_stream)


# ------------------------------------------------------------------------------------------------------------ a pass

def run(s):
    c, stream = s["case"], s["stream"]
    kind = c["kind"]
    if kind == "conv":
        pc.conv3x3(s["x"], s["y"], s["packed"], s["bias"], c["N"], c["H"], c["W"], c["stride"], c["pad"], s["flags"],
                   stream)
        return s["y"]
    if kind == "conv1x1":
        pc.conv1x1(s["x"], s["y"], s["packed"], s["bias"], c["N"], c["H"], c["W"], c["stride"], s["flags"], stream)
        return s["y"]
    if kind == "chain":
        x, t = s["x"], pc.F16 if c["dtype"] == "f16" else pc.F32
        for l in s["layers"]:
            pc.conv3x3(x, l["y"], l["packed"], l["bias"], c["N"], l["side"], l["side"], 1, 1, pc.FLAG_RELU, stream)
            x = l["y"]
            if l["pooled"] is not None:
                pc.maxpool2x2(x, l["pooled"], t, c["N"], l["packed"].F, l["side"], l["side"], stream)
                x = l["pooled"]
        return [l["y"] for l in s["layers"]] + [x]
    if kind == "select":
        dtype = pc.F16 if c["dtype"] == "f16" else pc.F32
        pc.admm_proximal(s["z"], s["mu"], 1.5, c["n"], c["K"], s["u"], s["mu_out"], stream)
        pc.admm_binarize(s["z"], c["n"], c["K"], s["hard"], stream)
        pc.assign_patterns_device(s["w"], dtype, c["n"], s["lib"], s["pid"], stream)
        pc.select_connectivity_device(s["w"], dtype, c["n"], s["lib"], s["pid"], c["keep"], s["mask"], s["work"],
                                      s["size"], stream)
        return {k: s[k] for k in ("u", "mu_out", "hard", "pid", "mask")}
    N, H, W = c["N"], c["H"], c["W"]
    if kind == "train":
        packed = pc.pack(s["w"], s["lib"], s["pid"], s["mask"])
        turned = pc.packed_transpose(packed)
        pc.conv3x3(s["x"], s["y"], packed, s["bias"], N, H, W, 1, 1, 0, stream)
    else:
        packed, turned = s["packed"], s["turned"]
    pc.conv3x3_grad_input(s["dy"], s["dx"], turned, N, H, W, stream)
    pc.conv3x3_grad_weight(s["x"], s["dy"], packed, s["dw"], N, H, W, 1, 1, s["work"], s["size"], stream)
    if kind == "train":
        torch.cuda.current_stream().synchronize()      # (the header: no launch may use a handle that is freed)
        packed.free()
        turned.free()
        return {k: s[k] for k in ("y", "dx", "dw")}
    return {k: s[k] for k in ("dx", "dw")}


# ------------------------------------------------------------------------------------------- what a pass cannot avoid

def _layer_work(size, N, C, F, H, W, Ho, Wo, kept, weights_each, taps_read=1.0):
    return (size * (N * C * H * W * taps_read + N * F * Ho * Wo + kept * weights_each) + 4 * F,
            2.0 * N * Ho * Wo * kept * weights_each)


def work(case):
    c, kind = case, case["kind"]
    size = 2 if c.get("dtype", "f16") == "f16" else 4
    if kind == "conv":
        kept = c["F"] * c["C"] * (c["keep"] if c["C"] > 3 else 1.0)
        b, f = _layer_work(size, c["N"], c["C"], c["F"], c["H"], c["W"], _out(c, c["H"], c["pad"]),
                           _out(c, c["W"], c["pad"]), kept, 4)
    elif kind == "conv1x1":
        kept = c["F"] * c["C"] * c["keep"] * 4 / 9
        b, f = _layer_work(size, c["N"], c["C"], c["F"], c["H"], c["W"], _out(c, c["H"], 0, 1), _out(c, c["W"], 0, 1),
                           kept, 1, 1.0 / c["stride"] ** 2)
    elif kind == "chain":
        b = f = 0.0
        for C, F, side, pool, keep in _chain_layers(c):
            lb, lf = _layer_work(size, c["N"], C, F, side, side, side, side, F * C * keep, 4)
            b, f = b + lb + (size * c["N"] * F * side * side * 1.25 if pool else 0), f + lf
    elif kind == "select":
        b = c["n"] * (4 * 4 * c["K"] + 9 * size + 4 + 4 + 1)
        f = c["n"] * (c["K"] * 20.0 + 2 * 9 * c["K"])
    else:
        px, kept = c["N"] * c["H"] * c["W"], c["F"] * c["C"] * c["keep"]
        b = 2.0 * px * (2 * c["C"] + c["F"]) + kept * (8 + 16)
        f = 2 * 2.0 * px * kept * 4
        if kind == "train":
            b, f = b + 2.0 * px * c["F"] + 2.0 * c["F"] * c["C"] * 9, f + 2.0 * px * kept * 4
    return {"bytes": b, "flops": f}


def tolerance(case):
    kind = case["kind"]
    if kind == "select":            # double arithmetic inside, single-precision results; indices and marks are exact
        return {"rel": 1e-6, "differ": 0.0}
    if case.get("dtype", "f16") == "f32":
        return {"rel": 1e-5, "max": 2e-4}          # fp32 sums in another order
    if kind == "chain":             # thirteen roundings to fp16, each of which the next layer reads
        return {"rel": 2e-3, "max": 2e-2}
    return {"rel": 1e-3, "max": 4e-3}              # fp32 sums, one rounding to fp16 (11 bits)
