"""The work that a user of this library has it do, as measurable cases: single masked layers, 8-bit layers, a ConvNeXt
block, the ResNet-50 trunk, and packing the weights of a network stage after an update.

A case is a dict of plain values; ``prepare`` draws its inputs on the GPU and packs its weights, ``run`` is one pass
through the public entry points.  Layer shapes are those of the library's own configurations (``workloads``: ResNet-50 at
224 x 224, ConvNeXt-T stage 1, configs 0..2) and ragged ones between them.
"""
from __future__ import annotations

import math

import torch

import paper_2411_00288_amd as ss

DTYPES = {"f16": ss.SS_F16, "bf16": ss.SS_BF16, "int8": ss.SS_I8, "fp8": ss.SS_F8}
ORDERS = {"crs": ss.SS_K_CRS, "rsc": ss.SS_K_RSC}
ACTS = {"none": ss.SS_ACT_NONE, "relu": ss.SS_ACT_RELU, "gelu": ss.SS_ACT_GELU}


def _conv(name, N, H, W, cin, cout, k, stride=1, pad=None, dtype="bf16", korder="crs", act="relu", residual=False, sparse=True):
    c = {"kind": "conv", "N": N, "H": H, "W": W, "cin": cin, "cout": cout, "k": k, "stride": stride,
         "pad": k // 2 if pad is None else pad, "dtype": dtype, "korder": korder, "act": act, "residual": residual, "sparse": sparse}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: one layer on one small image (config 0); latency and the host path count
        _conv("conv3x3_64_n1", 1, 16, 16, 64, 64, 3, dtype="f16", act="none"),
        # a mid-network 3x3 layer at an ordinary serving batch (config 1, the headline layer), in the flattening of the paper
        _conv("conv3x3_256_n32", 32, 14, 14, 256, 256, 3, dtype="f16"),
        # the same layer at the largest batch the benchmark uses: throughput of the 3x3 contraction
        _conv("conv3x3_256_n500", 500, 14, 14, 256, 256, 3, dtype="f16"),
        # a channel-reducing pointwise layer (config 2): bound by memory
        _conv("conv1x1_1024_256_n64", 64, 14, 14, 1024, 256, 1),
        # the ConvNeXt-T downsample at batch 128: 2x2, stride 2, no padding
        _conv("conv2x2s2_96_192_n128", 128, 56, 56, 96, 192, 2, stride=2, pad=0, act="none"),
        # ragged sizes of a pruned or hand-made network: odd image, channels that fill no tile, closing a residual block
        _conv("conv3x3_ragged_res", 6, 45, 61, 80, 136, 3, dtype="f16", residual=True),
        # 8-bit inference: the headline layer with int8 operands, and at the largest batch with FP8 operands
        _conv("int8_conv3x3_256_n32", 32, 14, 14, 256, 256, 3, dtype="int8"),
        _conv("fp8_conv3x3_256_n500", 500, 14, 14, 256, 256, 3, dtype="fp8"),
        # a ConvNeXt-T stage-1 block: dense 7x7 depthwise, then the masked inverted bottleneck with its skip connection
        {"name": "convnext_block_n128", "kind": "block", "N": 128, "H": 56, "W": 56, "C": 96, "k": 7, "dtype": "bf16", "sparse": True},
        # ResNet-50 trunk, one image: latency of a chain of small launches
        {"name": "trunk_n1", "kind": "trunk", "batch": 1, "image": 224, "sparse": True},
        # ResNet-50 trunk at the benchmark's batch: throughput
        {"name": "trunk_n64", "kind": "trunk", "batch": 64, "image": 224, "sparse": True},
        # re-packing the masked layers of ResNet-50's last stage after a weight update
        {"name": "repack_stage4", "kind": "pack", "width": 512, "blocks": 3, "dtype": "bf16", "mode": "update"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["conv", "conv", "conv", "conv", "conv8", "conv8", "block", "pack", "trunk"])
    if kind == "trunk":
        image = rng.randint(64, 256)
        return {"kind": "trunk", "batch": _log(rng, 1, max(1, min(64, 64 * 224 * 224 // (image * image)))), "image": image,
                "sparse": rng.random() < 0.75}
    if kind == "pack":
        return {"kind": "pack", "width": 8 * _log(rng, 8, 64), "blocks": rng.randint(1, 3), "dtype": rng.choice(["f16", "bf16"]),
                "mode": rng.choice(["update", "compress", "dense"])}
    if kind == "block":
        H, W = _log(rng, 7, 64), _log(rng, 7, 64)
        return {"kind": "block", "N": min(_log(rng, 1, 128), max(1, 128 * 56 * 56 // (H * W))), "H": H, "W": W,
                "C": rng.choice([32, 64, 96, 128]), "k": rng.choice([3, 5, 7, 7, 7]), "dtype": rng.choice(["f16", "bf16"]),
                "sparse": rng.random() < 0.75}
    k = rng.choice([1, 1, 2, 3, 3, 3])
    stride = 2 if k == 2 else rng.choice([1, 1, 1, 2])
    H, W = _log(rng, 7, 64), _log(rng, 7, 64)
    if kind == "conv8":
        # 8-bit layers: multiples of 64 channels (16 in the channels-last flattening)
        korder = rng.choice(["crs", "rsc"])
        unit = 64 if korder == "crs" and k > 1 else 16
        cin, cout, dtype = unit * _log(rng, 1, 512 // unit), 4 * _log(rng, 16, 128), rng.choice(["int8", "fp8"])
    elif rng.random() < 0.5:
        # channel counts of networks
        korder, dtype = rng.choice(["crs", "crs", "rsc"]), rng.choice(["f16", "bf16"])
        cin, cout = 32 * _log(rng, 2, 32 if k == 1 else 16), 32 * _log(rng, 2, 32)
    else:
        # ragged channel counts
        korder, dtype = rng.choice(["crs", "crs", "rsc"]), rng.choice(["f16", "bf16"])
        cin, cout = 4 * _log(rng, 8, 128 if k == 1 else 64), 2 * _log(rng, 20, 256)
    c = _conv(None, 1, H, W, cin, cout, k, stride=stride, pad=0 if k == 2 else k // 2, dtype=dtype, korder=korder,
              act=rng.choice(["none", "relu", "relu", "gelu"]), residual=kind == "conv" and rng.random() < 0.3,
              sparse=rng.random() < 0.8)
    one = work(c)
    most = max(1, min(500, int(6e10 / one["flops"]), int(2.4e8 / one["bytes"])))
    c["N"] = _log(rng, 1, most)
    return c


def _out(c):
    return (c["H"] + 2 * c["pad"] - c["k"]) // c["stride"] + 1, (c["W"] + 2 * c["pad"] - c["k"]) // c["stride"] + 1


def _weight_bytes(cout, K, sparse, esize):
    return cout * K * esize * 0.5 + cout * K / 8 if sparse else cout * K * esize


def _stage_layers(c):
    """(cout, cin, k) of the masked layers of a bottleneck stage."""
    w = c["width"]
    return [s for b in range(c["blocks"]) for s in ((w, 2 * w if b == 0 else 4 * w, 1), (w, w, 3), (4 * w, w, 1))]


def work(c):
    """Activations and (packed) weights once each; the products of the kept weights only where a mask drops half."""
    if c["kind"] == "conv":
        Ho, Wo = _out(c)
        P, K, es = c["N"] * Ho * Wo, c["cin"] * c["k"] ** 2, 1 if c["dtype"] in ("int8", "fp8") else 2
        b = c["N"] * c["H"] * c["W"] * c["cin"] * es + P * c["cout"] * 2 * (2 if c["residual"] else 1)
        return {"bytes": b + _weight_bytes(c["cout"], K, c["sparse"], es) + 4 * c["cout"],
                "flops": (1 if c["sparse"] else 2) * P * c["cout"] * K}
    if c["kind"] == "block":
        P, C = c["N"] * c["H"] * c["W"], c["C"]
        return {"bytes": 4 * P * C + c["k"] ** 2 * C * 2 + 2 * _weight_bytes(4 * C, C, c["sparse"], 2) + 4 * 6 * C,
                "flops": 2 * P * C * c["k"] ** 2 + (1 if c["sparse"] else 2) * 2 * P * 4 * C * C}
    if c["kind"] == "pack":
        n = sum(o * i * k * k for o, i, k in _stage_layers(c))
        return {"bytes": n * {"update": 2 + 2 + 1 + 2 + 1.125, "compress": 2 + 1 + 1.125, "dense": 2 + 1 + 2}[c["mode"]], "flops": n}
    from paper_2411_00288_amd import resnet50
    ops, shapes = resnet50.build_ops(c["batch"], c["image"])
    flops = bytes_ = 0.0
    for op in ops:
        if op.kind == "conv":
            L = op.layer
            masked = c["sparse"] and L.mask != "none"
            flops += L.dense_equiv_flop * (0.5 if masked else 1.0)
            bytes_ += _weight_bytes(L.cout, L.K, masked, 2) + 4 * L.cout
    return {"bytes": bytes_ + 2 * math.prod(shapes[0]) + 2 * math.prod(shapes[ops[-1].dst]), "flops": flops}


def tolerance(c):
    if c["kind"] == "pack":
        return "exact"                                   # bits are moved; the update's rounding is defined
    if c["kind"] == "trunk":
        return {"rel": 2e-2}                             # bf16 roundings that fall the other way, carried through 50 layers
    if c["kind"] == "block":
        return {"rel": 2e-3 if c["dtype"] == "f16" else 8e-3}
    return {"rel": 4e-3 if c["dtype"] == "bf16" else 1e-3}


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _randn(g, *shape):
    return torch.randn(shape, generator=g, device="cuda")


def _top2(mag):
    """2:4 mask of the two largest magnitudes of every four consecutive entries of a row."""
    m = mag.reshape(-1, 4)
    out = torch.zeros(m.shape, dtype=torch.uint8, device=m.device)
    out.scatter_(1, torch.topk(m, 2, dim=1).indices, 1)
    return out.reshape(mag.shape)


def _weights(g, cout, cin, k, dtype, korder, sparse, scale=1.0):
    """A packed 16-bit weight operand (descriptor, buffer, bias), He-normal with a top-2 mask."""
    K = cin * k * k
    desc = ss.make_desc(cout, cin, k, k, DTYPES[dtype], ORDERS[korder])
    W = (_randn(g, cout, K) * (scale * math.sqrt(2.0 / K))).to(ss.torch_dtype(DTYPES[dtype]))
    M = _top2(W.float().abs())
    buf = ss.ss_mask_compress(desc, W, M) if sparse else ss.ss_dense_pack(desc, W, M)
    return desc, buf, _randn(g, cout) * 0.1


def prepare(c, seed):
    g = _gen(seed)
    if c["kind"] == "trunk":
        from paper_2411_00288_amd import resnet50
        t = resnet50.Trunk(c["batch"], c["image"], sparse=c["sparse"], seed=int(seed))
        t.input.copy_(_randn(g, *t.input.shape))
        t.input[..., 3:] = 0                              # the image's padding channel
        return {"kind": "trunk", "trunk": t}
    if c["kind"] == "pack":
        tdt, layers = ss.torch_dtype(DTYPES[c["dtype"]]), []
        for cout, cin, k in _stage_layers(c):
            K = cin * k * k
            desc = ss.make_desc(cout, cin, k, k, DTYPES[c["dtype"]], ss.SS_K_CRS)
            W = (_randn(g, cout, K) * math.sqrt(2.0 / K)).to(tdt)
            U = (_randn(g, cout, K) * (1e-3 * math.sqrt(2.0 / K))).to(tdt)
            size = ss.ss_dense_bytes(desc) if c["mode"] == "dense" else ss.ss_packed_bytes(desc)
            layers.append((desc, W, U, _top2(W.float().abs()), torch.empty(size, dtype=torch.uint8, device="cuda")))
        return {"kind": "pack", "mode": c["mode"], "layers": layers}
    if c["kind"] == "block":
        C, tdt = c["C"], ss.torch_dtype(DTYPES[c["dtype"]])
        x = _randn(g, c["N"], c["H"], c["W"], C).to(tdt)
        dw = (_randn(g, c["k"], c["k"], C) / c["k"]).to(tdt)
        return {"kind": "block", "x": x, "dw": dw, "dwb": _randn(g, C) * 0.1, "pad": c["k"] // 2, "sparse": c["sparse"],
                "up": _weights(g, 4 * C, C, 1, c["dtype"], "crs", c["sparse"]),
                "down": _weights(g, C, 4 * C, 1, c["dtype"], "crs", c["sparse"])}
    s = {"kind": "conv", "stride": (c["stride"],) * 2, "pad": (c["pad"],) * 2, "act": ACTS[c["act"]], "residual": None, "scale": None}
    shape = (c["N"], c["H"], c["W"], c["cin"])
    x = torch.relu(_randn(g, *shape))
    if c["dtype"] in ("int8", "fp8"):
        # symmetric quantisation per output channel, activations with one step (four standard deviations)
        K, top, fp8 = c["cin"] * c["k"] ** 2, (448.0 if c["dtype"] == "fp8" else 127.0), c["dtype"] == "fp8"
        desc = ss.make_desc(c["cout"], c["cin"], c["k"], c["k"], DTYPES[c["dtype"]], ORDERS[c["korder"]])
        W = _randn(g, c["cout"], K) * math.sqrt(2.0 / K)
        step = W.abs().amax(dim=1, keepdim=True) / top

        def cast(v):
            v = v.clamp(-top, top)
            return v.to(torch.float8_e4m3fn).view(torch.uint8) if fp8 else v.round().to(torch.int8)
        Wq = cast(W / step)
        M = _top2(W.abs())
        s.update(q8=True, desc=desc, x=cast(x * (top / 4.0)), scale=(step * (4.0 / top)).reshape(-1).contiguous(), bias=_randn(g, c["cout"]) * 0.1,
                 w=ss.ss_mask_compress(desc, Wq, M) if c["sparse"] else ss.ss_dense_pack(desc, Wq, M))
        s["call"] = ss.ss_conv2d_q8_fwd if c["sparse"] else ss.ss_conv2d_q8_dense_fwd
        return s
    s.update(q8=False, x=x.to(ss.torch_dtype(DTYPES[c["dtype"]])))
    s["desc"], s["w"], s["bias"] = _weights(g, c["cout"], c["cin"], c["k"], c["dtype"], c["korder"], c["sparse"])
    if c["residual"]:
        s["residual"] = _randn(g, c["N"], *_out(c), c["cout"]).to(s["x"].dtype)
        s["call"] = ss.ss_conv2d_res_fwd if c["sparse"] else ss.ss_conv2d_dense_res_fwd
    else:
        s["call"] = ss.ss_conv2d_fwd if c["sparse"] else ss.ss_conv2d_dense_fwd
    return s


def run(s):
    if s["kind"] == "trunk":
        return s["trunk"].forward()
    if s["kind"] == "pack":
        out = []
        for desc, W, U, M, buf in s["layers"]:
            if s["mode"] == "update":
                out += [ss.ss_mask_update_compress(desc, W, U, M, packed=buf), W]
            elif s["mode"] == "compress":
                out.append(ss.ss_mask_compress(desc, W, M, packed=buf))
            else:
                out.append(ss.ss_dense_pack(desc, W, M, dense=buf))
        return out
    if s["kind"] == "block":
        t = ss.ss_dwconv2d_fwd(s["x"], s["dw"], s["dwb"], (s["pad"],) * 2)
        (d1, w1, b1), (d2, w2, b2) = s["up"], s["down"]
        fused = ss.ss_conv2d_pw_fused_fwd if s["sparse"] else ss.ss_conv2d_pw_fused_dense_fwd
        return fused(d1, t, w1, b1, (1, 1), (0, 0), ss.SS_ACT_GELU, d2, w2, b2, residual=s["x"])
    if s["q8"]:
        return s["call"](s["desc"], s["x"], s["w"], s["scale"], s["bias"], s["stride"], s["pad"], s["act"])
    if s["residual"] is not None:
        return s["call"](s["desc"], s["x"], s["w"], s["bias"], s["residual"], s["stride"], s["pad"], s["act"])
    return s["call"](s["desc"], s["x"], s["w"], s["bias"], s["stride"], s["pad"], s["act"])
