"""The work that users of this library have it do, as measurable cases.

A case is one call, or one block of calls, through the package's public entry
points: pruned convolutions forward (fp32 and bf16, NCHW and NHWC, plain and
with a folded batch norm and activation), the fully connected layer, the two
gradients of fine-tuning with the pattern fixed, and mask building on the GPU.
Shapes are those of the networks in ``workloads`` (ResNet-50, MobileNet-V2,
their pruned layers) and generic neighbours of them.

A case's ``op`` says which call it is:

``conv``   one ``PackedLayer.forward``
``block``  the four convolutions of a bottleneck block with a downsample path
``pair``   the two pointwise convolutions of an inverted-residual block
``fc``     one ``fc_fwd``
``bwd``    ``conv2d_bwd_data`` and ``conv2d_bwd_weight`` of one layer
``mask``   one ``build_mask_dev``
"""
import math

import torch

import paper_2105_14713_amd as onexn

_DT = {"f32": torch.float32, "bf16": torch.bfloat16}


def _conv(name, **kw):
    c = {"op": "conv", "dtype": "f32", "layout": "nchw", "k": 1, "stride": 1, "N": 32, "p": 0.5,
         "act": "none", "batch": 1, "cin": 64, "cout": 64, "H": 56, "W": 56}
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest call in use: one 3x3 layer of a batch-1 request at the
        # paper's N = 4; launches and host path count.
        _conv("conv3x3_b1_n4", k=3, N=4),
        # A 3x3 layer of the ResNet-50 inference pass with its batch norm and
        # ReLU folded in: the bulk of that network's multiply-adds.
        _conv("conv3x3_b64_n32", k=3, batch=64, cin=128, cout=128, H=28, W=28, act="relu"),
        # A widening 1x1 layer with rearranged output channels at N = 16.
        _conv("conv1x1_b32_n16", N=16, batch=32, cin=256, cout=512, H=28, W=28),
        # The largest call: a wide bf16 1x1 layer at the last stage's channel
        # counts and a large batch.
        _conv("conv1x1_bf16_b256_n32", dtype="bf16", p=0.7, batch=256, cin=2048, cout=2048, H=14, W=14),
        # Half-precision inference of the same network's 3x3 layers.
        _conv("conv3x3_bf16_b64_n32", dtype="bf16", k=3, batch=64, cin=256, cout=256, H=14, W=14,
              act="relu"),
        # channels_last inference: an expand layer with ReLU6.
        _conv("conv1x1_nhwc_b128_n32", layout="nhwc", batch=128, cin=96, cout=576, H=14, W=14,
              act="relu6"),
        # A whole bottleneck block with stride and downsample path, at an odd
        # image size (detection and segmentation crops are ragged).
        {"name": "block_b16_odd_n32", "op": "block", "dtype": "f32", "N": 32, "p": 0.5, "batch": 16,
         "cin": 256, "width": 128, "H": 57, "W": 51, "stride": 2},
        # The pointwise convolutions of a MobileNet-V2 block at N = 4, the
        # block length the paper deploys.
        {"name": "pair_b128_n4", "op": "pair", "dtype": "f32", "N": 4, "p": 0.5, "batch": 128,
         "cin": 32, "hidden": 192, "H": 28, "W": 28},
        # The classifier as a fully connected layer, one row per sample; 1000
        # outputs leave the last col-group ragged.
        {"name": "fc_rows_b256_n32", "op": "fc", "dtype": "f32", "layout": "rows", "N": 32, "p": 0.5,
         "batch": 256, "cin": 2048, "cout": 1000},
        # Fine-tuning: both gradients of a 3x3 layer.
        {"name": "bwd3x3_b64_n32", "op": "bwd", "dtype": "f32", "k": 3, "stride": 1, "N": 32, "p": 0.5,
         "batch": 64, "cin": 128, "cout": 128, "H": 28, "W": 28},
        # Fine-tuning in bf16: both gradients of a widening 1x1 layer.
        {"name": "bwd1x1_bf16_b64_n32", "op": "bwd", "dtype": "bf16", "k": 1, "stride": 1, "N": 32,
         "p": 0.5, "batch": 64, "cin": 256, "cout": 1024, "H": 14, "W": 14},
        # Mask building on the device with filter rearrangement, as when the
        # pattern is chosen anew during pruning.
        {"name": "mask_2048x2048_n32", "op": "mask", "dtype": "f32", "k": 1, "N": 32, "p": 0.7,
         "cin": 2048, "cout": 2048, "rearrange": True},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _chan(rng, lo, hi):
    """A channel count: mostly multiples of 8, as networks have them, some odd."""
    c = _log(rng, lo, hi)
    return c if rng.random() < 0.25 else max(8, c // 8 * 8)


def _fit(case, flops, nbytes):
    """Shrinks the batch, then the image, until one pass costs no more than that."""
    while True:
        w = work(case)
        if w["flops"] <= flops and w["bytes"] <= nbytes:
            return case
        if case["batch"] > 1:
            case["batch"] = max(1, case["batch"] * 3 // 4)
        else:
            case["H"], case["W"] = case["H"] * 3 // 4, case["W"] * 3 // 4


def draw(rng):
    """One more case: the same calls over the whole range of sizes they are made with."""
    op = rng.choice(["conv", "conv", "conv", "block", "pair", "fc", "bwd", "bwd", "mask"])
    p = rng.choice([0.3, 0.5, 0.7])
    side = _log(rng, 7, 112)
    H, W = side, (side if rng.random() < 0.6 else max(7, min(112, side + rng.randint(-9, 9))))
    if op == "conv":
        kind = rng.choice(["f32", "f32", "bf16", "nhwc"])
        batch = _log(rng, 1, 256)
        if kind == "f32":
            c = _conv(None, k=rng.choice([1, 3]), stride=rng.choice([1, 1, 2]), N=rng.choice([4, 8, 16, 32]),
                      p=p, act=rng.choice(["none", "relu", "relu6"]), batch=batch,
                      cin=_chan(rng, 16, 1024), cout=_chan(rng, 16, 1024), H=H, W=W)
        elif kind == "bf16":
            c = _conv(None, dtype="bf16", k=rng.choice([1, 3]), stride=rng.choice([1, 1, 2]),
                      N=rng.choice([16, 32]), p=p, act=rng.choice(["none", "relu"]), batch=batch,
                      cin=_chan(rng, 32, 2048), cout=_chan(rng, 32, 2048), H=H, W=W)
        else:
            c = _conv(None, layout="nhwc", N=rng.choice([16, 32]), p=p, act=rng.choice(["none", "relu6"]),
                      batch=batch, cin=_chan(rng, 16, 960), cout=_chan(rng, 16, 960), H=H, W=W)
        return _fit(c, 1.5e10 if c["dtype"] == "bf16" else 7e9, 4e8)
    if op == "block":
        c = {"op": "block", "dtype": "f32", "N": rng.choice([16, 32]), "p": p, "batch": _log(rng, 1, 64),
             "cin": _chan(rng, 64, 1024), "width": _chan(rng, 32, 256), "H": H, "W": W,
             "stride": rng.choice([1, 2])}
        return _fit(c, 1.2e10, 4e8)
    if op == "pair":
        cin = _chan(rng, 16, 160)
        c = {"op": "pair", "dtype": "f32", "N": rng.choice([4, 8, 16, 32]), "p": p,
             "batch": _log(rng, 1, 128), "cin": cin, "hidden": 6 * cin, "H": H, "W": W}
        return _fit(c, 7e9, 4e8)
    if op == "fc":
        return {"op": "fc", "dtype": "f32", "layout": rng.choice(["rows", "rows", "cols"]),
                "N": rng.choice([4, 16, 32]), "p": p, "batch": _log(rng, 1, 512),
                "cin": _chan(rng, 256, 4096), "cout": _chan(rng, 100, 4096)}
    if op == "bwd":
        c = {"op": "bwd", "dtype": rng.choice(["f32", "f32", "bf16"]), "k": rng.choice([1, 3]),
             "stride": rng.choice([1, 1, 2]), "N": rng.choice([16, 32]), "p": p, "batch": _log(rng, 4, 128),
             "cin": _chan(rng, 32, 1024), "cout": _chan(rng, 32, 1024), "H": H, "W": W}
        return _fit(c, 1.5e10 if c["dtype"] == "f32" else 8e9, 4e8)
    return {"op": "mask", "dtype": rng.choice(["f32", "bf16"]), "k": rng.choice([1, 3]),
            "N": rng.choice([4, 8, 16, 32]), "p": p, "cin": _chan(rng, 64, 1024),
            "cout": _chan(rng, 64, 1024), "rearrange": rng.random() < 0.5}


def _out(n, k, stride, pad):
    return (n + 2 * pad - k) // stride + 1


def _convs(case):
    """[(cin, cout, k, stride, H, W)] of a case's convolutions, in call order."""
    op = case["op"]
    if op in ("conv", "bwd"):
        return [(case["cin"], case["cout"], case["k"], case["stride"], case["H"], case["W"])]
    if op == "fc":
        return [(case["cin"], case["cout"], 1, 1, 1, 1)]
    H, W = case["H"], case["W"]
    if op == "pair":
        return [(case["cin"], case["hidden"], 1, 1, H, W), (case["hidden"], case["cin"], 1, 1, H, W)]
    s, w = case["stride"], case["width"]
    H2, W2 = _out(H, 3, s, 1), _out(W, 3, s, 1)
    return [(case["cin"], w, 1, 1, H, W), (w, w, 3, s, H, W), (w, 4 * w, 1, 1, H2, W2),
            (case["cin"], 4 * w, 1, s, H, W)]


def _gen(seed, device):
    return torch.Generator(device).manual_seed(seed)


def _weight(case, i, conv, seed):
    """He-normal weights of convolution i, on the host (where layers are packed)."""
    cin, cout, k = conv[:3]
    w = torch.randn((cout, cin, k, k), generator=_gen(1000 * seed + i, "cpu")) * math.sqrt(2.0 / (cin * k * k))
    return w.to(_DT[case["dtype"]])


def _affine(case, i, n, seed):
    """A folded batch norm's scale and bias (rearranged channel order)."""
    g = _gen(1000 * seed + 500 + i, "cuda")
    return (torch.rand(n, generator=g, device="cuda") + 0.5,
            torch.randn(n, generator=g, device="cuda") * 0.25)


def _activation(shape, gen, dtype, act):
    x = torch.randn(shape, generator=gen, device="cuda")
    if act == "relu6":
        x.clamp_(0.0, 6.0)
    elif act == "relu":
        x.clamp_min_(0.0)
    return x.to(_DT[dtype])


def _inputs(case, seed):
    """The case's input tensors, in the order that the calls take them."""
    g = _gen(1000 * seed + 900, "cuda")
    op, dt = case["op"], case["dtype"]
    if op == "mask":
        return []
    if op == "fc":
        b, m = case["batch"], case["cin"]
        return [_activation((b, m) if case["layout"] == "rows" else (m, b), g, dt, "relu")]
    convs = _convs(case)
    cin, cout, k, s, H, W = convs[0]
    b = case["batch"]
    shape = (b, H, W, cin) if case.get("layout") == "nhwc" else (b, cin, H, W)
    xs = [_activation(shape, g, dt, "relu6" if op == "pair" or case.get("act") == "relu6" else "relu")]
    if op == "pair":
        xs.append(_activation((b, case["hidden"], H, W), g, dt, "relu6"))
    elif op == "bwd":
        pad = k // 2
        xs.append(_activation((b, cout, _out(H, k, s, pad), _out(W, k, s, pad)), g, dt, "none"))
    return xs


def _rearranged(case):
    return case["op"] == "conv" and case["N"] == 16


def prepare(case, seed):
    """Packed layers, folded batch-norm parameters and inputs, on the GPU."""
    st = {"case": case, "xs": _inputs(case, seed)}
    if case["op"] == "mask":
        st["w"] = _weight(case, 0, (case["cin"], case["cout"], case["k"]), seed).cuda()
        st["ws"] = torch.empty(max(8, onexn.mask_workspace_bytes(case["cout"], case["cin"], case["N"])),
                               dtype=torch.uint8, device="cuda")
        return st
    st["layers"] = [onexn.prepare_layer(_weight(case, i, c, seed), case["N"], case["p"], _rearranged(case))
                    for i, c in enumerate(_convs(case))]
    st["affine"] = [_affine(case, i, c[1], seed) for i, c in enumerate(_convs(case))]
    return st


def run(st):
    case, xs = st["case"], st["xs"]
    op = case["op"]
    if op == "mask":
        perm, mask, t = onexn.build_mask_dev(st["w"], case["N"], case["p"], case["rearrange"], st["ws"])
        return {"perm": perm, "mask": mask, "t": t}
    layers, affine = st["layers"], st["affine"]
    if op == "conv":
        k, act = case["k"], case["act"]
        if act == "none":
            return layers[0].forward(xs[0], case["stride"], k // 2, case["layout"])
        return layers[0].forward(xs[0], case["stride"], k // 2, case["layout"], scale=affine[0][0],
                                 bias=affine[0][1], act=act)
    if op == "pair":     # the depthwise convolution between the two is not pruned, and not here
        return [layers[0].forward(xs[0], scale=affine[0][0], bias=affine[0][1], act="relu6"),
                layers[1].forward(xs[1], scale=affine[1][0], bias=affine[1][1])]
    if op == "block":
        s = case["stride"]
        h = layers[0].forward(xs[0], scale=affine[0][0], bias=affine[0][1], act="relu")
        h = layers[1].forward(h, s, 1, scale=affine[1][0], bias=affine[1][1], act="relu")
        main = layers[2].forward(h, scale=affine[2][0], bias=affine[2][1])
        return [main, layers[3].forward(xs[0], s, scale=affine[3][0], bias=affine[3][1])]
    L = layers[0]
    if op == "fc":
        return onexn.fc_fwd(L.P, L.I, L.D, L.n, xs[0], case["layout"], bias=affine[0][1])
    s, pad = case["stride"], case["k"] // 2
    return {"dx": onexn.conv2d_bwd_data(L.P, L.I, L.D, L.n, L.m, xs[1], (case["H"], case["W"]), s, pad),
            "dD": onexn.conv2d_bwd_weight(L.P, L.I, L.n, L.N, (L.kh, L.kw), xs[0], xs[1], s, pad)}


def _kept(case, cin, cout):
    K = cin * -(-cout // case["N"])
    return K - min(K, max(0, int(math.floor(case["p"] * K + 0.5))))


def work(case):
    """Bytes: every input, packed array and output once.  Flops: the kept blocks'
    multiply-adds (the mask: one add per weight for each of its two sums)."""
    es = 4 if case["dtype"] == "f32" else 2
    if case["op"] == "mask":
        nw = case["cin"] * case["cout"] * case["k"] ** 2
        groups = -(-case["cout"] // case["N"])
        return {"bytes": nw * es + 4 * case["cout"] + case["cin"] * groups, "flops": 2 * nw}
    nbytes = flops = 0
    convs, op = _convs(case), case["op"]
    for i, (cin, cout, k, s, H, W) in enumerate(convs):
        pad = k // 2
        px_in, px = case["batch"] * H * W, case["batch"] * _out(H, k, s, pad) * _out(W, k, s, pad)
        t = _kept(case, cin, cout)
        if s > 1 and k == 1:
            px_in = px                                   # the rest of the input is never needed
        wvals = t * case["N"] * k * k
        nbytes += wvals * es + 4 * (t - (-cout // case["N"]) + 1)
        if op == "bwd":
            px_dx = case["batch"] * H * W
            nbytes += (px_in * cin + px * cout + px_dx * cin) * es + 4 * wvals
            flops += 4 * px * wvals
        else:
            shared = op == "block" and i == 3            # the downsample path reads the block's input again
            nbytes += ((0 if shared else px_in * cin) + px * cout) * es
            flops += 2 * px * wvals
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["op"] == "mask":
        return "exact"
    if case["dtype"] == "bf16":
        return {"rel": 7e-3}        # one rounding to 8 bits of an fp32 sum: 1.7e-3 measured
    # fp32 sums of up to 9216 products: 1e-7 (short ones) to 4.7e-7 (a 3x3
    # layer's gradients) measured, a chain of layers a little more.
    return {"rel": 3e-6 if case["op"] == "block" else 2e-6}


# --- the same in 64 bits, in plain torch ---------------------------------------------------------


def _masked(case, w):
    """(perm, mask [cin][G], masked rearranged weight in float64) of a host weight."""
    n, m = w.shape[:2]
    N, G = case["N"], -(-w.shape[0] // case["N"])
    w = w.double()
    rearrange = case["rearrange"] if case["op"] == "mask" else _rearranged(case)
    perm = torch.arange(n)
    if rearrange:
        perm = torch.sort(w.abs().sum((1, 2, 3)), descending=True, stable=True).indices
    w = w[perm]
    rows = w.abs().sum((2, 3))                                    # [n][m]
    rows = torch.cat([rows, rows.new_zeros(G * N - n, m)]).view(G, N, m).sum(1)
    order = torch.sort(rows.t().reshape(-1), descending=True, stable=True).indices
    mask = torch.zeros(m * G, dtype=torch.uint8)
    mask[order[: _kept(case, m, n)]] = 1
    mask = mask.view(m, G)
    keep = mask.t().repeat_interleave(N, 0)[:n]                   # [n][m]
    return perm, mask, (w * keep[:, :, None, None]).cuda()


def _patch(x, q, r, s, Ho, Wo):
    return x[:, :, q:q + (Ho - 1) * s + 1:s, r:r + (Wo - 1) * s + 1:s]


def _conv64(x, w, s, scale=None, bias=None, act="none"):
    """conv2d in float64: one matrix product per tap."""
    n, m, k = w.shape[0], w.shape[1], w.shape[2]
    pad = k // 2
    B, H, W = x.shape[0], x.shape[2], x.shape[3]
    Ho, Wo = _out(H, k, s, pad), _out(W, k, s, pad)
    xp = torch.nn.functional.pad(x, (pad, pad, pad, pad))
    y = torch.zeros(n, B * Ho * Wo, dtype=torch.float64, device="cuda")
    for q in range(k):
        for r in range(k):
            cols = _patch(xp, q, r, s, Ho, Wo).permute(1, 0, 2, 3).reshape(m, -1)
            y.addmm_(w[:, :, q, r].contiguous(), cols)
    if scale is not None:
        y.mul_(scale.double()[:, None])
    if bias is not None:
        y.add_(bias.double()[:, None])
    if act != "none":
        y.clamp_(0.0, 6.0 if act == "relu6" else math.inf)
    return y.view(n, B, Ho, Wo).permute(1, 0, 2, 3).contiguous()


def exact(case, seed):
    op = case["op"]
    if op == "mask":
        return None                                               # whole numbers
    convs = _convs(case)
    ws = [_masked(case, _weight(case, i, c, seed))[2] for i, c in enumerate(convs)]
    af = [_affine(case, i, c[1], seed) for i, c in enumerate(convs)]
    xs = [x.double() for x in _inputs(case, seed)]
    if op == "conv":
        x = xs[0].permute(0, 3, 1, 2) if case["layout"] == "nhwc" else xs[0]
        y = _conv64(x, ws[0], case["stride"], *(() if case["act"] == "none" else (*af[0], case["act"])))
        return y.permute(0, 2, 3, 1).contiguous() if case["layout"] == "nhwc" else y
    if op == "pair":
        return [_conv64(xs[0], ws[0], 1, *af[0], "relu6"), _conv64(xs[1], ws[1], 1, *af[1])]
    if op == "block":
        h = _conv64(xs[0], ws[0], 1, *af[0], "relu")
        h = _conv64(h, ws[1], case["stride"], *af[1], "relu")
        return [_conv64(h, ws[2], 1, *af[2]), _conv64(xs[0], ws[3], case["stride"], *af[3])]
    if op == "fc":
        w = ws[0][:, :, 0, 0]
        if case["layout"] == "rows":
            return xs[0] @ w.t().contiguous() + af[0][1].double()
        return w @ xs[0] + af[0][1].double()[:, None]
    # the gradients: dX one matrix product per tap, dD gathered from the dense gradient at the kept blocks
    cin, cout, k, s, H, W = convs[0]
    pad, N, (x, dy) = k // 2, case["N"], xs
    B, Ho, Wo = case["batch"], dy.shape[2], dy.shape[3]
    mask = _masked(case, _weight(case, 0, convs[0], seed))[1]
    G = mask.shape[1]
    xp = torch.nn.functional.pad(x, (pad, pad, pad, pad))
    dxp = torch.zeros_like(xp)
    dyc = dy.permute(1, 0, 2, 3).reshape(cout, -1)
    dw = torch.zeros(G * N, cin, k, k, dtype=torch.float64, device="cuda")
    for q in range(k):
        for r in range(k):
            part = ws[0][:, :, q, r].t().contiguous() @ dyc
            _patch(dxp, q, r, s, Ho, Wo).add_(part.view(cin, B, Ho, Wo).permute(1, 0, 2, 3))
            cols = _patch(xp, q, r, s, Ho, Wo).permute(0, 2, 3, 1).reshape(-1, cin)
            dw[:cout, :, q, r] = dyc @ cols
    kept = mask.t().nonzero().cuda()                              # (g, c), channels ascending in a group
    dD = dw.view(G, N, cin, k, k)[kept[:, 0], :, kept[:, 1]]
    return {"dx": dxp[:, :, pad:pad + H, pad:pad + W].contiguous(), "dD": dD.contiguous()}
