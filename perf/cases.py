"""The calls a training program makes to this library, as measured cases.

One worker's iteration consists of three kinds of work, and each is here at its smallest, at an ordinary and at its
largest size: the statistic of every layer (`vgc.sqgrad*`), the pass over the parameters with the packing of the message
(`vgc.accumulate_select*`, `vgc.pack*`), and the decoding of all workers' messages (`vgc.unpack*`).  The parameter sets are
the ones of `paper_1802_06058_amd.workloads`: a 784-1000-1000-10 perceptron, ResNet-50, VGG-16, a flat 10^9-parameter
stream.  Gradients are synthetic: normal per-sample gradients whose scale differs per layer and per parameter.
"""
import math

import torch
import torch.nn.functional as F

from paper_1802_06058_amd import vgc
from paper_1802_06058_amd import workloads as W

CHUNK = 1 << 26      # elements generated at a time: bounds the temporaries of the 10^9-parameter cases
ZETA = 0.999


# ---------------------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------------------
def listed():
    return [
        # smallest: three fully-connected layers of a perceptron, batch 128, one statistic call per layer
        dict(name="mlp_statistic_f32", kind="stat_fc", dims="784-1000-1000-10", B=128, dtype="f32", g=False),
        # smallest whole exchange: 1.8 M parameters; select, pack, then decode of 8 workers' messages with the SGD step
        dict(name="mlp_exchange", kind="exchange", model="mlp", alpha=2.0, p=8, rho=0.17),
        # the largest fully-connected layer in use, g and s in one call (no framework gradient at hand)
        dict(name="fc6_statistic_bf16", kind="stat_fc", dims="25088-4096", B=64, dtype="bf16", g=True),
        # the same layer with the statistic formed inside the select pass, then the message
        dict(name="fc6_fused_bf16", kind="fused_fc", J=25088, C=4096, B=64, dtype="bf16", alpha=1.0),
        # s of all convolutions of a network in one call: 16-bit activations, batch 64
        dict(name="vgg16_statistic_bf16", kind="stat_net", net="vgg16", B=64, dtype="bf16"),
        # the same in 32 bits on many small layers, batch 32 (1x1, 3x3, strided, 7x7 first layer)
        dict(name="resnet50_statistic_f32", kind="stat_net", net="resnet50", B=32, dtype="f32"),
        # an ordinary model of 161 ragged groups through the hybrid algorithm and the packer
        dict(name="resnet50_hybrid_pack", kind="select_pack", model="resnet50", alpha=2.0, tau=1e-4),
        # the largest parameter set, Alg. 1 and the packer: the memory-bound end of the range
        dict(name="flat_select_pack", kind="select_pack", model="flat-1000000000", alpha=4.0, tau=-1.0),
        # decode and sum of 8 dense messages into a fresh gradient buffer at that size
        dict(name="flat_decode_8", kind="decode", model="flat-1000000000", p=8, rho=0.17, call="overwrite"),
        # the paper's own regime: messages of a thousandth of the parameters, decode fused with Momentum SGD
        dict(name="vgg16_apply_sgd_sparse", kind="apply", model="vgg16", p=8, rho=0.001, opt="sgd"),
        # early training: dense messages, decode fused with Adam
        dict(name="resnet50_apply_adam", kind="apply", model="resnet50", p=8, rho=0.17, opt="adam"),
        # compressed indexes: encode the own message, decode those of 8 workers
        dict(name="vgg16_compact", kind="compact", model="vgg16", p=8, rho=0.17, alpha=4.0),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _model(rng, hi=5e8):
    k = rng.randrange(5)
    if k < 2:
        return ("resnet50", "vgg16")[k]
    if k == 2:
        return "flat-%d" % int(_log(rng, 2e4, hi))
    return "ragged-%d-%d" % (int(_log(rng, 2e4, min(hi, 2e8))), rng.randrange(1 << 20))


def draw(rng):
    kind = rng.choice(["stat_fc", "fused_fc", "stat_conv", "stat_conv", "select_pack", "decode", "apply", "compact"])
    dtype = rng.choice(["f32", "bf16"])
    alpha = round(rng.choice([0.5, 1.0, 2.0, 4.0]) * rng.uniform(0.9, 1.1), 3)
    rho = round(_log(rng, 5e-4, 0.3), 6)
    if kind == "stat_fc":
        return dict(kind=kind, dims="%d-%d" % (int(_log(rng, 64, 25088)), int(_log(rng, 10, 4096))), B=rng.randrange(8, 129),
                    dtype=dtype, g=rng.random() < 0.5)
    if kind == "fused_fc":
        return dict(kind=kind, J=int(_log(rng, 256, 25088)), C=rng.choice([256, 512, 1024, 2048, 4096]), B=rng.randrange(8, 129),
                    dtype=dtype, alpha=alpha)
    if kind == "stat_conv":
        k, st = rng.choice([(1, 1), (1, 2), (3, 1), (3, 1), (3, 2), (5, 1), (7, 2)])
        H = int(_log(rng, 7, 113))
        most = min(512, int(2e5 / (H * H)) + 64)                 # channels get fewer as the extent grows, as in a network
        first = k == 7 or rng.random() < 0.1
        return dict(kind=kind, H=H, W=max(7, H + rng.choice([0, 0, 0, -1, 1, 3])), Cin=3 if first else 8 * int(_log(rng, 2, most / 8)),
                    C=8 * int(_log(rng, 2, most / 8 + 1)), k=min(k, 7), stride=st, pad=k // 2, B=rng.randrange(8, 65), dtype=dtype,
                    g=rng.random() < 0.3)
    if kind == "select_pack":
        return dict(kind=kind, model=_model(rng), alpha=alpha, tau=rng.choice([-1.0, -1.0, 1e-4]))
    if kind == "decode":
        return dict(kind=kind, model=_model(rng), p=rng.randrange(1, 12), rho=rho, call=rng.choice(["overwrite", "add", "each"]))
    if kind == "apply":
        return dict(kind=kind, model=_model(rng), p=rng.randrange(1, 17), rho=rho, opt=rng.choice(["sgd", "adam"]))
    return dict(kind=kind, model=_model(rng, 2e8), p=rng.randrange(1, 10), rho=max(rho, 0.002), alpha=alpha)


# ---------------------------------------------------------------------------------------
# shapes
# ---------------------------------------------------------------------------------------
def _sizes(model):
    if model == "mlp":
        return [L["size"] for L in W.mlp_layers()]
    if model == "resnet50":
        return [L["size"] for L in W.resnet50_layers()]
    if model == "vgg16":
        return [L["size"] for L in W.vgg16_layers()]
    word = model.split("-")
    n = int(word[1])
    if word[0] == "flat":
        return [size for _, size in W.flat_groups(n)]
    # ragged: weight matrices of every size with bias-sized groups between them
    rng, out, left = torch.Generator().manual_seed(int(word[2])), [], n
    while left > 0:
        u, b = torch.rand(2, generator=rng).tolist()
        w = min(left, max(64, int(n ** (0.5 + 0.45 * u))))
        out.append(w)
        left -= w
        b = min(left, 16 + int(2000 * b))
        if b:
            out.append(b)
            left -= b
    return out


def _resnet50_convs():
    """(Cin, C, input extent, kernel, stride) of the 53 convolutions; the stride sits in the 3x3 convolution."""
    out, cin, prev = [(3, 64, 224, 7, 2)], 64, 56
    for width, blocks, sp in ((64, 3, 56), (128, 4, 28), (256, 6, 14), (512, 3, 7)):
        for b in range(blocks):
            into = prev if b == 0 else sp
            out += [(cin, width, into, 1, 1), (width, width, into, 3, into // sp), (width, 4 * width, sp, 1, 1)]
            if b == 0:
                out.append((cin, 4 * width, into, 1, into // sp))
            cin = 4 * width
        prev = sp
    return out


def _vgg16_convs():
    return [(L["J"] // 9, L["C"], math.isqrt(L["P"]), 3, 1) for L in W.vgg16_layers() if L["kind"] == "conv"]


def _convs(case):
    """[(H, W, Cin, C, k, stride, pad)] of a statistic case on convolutions."""
    if case["kind"] == "stat_conv":
        return [(case["H"], case["W"], case["Cin"], case["C"], case["k"], case["stride"], case["pad"])]
    table = _vgg16_convs() if case["net"] == "vgg16" else _resnet50_convs()
    return [(sp, sp, cin, c, k, st, k // 2) for cin, c, sp, k, st in table]


def _fcs(case):
    d = [int(x) for x in case["dims"].split("-")]
    return list(zip(d, d[1:]))


# ---------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _randn(gen, *shape):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _layer_inputs(gen, shape_x, shape_d, dtype, first, sigma=1e-3):
    """Activations (those of a network's first layer are standardised pixels, all others come out of a ReLU) and output
    gradients of one layer."""
    X = _randn(gen, *shape_x)
    if not first:
        X = X.relu_()
    return X.to(dtype), _randn(gen, *shape_d).mul_(sigma).to(dtype)


def _stream(gen, sizes, batch, alpha):
    """g, s of a step and the state r, v of a running training, flat over all groups: per-sample gradients are
    N(0, sigma^2) with sigma spread over layers (1e-5 .. 1e-2) and over parameters (log-normal).  The mean and the sum of
    squares of `batch` such draws are taken from their own distributions (normal; chi-square by Wilson and Hilferty)."""
    n = sum(sizes)
    layer = torch.empty(len(sizes), device="cuda").uniform_(math.log(1e-5), math.log(1e-2), generator=gen).exp_()
    ends = torch.tensor(sizes, device="cuda").cumsum(0)
    g, s, r, v = (torch.empty(n, device="cuda") for _ in range(4))
    k = batch - 1
    for lo in range(0, n, CHUNK):
        hi = min(n, lo + CHUNK)
        m = hi - lo
        sigma = layer[torch.searchsorted(ends, torch.arange(lo, hi, device="cuda"), right=True)]
        sigma *= _randn(gen, m).mul_(0.5).exp_()
        mean = _randn(gen, m).mul_(sigma).div_(math.sqrt(batch))
        chi = _randn(gen, m).mul_(math.sqrt(2 / (9 * k))).add_(1 - 2 / (9 * k)).clamp_(min=0.05).pow_(3).mul_(k)
        g[lo:hi] = mean
        s[lo:hi] = (mean * mean * batch + sigma * sigma * chi) / batch ** 2
        v[lo:hi] = s[lo:hi] * torch.rand(m, generator=gen, device="cuda").mul_(4)
        r[lo:hi] = (v[lo:hi] * alpha).sqrt_() * torch.rand(m, generator=gen, device="cuda").mul_(1.4).sub_(0.7)
    return g, s, r, v


def _message(gen, sizes, rho):
    """One worker's message before encoding: global element numbers (ascending), their 4-bit values sign << 3 | d,
    group of every element, words per group and the groups' exponent fields."""
    n, n_groups = sum(sizes), len(sizes)
    ends = torch.tensor(sizes, device="cuda").cumsum(0)
    at, code, group = [], [], []
    for lo in range(0, n, CHUNK):
        m = min(n, lo + CHUNK) - lo
        i = (torch.rand(m, generator=gen, device="cuda") < rho).nonzero().flatten().add_(lo)
        at.append(i)
        code.append(torch.randint(0, 16, (i.numel(),), generator=gen, device="cuda", dtype=torch.int32))
        group.append(torch.searchsorted(ends, i, right=True).to(torch.int32))
    at, code, group = torch.cat(at), torch.cat(code), torch.cat(group)
    count = torch.bincount(group, minlength=n_groups)
    field = torch.randint(100, 119, (n_groups,), generator=gen, device="cuda")
    return at, code, group, count, torch.where(count > 0, field, 0)


def _starts(sizes):
    t = torch.tensor(sizes, device="cuda")
    return t.cumsum(0) - t


def _headers(field, count, word_offset):
    lo = (count << 32) | field
    return torch.stack([lo, word_offset], 1).view(torch.uint8).flatten()


def _words(sizes, msg):
    """The message as 32-bit words and headers."""
    at, code, group, count, field = msg
    local = at - _starts(sizes)[group.long()]
    return (local.to(torch.int32) | (code << 28)), _headers(field, count, count.cumsum(0) - count)


def _compact(sizes, msg):
    """The message with compressed indexes: stream, bytes per tile, byte offset of every run of 64 tiles, headers."""
    at, code, group, count, field = msg
    T, size = vgc.tile_size(), torch.tensor(sizes, device="cuda")
    tiles = (size + T - 1) // T
    first_tile = tiles.cumsum(0) - tiles
    n_tiles = int(tiles.sum())
    local = at - _starts(sizes)[group.long()]
    tile = first_tile[group.long()] + local // T
    pos = local % T
    before = torch.full_like(pos, -1)
    before[1:] = torch.where(tile[1:] == tile[:-1], pos[:-1], -1)
    gap = pos - before - 1
    long = gap >= 8
    width = 1 + long.to(torch.int64)
    begin = width.cumsum(0) - width
    stream = torch.zeros(int(width.sum()) if at.numel() else 0, dtype=torch.uint8, device="cuda")
    stream[begin] = (torch.where(long, 0x80, 0) | ((gap & 7) << 4) | code).to(torch.uint8)
    stream[begin[long] + 1] = (gap[long] >> 3).to(torch.uint8)
    tile_bytes = torch.zeros(n_tiles, dtype=torch.int64, device="cuda").index_add_(0, tile, width)
    tile_begin = tile_bytes.cumsum(0) - tile_bytes
    runs = torch.cat([torch.arange(f, f + t, 64) for f, t in zip(first_tile.tolist(), tiles.tolist())]).cuda()
    return stream, tile_bytes.to(torch.int16), tile_begin[runs], _headers(field, count, tile_begin[first_tile])


def _received(gen, sizes, p, rho, encode):
    out = []
    for _ in range(p):
        out.append(encode(sizes, _message(gen, sizes, rho)))
    return out


def _groups(sizes):
    return W.groups_from_sizes(sizes)


BATCH = 32           # per-sample gradients behind one (g, s) of the synthetic streams


def prepare(case, seed):
    gen, kind = _gen(seed), case["kind"]
    st = dict(case=case)
    if kind == "stat_fc":
        B, dt, st["layers"] = case["B"], _dtype(case), []
        for n, (J, C) in enumerate(_fcs(case)):
            X, D = _layer_inputs(gen, (B, J), (B, C), dt, n == 0)
            nb = vgc.sqgrad_workspace_bytes(vgc.FC, vgc.BF16 if dt == torch.bfloat16 else vgc.F32, B, 1, J, C)
            st["layers"].append(dict(X=X, D=D, s=torch.empty(J, C, device="cuda"), g=torch.empty(J, C, device="cuda") if case["g"] else None,
                                     ws=torch.empty(nb, dtype=torch.uint8, device="cuda") if nb else None))
    elif kind in ("stat_net", "stat_conv"):
        B, dt, st["layers"] = case["B"], _dtype(case), []
        want_g = case.get("g", False)
        for H, Wd, Cin, C, k, stride, pad in _convs(case):
            Ho, Wo = (H + 2 * pad - k) // stride + 1, (Wd + 2 * pad - k) // stride + 1
            A, D = _layer_inputs(gen, (B, H, Wd, Cin), (B, Ho, Wo, C), dt, Cin == 3)
            J = k * k * Cin
            nb = vgc.sqgrad_conv2d_workspace_bytes(vgc.BF16 if dt == torch.bfloat16 else vgc.F32, B, H, Wd, Cin, C, k, k, (stride, stride), (pad, pad))
            st["layers"].append(dict(act=A, D=D, kh=k, kw=k, stride=(stride, stride), pad=(pad, pad), c=1.0 / B,
                                     s_out=torch.empty(J, C, device="cuda"), g_out=torch.empty(J, C, device="cuda") if want_g else None,
                                     workspace=torch.empty(nb, dtype=torch.uint8, device="cuda") if nb else None))
    elif kind == "fused_fc":
        B, J, C, dt = case["B"], case["J"], case["C"], _dtype(case)
        st["X"], st["D"] = _layer_inputs(gen, (B, J), (B, C), dt, False)
        st["plan"] = plan = vgc.Plan(_groups([J * C]), "cuda")
        v = torch.rand(J * C, generator=gen, device="cuda").mul_(2e-6 / B)         # a few steps' worth of s
        st["v"], st["r"] = v, (v * case["alpha"]).sqrt_() * torch.rand(J * C, generator=gen, device="cuda").mul_(1.4).sub_(0.7)
        nb = vgc.sqgrad_accumulate_select_workspace_bytes(vgc.BF16 if dt == torch.bfloat16 else vgc.F32, B, J, C)
        st["ws"] = torch.empty(nb, dtype=torch.uint8, device="cuda")
        _sender(st, plan)
    else:
        sizes = _sizes(case["model"])
        st["plan"] = plan = vgc.Plan(_groups(sizes), "cuda")
        n = plan.n
        if kind in ("select_pack", "exchange", "compact"):
            st["g"], st["s"], st["r"], st["v"] = _stream(gen, sizes, BATCH, case["alpha"])
            if kind == "compact":
                st["scratch"] = plan.new_scratch()
                vgc.accumulate_select(st["g"], st["s"], st["r"], st["v"], plan, case["alpha"], ZETA, st["scratch"])
                for name in ("g", "s", "r", "v"):
                    del st[name]
                st["stream"] = torch.zeros(2 * n, dtype=torch.uint8, device="cuda")
                st["tile_bytes"] = torch.zeros(plan.n_tiles, dtype=torch.int16, device="cuda")
                st["run_offsets"] = torch.zeros(plan.n_runs, dtype=torch.int64, device="cuda")
                st["hdrs"], st["status"] = plan.new_headers(), plan.new_status()
            else:
                _sender(st, plan)
        if kind in ("decode", "compact"):
            st["dense"] = torch.zeros(n, device="cuda")
        if kind in ("decode", "apply", "exchange"):
            others = case["p"] - (1 if kind == "exchange" else 0)
            msgs = _received(gen, sizes, others, case["rho"], _words)
            st["words_in"], st["hdrs_in"] = [m[0] for m in msgs], [m[1] for m in msgs]
            st["n_in"] = [w.numel() for w in st["words_in"]]
            if kind == "exchange":                     # this worker's own message; its length is bounded by n
                st["words_in"].append(st["words"]); st["hdrs_in"].append(st["hdrs"]); st["n_in"].append(n)
        if kind == "compact":
            msgs = _received(gen, sizes, case["p"], case["rho"], _compact)
            st["streams_in"], st["tile_bytes_in"], st["runs_in"], st["hdrs_in"] = ([m[i] for m in msgs] for i in range(4))
            st["n_in"] = [x.numel() for x in st["streams_in"]]
        if kind in ("apply", "exchange"):
            st["param"] = _randn(gen, n).mul_(0.02)
            st["m"] = _randn(gen, n).mul_(1e-4)
            if case.get("opt") == "adam":
                st["m2"] = _randn(gen, n).mul_(1e-4).square_()
    return st


def _sender(st, plan):
    st["scratch"] = plan.new_scratch()
    st["words"] = torch.zeros(plan.n, dtype=torch.int32, device="cuda")
    st["hdrs"], st["status"] = plan.new_headers(), plan.new_status()


SGD = dict(lr=0.1, momentum=0.9)
ADAM = dict(lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-8, step=7)


# ---------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------
def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "stat_fc":
        for L in st["layers"]:
            vgc.sqgrad(vgc.FC, L["X"], L["D"], 1.0 / case["B"], L["s"], L["g"], L["ws"])
        return [(L["s"], L["g"]) for L in st["layers"]]
    if kind == "stat_net":
        vgc.sqgrad_conv2d_batch(st["layers"])
        return [(L["s_out"], L["g_out"]) for L in st["layers"]]
    if kind == "stat_conv":
        L = st["layers"][0]
        vgc.sqgrad_conv2d(**L)
        return [(L["s_out"], L["g_out"])]
    plan = st["plan"]
    if kind == "fused_fc":
        vgc.sqgrad_accumulate_select(st["X"], st["D"], 1.0 / case["B"], st["r"], st["v"], plan, 0, case["alpha"], ZETA, st["scratch"], st["ws"])
        vgc.pack(plan, st["scratch"], st["words"], st["hdrs"], st["status"])
        return _sent(st)
    if kind in ("select_pack", "exchange"):
        if case.get("tau", -1.0) >= 0:
            vgc.accumulate_select_hybrid(st["g"], st["s"], st["r"], st["v"], plan, case["alpha"], ZETA, case["tau"], st["scratch"])
        else:
            vgc.accumulate_select(st["g"], st["s"], st["r"], st["v"], plan, case["alpha"], ZETA, st["scratch"])
        vgc.pack(plan, st["scratch"], st["words"], st["hdrs"], st["status"])
        if kind == "select_pack":
            return _sent(st)
    if kind == "decode":
        scale = 1.0 / case["p"]
        if case["call"] == "each":
            for w, k, h in zip(st["words_in"], st["n_in"], st["hdrs_in"]):
                vgc.unpack_add(w, k, h, plan, scale, st["dense"])
        else:
            vgc.unpack_add_batch(st["words_in"], st["n_in"], st["hdrs_in"], plan, scale, st["dense"], overwrite=case["call"] == "overwrite")
        return st["dense"]
    if kind == "compact":
        vgc.pack_compact(plan, st["scratch"], st["stream"], st["tile_bytes"], st["run_offsets"], st["hdrs"], st["status"])
        vgc.unpack_compact_add_batch(st["streams_in"], st["n_in"], st["tile_bytes_in"], st["runs_in"], st["hdrs_in"], plan, 1.0 / case["p"],
                                     st["dense"], overwrite=True)
        return dict(dense=st["dense"], stream=st["stream"], tile_bytes=st["tile_bytes"], run_offsets=st["run_offsets"], hdrs=st["hdrs"],
                    status=st["status"])
    adam = case.get("opt") == "adam"
    vgc.unpack_apply(st["words_in"], st["n_in"], st["hdrs_in"], plan, 1.0 / case["p"], st["param"], st["m"], st.get("m2"),
                     kind=vgc.ADAM if adam else vgc.MOMENTUM_SGD, **(ADAM if adam else SGD))
    out = dict(param=st["param"], m=st["m"], m2=st.get("m2"))
    return {**out, **_sent(st)} if kind == "exchange" else out


def _sent(st):
    return dict(r=st["r"], v=st["v"], words=st["words"], hdrs=st["hdrs"], status=st["status"])


# ---------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------
def work(case):
    kind, size = case["kind"], 2 if case.get("dtype") == "bf16" else 4
    by, fl = 0.0, 0.0
    if kind == "stat_fc":
        outs = 2 if case["g"] else 1
        for J, C in _fcs(case):
            by += size * case["B"] * (J + C) + 4.0 * outs * J * C
            fl += 2.0 * outs * case["B"] * J * C
    elif kind in ("stat_net", "stat_conv"):
        for H, Wd, Cin, C, k, stride, pad in _convs(case):
            P = ((H + 2 * pad - k) // stride + 1) * ((Wd + 2 * pad - k) // stride + 1)
            J = k * k * Cin
            by += size * case["B"] * (H * Wd * Cin + P * C) + 4.0 * J * C * (2 if case.get("g") else 1)
            fl += 2.0 * case["B"] * P * J * C
    elif kind == "fused_fc":
        J, C, B = case["J"], case["C"], case["B"]
        by = size * B * (J + C) + 16.0 * J * C + 4.0 * _density(case) * J * C
        fl = 4.0 * B * J * C
    else:
        n = float(sum(_sizes(case["model"])))
        if kind in ("select_pack", "exchange"):
            by += 24 * n + 4 * _density(case) * n
        if kind == "compact":                          # the staged result (two bytes an element), its code and the decoded messages
            by += (2 + 1.3) * _density(case) * n + 1.3 * case["p"] * case["rho"] * n + 4 * n
        if kind == "decode":
            by += 4 * case["p"] * case["rho"] * n
            touched = 1 - (1 - case["rho"]) ** case["p"]
            by += 4 * n if case["call"] == "overwrite" else 8 * n * touched
        if kind in ("apply", "exchange"):
            by += 4 * case["p"] * case["rho"] * n + (24 if case.get("opt") == "adam" else 16) * n
        fl = n
    return {"bytes": by, "flops": fl}


def _density(case):
    """About the share of the parameters that one pass sends (normal gradients, this alpha)."""
    return 0.3 / max(1.0, math.sqrt(case["alpha"]))


def tolerance(case):
    kind = case["kind"]
    if kind in ("stat_net", "stat_conv"):              # 32-bit sums in any order (1e-7 to 3e-7 from 64 bits; more where few samples cancel)
        return {"rel": 4e-6}
    if kind == "stat_fc":                              # 16-bit inputs: the squares are rounded to 16 bits, 2^-9 a factor (9e-4 from 64 bits)
        return {"rel": 4e-3 if case["dtype"] == "bf16" else 2e-6}
    if kind == "fused_fc":                             # r, v after a test against sums in another order: single elements flip
        return {"rel": 3e-3, "max": 0.99, "differ": 0.01}
    return "exact"                                     # one rounding per operation, in the order the interface states


# ---------------------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------------------
def _conv_sums(A, D, k, stride, pad, c):
    """c sum_z G_z and c^2 sum_z G_z^2 of one convolution in 64 bits, rows (ky, kx, i), a few samples at a time."""
    B, H, Wd, Cin = A.shape
    C, P = D.shape[3], D.shape[1] * D.shape[2]
    J = k * k * Cin
    g = torch.zeros(J, C, dtype=torch.float64, device="cuda")
    s = torch.zeros_like(g)
    step = max(1, min(B, int(3e8 // (J * P + J * C))))
    for z in range(0, B, step):
        x = A[z:z + step].double().permute(0, 3, 1, 2).contiguous()
        U = x.reshape(x.shape[0], Cin, -1) if k == 1 and stride == 1 else F.unfold(x, k, padding=pad, stride=stride)
        G = torch.bmm(U, D[z:z + step].double().reshape(-1, P, C))
        g += G.sum(0)
        s += G.square_().sum(0)
    order = lambda t: (t.reshape(Cin, k * k, C).transpose(0, 1).reshape(J, C))
    return order(g) * c, order(s) * (c * c)


def _f32(x):
    return float(torch.tensor(x, dtype=torch.float32))


def _selected(st, g, s):
    """r, v after the step, the accumulated gradient and the send mask, in 64 bits."""
    case = st["case"]
    alpha, zeta, tau = _f32(case["alpha"]), _f32(ZETA), case.get("tau", -1.0)
    r, v = torch.empty_like(st["r"], dtype=torch.float64), torch.empty_like(st["v"], dtype=torch.float64)
    acc, send = torch.empty_like(r), torch.empty_like(st["r"], dtype=torch.bool)
    for lo in range(0, r.numel(), CHUNK):
        at = slice(lo, min(lo + CHUNK, r.numel()))
        ra, va = st["r"][at].double() + g[at].double(), st["v"][at].double() + s[at].double()
        sent = ra * ra > alpha * va
        acc[at] = ra
        if tau >= 0:
            t = _f32(tau)
            sent &= ra.abs() > t
            r[at] = torch.where(sent, ra - torch.sign(ra) * t, ra)
            v[at] = zeta * torch.where(sent, (va - 2 * t * ra.abs() + t * t).clamp_(min=0), va)
        else:
            r[at] = torch.where(sent, 0.0, ra)
            v[at] = torch.where(sent, 0.0, zeta * va)
        send[at] = sent
    return r, v, acc, send


def _decoded(gen, sizes, p, rho, scale):
    """The sum of p received messages, drawn as prepare() draws them."""
    out = torch.zeros(sum(sizes), dtype=torch.float64, device="cuda")
    for _ in range(p):
        at, code, group, _, field = _message(gen, sizes, rho)
        val = torch.ldexp(torch.ones_like(at, dtype=torch.float64), field[group.long()] - (code & 7) - 127)
        out[at] += torch.where(code >= 8, -val, val) * scale
    return out


def _own(sizes, acc, send, scale):
    """What this worker's own message decodes to: the sent elements rounded to powers of two, group by group."""
    out = torch.zeros_like(acc)
    for (lo, size) in _groups(sizes):
        a, on = acc[lo:lo + size], send[lo:lo + size]
        m, e = torch.frexp(a.abs())
        top = torch.where(on, e, -1000).max()
        er = torch.minimum(torch.where(m >= 0.75, e, e - 1), top - 1)
        keep = on & (top - 1 - er <= 7)
        out[lo:lo + size] = torch.where(keep, torch.sign(a) * torch.ldexp(torch.ones_like(a), er), 0.0) * scale
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind in ("stat_net", "stat_conv"):
        out = []
        for L in prepare(case, seed)["layers"]:
            g, s = _conv_sums(L["act"], L["D"], L["kh"], L["stride"][0], L["pad"][0], _f32(L["c"]))
            out.append((s, g if L["g_out"] is not None else None))
        return out
    if kind == "stat_fc":
        out, c = [], _f32(1.0 / case["B"])
        for L in prepare(case, seed)["layers"]:
            x, d = L["X"].double().t().contiguous(), L["D"].double()
            out.append(((x * x) @ (d * d) * (c * c), x @ d * c if case["g"] else None))
        return out
    nothing = dict(words=None, hdrs=None, status=None)
    st = prepare(case, seed)
    if kind == "fused_fc":
        c = _f32(1.0 / case["B"])
        x, d = st["X"].double().t().contiguous(), st["D"].double()
        r, v, _, _ = _selected(st, (x @ d * c).flatten(), ((x * x) @ (d * d) * (c * c)).flatten())
        return dict(r=r, v=v, **nothing)
    if kind in ("select_pack", "exchange"):
        r, v, acc, send = _selected(st, st["g"], st["s"])
        if kind == "select_pack":
            return dict(r=r, v=v, **nothing)
    # the received messages are drawn after what prepare() drew for the sending side
    sizes, scale = _sizes(case["model"]), _f32(1.0 / case["p"])
    gen = _gen(seed)
    if kind in ("exchange", "compact"):
        _stream(gen, sizes, BATCH, case["alpha"])
    ghat = _decoded(gen, sizes, case["p"] - (kind == "exchange"), case["rho"], scale)
    if kind == "decode":
        return ghat
    if kind == "compact":
        return dict(dense=ghat, stream=None, tile_bytes=None, run_offsets=None, hdrs=None, status=None)
    if kind == "exchange":
        ghat += _own(sizes, acc, send, scale)
    if case.get("opt") == "adam":
        lr, b1, b2, eps = (_f32(ADAM[k]) for k in ("lr", "beta1", "beta2", "eps"))
        m = b1 * st["m"].double() + _f32(1 - b1) * ghat
        m2 = b2 * st["m2"].double() + _f32(1 - b2) * ghat * ghat
        step = lr * (m / _f32(1 - b1 ** ADAM["step"])) / ((m2 / _f32(1 - b2 ** ADAM["step"])).sqrt() + eps)
        return dict(param=st["param"].double() - step, m=m, m2=m2)
    m = _f32(SGD["momentum"]) * st["m"].double() - _f32(SGD["lr"]) * ghat
    out = dict(param=st["param"].double() + m, m=m, m2=None)
    return dict(**out, r=r, v=v, **nothing) if kind == "exchange" else out
