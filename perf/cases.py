"""The workloads this framework is timed on, and their 64-bit references.

A case is one pass of a per-replica BigGAN workload through the public entry
points of paragan_2411_03999_amd.lib: a training forward and backward of one
module (spectral norm, generator block, discriminator block, self-attention,
generator output layer), sampling from the generator, a discriminator step,
or the whole training iteration.  listed() holds the fixed cases, draw() one
more case of the same ranges, prepare() / run() / work() / tolerance() their
inputs, call, unavoidable work and accuracy, exact() the same outputs in
float64 from plain torch (matrix products, no code of this package).
"""
import ctypes
import math

import torch

from paragan_2411_03999_amd import lib

DEV = "cuda"
BN_EPS, SN_EPS = 1e-5, 1e-12

# img, ch, g_mult, d_mult, d_down, attn_res, n_classes, dz, shared_dim
ARCHS = {
    "biggan128": (128, 96, (16, 16, 8, 4, 2, 1), (1, 2, 4, 8, 16, 16), (1, 1, 1, 1, 1, 0), 64, 1000, 120, 128),
    "biggan512": (512, 64, (16, 16, 8, 8, 4, 2, 1, 1), (1, 1, 2, 4, 8, 8, 16, 16), (1, 1, 1, 1, 1, 1, 1, 0), 64, 1000,
                  128, 128),
}


def listed():
    return [
        # one SN weight normalised on its own: launch latency
        {"name": "sn_192x1728", "kind": "sn", "rows": 192, "cols": 1728, "iters": 1},
        # the small fp32 generator block (8 x 8, 64 channels, batch 4): a step of a
        # small model or a numerics check, many short launches
        {"name": "gblock_f32_b4_8x8_64", "kind": "gblock", "f32": 1, "B": 4, "H": 8, "W": 8, "cin": 64, "cout": 64,
         "dc": 128},
        # BigGAN-128's first generator block at a small per-GPU batch: 35 M
        # weights against 1024 output pixels
        {"name": "gblock_b16_4x4_1536", "kind": "gblock", "f32": 0, "B": 16, "H": 4, "W": 4, "cin": 1536, "cout": 1536,
         "dc": 148},
        # BigGAN-128's last generator block: few channels, 128 x 128 pixels
        {"name": "gblock_b32_64x64_192_96", "kind": "gblock", "f32": 0, "B": 32, "H": 64, "W": 64, "cin": 192,
         "cout": 96, "dc": 148},
        # the discriminator block of the framework's block benchmark
        {"name": "dblock_b64_32x32_256_512", "kind": "dblock", "B": 64, "H": 32, "W": 32, "cin": 256, "cout": 512,
         "pre": 1, "down": 1, "lsc": 1},
        # BigGAN-128's last discriminator block (identity skip) on the 32 + 32 images of a D step
        {"name": "dblock_b64_4x4_1536", "kind": "dblock", "B": 64, "H": 4, "W": 4, "cin": 1536, "cout": 1536, "pre": 1,
         "down": 0, "lsc": 0},
        # a discriminator block of a model with other widths and image sides: nothing is a tile multiple
        {"name": "dblock_b7_28x20_72_136", "kind": "dblock", "B": 7, "H": 28, "W": 20, "cin": 72, "cout": 136, "pre": 1,
         "down": 1, "lsc": 1},
        # the discriminator's self-attention at 64 x 64
        {"name": "attn_b32_64x64_96", "kind": "attn", "B": 32, "H": 64, "W": 64, "C": 96},
        # the generator's output layer at 128 x 128
        {"name": "gout_b32_128x128_96", "kind": "gout", "B": 32, "H": 128, "W": 128, "C": 96},
        # sampling: a handful of images from the BigGAN-128 generator
        {"name": "g_sample_128_b8", "kind": "g_sample", "arch": "biggan128", "B": 8},
        # a discriminator step on 32 real + 32 fake images
        {"name": "d_step_128_b32", "kind": "d_step", "arch": "biggan128", "B": 32},
        # the training iteration at the per-GPU batch of the headline benchmark
        {"name": "train_128_b256", "kind": "train", "arch": "biggan128", "B": 256, "n_D": 2},
    ]


def _log(rng, a, b):
    return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))


def draw(rng):
    kind = rng.choice(["sn", "gblock", "gblock", "gblock_f32", "dblock", "dblock", "attn", "gout", "g_sample", "d_step",
                       "train"])
    if kind == "sn":
        return {"kind": "sn", "rows": _log(rng, 3, 1536), "cols": _log(rng, 20, 13824), "iters": rng.choice([1, 1, 2])}
    if kind == "gblock_f32":
        return {"kind": "gblock", "f32": 1, "B": _log(rng, 1, 8), "H": _log(rng, 4, 16), "W": _log(rng, 4, 16),
                "cin": _log(rng, 8, 96), "cout": _log(rng, 8, 96), "dc": rng.randint(16, 148)}
    while kind in ("gblock", "dblock"):
        if rng.random() < 0.5:   # the widths and sides of the BigGAN models
            ch = rng.choice([64, 96])
            side, hi, lo = rng.choice([(4, 16, 16), (8, 16, 8), (16, 8, 4), (32, 4, 2), (64, 2, 1)])
            c = {"B": _log(rng, 2, 128), "H": side, "W": side, "cin": hi * ch, "cout": lo * ch}
        else:
            c = {"B": _log(rng, 1, 64), "H": _log(rng, 4, 48), "W": _log(rng, 4, 48), "cin": _log(rng, 16, 512),
                 "cout": _log(rng, 16, 512)}
        if kind == "gblock":
            c = {"kind": "gblock", "f32": 0, "dc": rng.randint(100, 160), **c}
        else:
            down = rng.random() < 0.75
            c["cin"], c["cout"] = c["cout"], c["cin"]
            if down:
                c["H"], c["W"] = 2 * c["H"], 2 * c["W"]
            c = {"kind": "dblock", "pre": 1, "down": int(down), "lsc": int(down or c["cin"] != c["cout"]), **c}
        if work(c)["flops"] <= 1.5e12:
            return c
    if kind == "attn":
        return {"kind": "attn", "B": _log(rng, 1, 64), "H": 2 * _log(rng, 4, 32), "W": 2 * _log(rng, 4, 32),
                "C": 8 * rng.randint(4, 32)}
    if kind == "gout":
        return {"kind": "gout", "B": _log(rng, 1, 48), "H": _log(rng, 16, 160), "W": 4 * _log(rng, 4, 40),
                "C": 8 * rng.randint(3, 16)}
    if kind == "g_sample":
        arch = rng.choice(["biggan128", "biggan128", "biggan512"])
        return {"kind": "g_sample", "arch": arch, "B": _log(rng, 2, 64 if arch == "biggan128" else 8)}
    if kind == "d_step":
        arch = rng.choice(["biggan128", "biggan128", "biggan512"])
        return {"kind": "d_step", "arch": arch, "B": _log(rng, 4, 64 if arch == "biggan128" else 8)}
    arch = rng.choice(["biggan128", "biggan512"])
    return {"kind": "train", "arch": arch, "B": _log(rng, 8, 128) if arch == "biggan128" else _log(rng, 4, 16),
            "n_D": rng.randint(1, 2)}


# ------------------------------------------------------------- parameters
def cpad(c):
    return (c + 31) // 32 * 32


def _gblock_shapes(cin, cout, dc, pre=""):
    return [(pre + n, s, sn) for n, s, sn in (
        ("bn1.gain", (cin, dc), 1), ("bn1.bias", (cin, dc), 1), ("conv1.w", (cout, 3, 3, cin), 1),
        ("conv1.b", (cout,), 0), ("bn2.gain", (cout, dc), 1), ("bn2.bias", (cout, dc), 1),
        ("conv2.w", (cout, 3, 3, cout), 1), ("conv2.b", (cout,), 0), ("sc.w", (cout, 1, 1, cin), 1),
        ("sc.b", (cout,), 0))]


def _dblock_shapes(cin, cout, lsc, pre=""):
    v = [(pre + "conv1.w", (cout, 3, 3, cin), 1), (pre + "conv1.b", (cout,), 0),
         (pre + "conv2.w", (cout, 3, 3, cout), 1), (pre + "conv2.b", (cout,), 0)]
    return v + ([(pre + "sc.w", (cout, 1, 1, cin), 1), (pre + "sc.b", (cout,), 0)] if lsc else [])


def _attn_shapes(c, pre=""):
    return [(pre + "theta", (c // 8, 1, 1, c), 1), (pre + "phi", (c // 8, 1, 1, c), 1), (pre + "g", (c // 2, 1, 1, c), 1),
            (pre + "o", (c, 1, 1, c // 2), 1), (pre + "gamma", (1,), 0)]


def _gout_shapes(c):
    return [("out_bn.gain", (c,), 0), ("out_bn.bias", (c,), 0), ("out_conv.w", (3, 3, 3, c), 1), ("out_conv.b", (3,), 0)]


def _d_specs(arch):
    img, ch, _, dm, dd, attn, _, _, _ = ARCHS[arch]
    out, res, cin, placed = [], img, 3, False
    for j, (m, down) in enumerate(zip(dm, dd)):
        cout, side = m * ch, res
        res = res // 2 if down else res
        at = not placed and res == attn
        placed = placed or at
        out.append({"cin": cin, "cout": cout, "H": side, "pre": int(j > 0), "down": down,
                    "lsc": int(cin != cout or bool(down)), "attn": at})
        cin = cout
    return out


def _net_shapes(arch, which):
    _, ch, gm, dm, _, attn, ncls, dz, sd = ARCHS[arch]
    v = []
    if which == 0:
        zc = dz // len(gm)
        c0 = gm[0] * ch
        v += [("shared", (ncls, sd), 0), ("linear.w", (16 * c0, zc), 1), ("linear.b", (16 * c0,), 0)]
        for i in range(len(gm) - 1):
            v += _gblock_shapes(gm[i] * ch, gm[i + 1] * ch, sd + zc, "g%d." % i)
            if 4 << (i + 1) == attn:
                v += _attn_shapes(gm[i + 1] * ch, "attn.")
        return v + _gout_shapes(gm[-1] * ch)
    for j, s in enumerate(_d_specs(arch)):
        v += _dblock_shapes(s["cin"], s["cout"], s["lsc"], "d%d." % j)
        if s["attn"]:
            v += _attn_shapes(s["cout"], "attn.")
    c = dm[-1] * ch
    return v + [("head.w", (1, c), 1), ("head.b", (1,), 0), ("embed", (ncls, c), 1)]


def _count(shapes):
    return sum(math.prod(s) for _, s, _ in shapes), sum(s[0] for _, s, sn in shapes if sn)


def _params(shapes, gen):
    """Flat fp32 parameters (weights N(0, 1/fan_in), gains near 1, biases small) and SN vectors u ~ N(0, 1)."""
    n, nu = _count(shapes)
    P = torch.empty(n, device=DEV)
    o = 0
    for name, shape, _ in shapes:
        k = math.prod(shape)
        view = P[o:o + k]
        o += k
        if name.endswith("gamma"):
            view.fill_(0.5)
        elif name == "out_bn.gain":
            view.normal_(1.0, 0.1, generator=gen)
        elif len(shape) >= 2:
            view.normal_(0.0, (k // shape[0]) ** -0.5, generator=gen)
        else:
            view.normal_(0.0, 0.02, generator=gen)
    return P, torch.empty(nu, device=DEV).normal_(generator=gen)


def _nhwc(gen, B, H, W, c, f32, scale=1.0):
    """N(0, scale^2) activations, zero in the padded channels."""
    t = torch.zeros((B, H, W, cpad(c)), device=DEV)
    t[..., :c] = torch.randn((B, H, W, c), device=DEV, generator=gen) * scale
    return t if f32 else t.to(torch.bfloat16)


def _labels(gen, B, n):
    return torch.randint(0, n, (B,), device=DEV, generator=gen, dtype=torch.int32)


def _inputs(case, seed):
    """What the case is computed from, made from the seed alone."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    k, d = case["kind"], {}
    if k == "sn":
        d["W"] = torch.randn((case["rows"], case["cols"]), device=DEV, generator=gen) * case["cols"] ** -0.5
        d["u"] = torch.randn(case["rows"], device=DEV, generator=gen)
        return d
    if k in ("gblock", "dblock", "attn", "gout"):
        B, H, W = case["B"], case["H"], case["W"]
        f32 = case.get("f32", 0)
        if k == "gblock":
            d["P"], d["u"] = _params(_gblock_shapes(case["cin"], case["cout"], case["dc"]), gen)
            d["x"] = _nhwc(gen, B, H, W, case["cin"], f32)
            d["cond"] = torch.randn((B, case["dc"]), device=DEV, generator=gen)
            d["dy"] = _nhwc(gen, B, 2 * H, 2 * W, case["cout"], f32, 1e-2)
        elif k == "dblock":
            s = 2 if case["down"] else 1
            d["P"], d["u"] = _params(_dblock_shapes(case["cin"], case["cout"], case["lsc"]), gen)
            d["x"] = _nhwc(gen, B, H, W, case["cin"], 0)
            d["dy"] = _nhwc(gen, B, H // s, W // s, case["cout"], 0, 1e-2)
        elif k == "attn":
            d["P"], d["u"] = _params(_attn_shapes(case["C"]), gen)
            d["x"] = _nhwc(gen, B, H, W, case["C"], 0)
            d["dy"] = _nhwc(gen, B, H, W, case["C"], 0, 1e-2)
        else:
            d["P"], d["u"] = _params(_gout_shapes(case["C"]), gen)
            d["x"] = _nhwc(gen, B, H, W, case["C"], 0)
            d["dimg"] = torch.randn((B, H, W, 3), device=DEV, generator=gen) * 1e-2
        return d
    img, _, _, _, _, _, ncls, dz, _ = ARCHS[case["arch"]]
    B = case["B"]

    def images():
        return torch.rand((B, img, img, 3), device=DEV, generator=gen) * 2 - 1
    if k in ("g_sample", "train"):
        d["GP"], d["Gu"] = _params(_net_shapes(case["arch"], 0), gen)
        d["z"], d["y"] = torch.randn((B, dz), device=DEV, generator=gen), _labels(gen, B, ncls)
    if k in ("d_step", "train"):
        d["DP"], d["Du"] = _params(_net_shapes(case["arch"], 1), gen)
    if k == "d_step":
        d["xr"], d["yr"], d["xf"], d["yf"] = images(), _labels(gen, B, ncls), images(), _labels(gen, B, ncls)
    if k == "train":
        n = case["n_D"]
        d["xr"], d["yr"] = [images() for _ in range(n)], [_labels(gen, B, ncls) for _ in range(n)]
        d["zf"] = [torch.randn((B, dz), device=DEV, generator=gen) for _ in range(n)]
        d["yf"] = [_labels(gen, B, ncls) for _ in range(n)]
    return d


# ------------------------------------------------------------- the calls
def _biggan_desc(arch, B):
    img, ch, gm, dm, dd, attn, ncls, dz, sd = ARCHS[arch]
    d = lib.BigganDesc()
    d.img, d.ch, d.n_g, d.n_d = img, ch, len(gm) - 1, len(dm)
    for i, m in enumerate(gm):
        d.g_mult[i] = m
    for j, (m, dn) in enumerate(zip(dm, dd)):
        d.d_mult[j], d.d_down[j] = m, dn
    d.attn_res, d.n_classes, d.dz, d.shared_dim, d.B = attn, ncls, dz, sd, B
    d.n_power_iter, d.bn_eps, d.sn_eps = 1, BN_EPS, SN_EPS
    d.opt_g = lib.Optim(lib.ADABELIEF, 1e-4, 0.5, 0.999, 1e-12)
    d.opt_d = lib.Optim(lib.ADAM, 4e-4, 0.0, 0.999, 1e-6)
    return d


def _net_state(P, u):
    bufs = [P, u] + [torch.zeros_like(P) for _ in range(3)]
    return bufs, lib.NetState(*[t.data_ptr() for t in bufs], 0)


def prepare(case, seed):
    s = _inputs(case, seed)
    k = s["kind"] = case["kind"]
    ctx = s["ctx"] = lib.Context()
    assert ctx.h
    if k == "sn":
        s["v"] = torch.empty(case["cols"], device=DEV)
        s["sigma"] = torch.empty(1, device=DEV)
        s["ws"] = lib.workspace(lib.paragan_sn_ws_size(case["rows"], case["cols"]))
        s["iters"] = case["iters"]
        return s
    if k in ("gblock", "dblock", "attn", "gout"):
        B, H, W = case["B"], case["H"], case["W"]
        if k == "gblock":
            d = lib.GBlockDesc(B, H, W, case["cin"], case["cout"], case["dc"], lib.F32 if case["f32"] else lib.BF16, 1,
                               BN_EPS, SN_EPS)
            (saved, ws), n = lib.paragan_gblock_sizes(d), lib.paragan_gblock_layout(d)[1]
            s["out"], s["dcond"] = torch.zeros_like(s["dy"]), torch.empty_like(s["cond"])
        elif k == "dblock":
            d = lib.DBlockDesc(B, H, W, case["cin"], case["cout"], case["pre"], case["down"], case["lsc"], lib.BF16, 1,
                               SN_EPS)
            (saved, ws), n = lib.paragan_dblock_sizes(d), lib.paragan_dblock_layout(d)[1]
            s["out"] = torch.zeros_like(s["dy"])
        elif k == "attn":
            d = lib.AttnDesc(B, H, W, case["C"], 1, SN_EPS)
            (saved, ws), n = lib.paragan_attn_sizes(d), lib.paragan_attn_layout(d)[1]
            s["out"] = torch.zeros_like(s["dy"])
        else:
            d = lib.GoutDesc(B, H, W, case["C"], 1, BN_EPS, SN_EPS)
            (saved, ws), n = lib.paragan_gout_sizes(d), lib.paragan_gout_layout(d)[1]
            s["out"] = torch.empty_like(s["dimg"])
        assert n == s["P"].numel()
        s["desc"], s["saved"], s["ws"] = d, lib.workspace(saved), lib.workspace(ws)
        s["dx"], s["grads"] = torch.zeros_like(s["x"]), torch.zeros_like(s["P"])
        return s
    d = s["desc"] = _biggan_desc(case["arch"], case["B"])
    s["ws"] = lib.workspace(lib.paragan_train_step_ws_size(d))
    if "GP" in s:
        assert lib.paragan_net_layout(d, 0)[1] == s["GP"].numel()
        s["Gbufs"], s["G"] = _net_state(s["GP"], s["Gu"])
    if "DP" in s:
        assert lib.paragan_net_layout(d, 1)[1] == s["DP"].numel()
        s["Dbufs"], s["D"] = _net_state(s["DP"], s["Du"])
    if k == "g_sample":
        s["img"] = torch.empty((case["B"], d.img, d.img, 3), device=DEV)
    else:
        n = s["n_D"] = case.get("n_D", 1)
        s["loss"] = (ctypes.c_float * (n + 1))()
        if k == "train":
            ptrs = [(ctypes.c_void_p * n)(*[t.data_ptr() for t in s[a]]) for a in ("xr", "yr", "zf", "yf")]
            s["in"] = lib.StepInputs(*ptrs, s["z"].data_ptr(), s["y"].data_ptr())
    return s


def run(s):
    k, ctx = s["kind"], s["ctx"]
    if k == "sn":
        lib.paragan_sn_power_iter(ctx, s["W"], *s["W"].shape, s["u"], s["v"], s["sigma"], s["iters"], SN_EPS, s["ws"])
        return {"u": s["u"], "v": s["v"], "sigma": s["sigma"]}
    if k == "gblock":
        lib.paragan_gblock_fwd(ctx, s["desc"], s["P"], s["u"], s["x"], s["cond"], s["out"], s["saved"], s["ws"])
        lib.paragan_gblock_bwd(ctx, s["desc"], s["P"], s["x"], s["cond"], s["saved"], s["dy"], s["dx"], s["dcond"],
                               s["grads"], s["ws"])
        return {"y": s["out"], "u": s["u"], "dx": s["dx"], "dcond": s["dcond"], "grads": s["grads"]}
    if k in ("dblock", "attn"):
        fwd, bwd = ((lib.paragan_dblock_fwd, lib.paragan_dblock_bwd) if k == "dblock"
                    else (lib.paragan_attn_fwd, lib.paragan_attn_bwd))
        fwd(ctx, s["desc"], s["P"], s["u"], s["x"], s["out"], s["saved"], s["ws"])
        bwd(ctx, s["desc"], s["P"], s["x"], s["saved"], s["dy"], s["dx"], s["grads"], s["ws"])
        return {"y": s["out"], "u": s["u"], "dx": s["dx"], "grads": s["grads"]}
    if k == "gout":
        lib.paragan_gout_fwd(ctx, s["desc"], s["P"], s["u"], s["x"], s["out"], s["saved"], s["ws"])
        lib.paragan_gout_bwd(ctx, s["desc"], s["P"], s["x"], s["out"], s["saved"], s["dimg"], s["dx"], s["grads"],
                             s["ws"])
        return {"img": s["out"], "u": s["u"], "dx": s["dx"], "grads": s["grads"]}
    if k == "g_sample":
        ctx.check(lib.paragan_g_sample(ctx, s["desc"], s["G"], s["z"], s["y"], s["img"], s["ws"]))
        return {"img": s["img"], "u": s["Gu"]}
    # The step calls return the updated networks and the losses.  (The raw
    # gradients of a whole step amplify a last-bit difference of an early
    # layer to several percent; the updated weights carry them.)
    if k == "d_step":
        ctx.check(lib.paragan_d_step(ctx, s["desc"], s["D"], s["xr"], s["yr"], s["xf"], s["yf"], s["ws"], s["loss"]))
        return {"loss": s["loss"][0], "params": s["DP"], "u": s["Du"]}
    ctx.check(lib.paragan_train_step(ctx, s["desc"], s["G"], s["D"], s["in"], s["n_D"], s["ws"], s["loss"]))
    return {"losses": list(s["loss"]), "g_params": s["GP"], "d_params": s["DP"], "g_u": s["Gu"], "d_u": s["Du"]}


# ------------------------------------------------------------- the work
# FLOPs per pass in the cheapest exact form: a 3x3 conv over a nearest 2x
# upsample is four 2x2 convs over its source, one followed by a 2x2 average
# pool a 4x4 conv at the pooled pixels.  A training pass is three times the
# forward (data and weight gradients), attention recomputes its scores.
def _g_flops(B, H, W, cin, cout):
    return B * H * W * (34.0 * cin * cout + 72.0 * cout * cout)


def _d_flops(B, H, W, cin, cout, down, lsc):
    M = B * H * W
    return M * (18.0 * cin * cout + (8.0 if down else 18.0) * cout * cout + (2.0 / (4 if down else 1)) * cin * cout * lsc)


def _attn_flops(B, H, W, C):
    """(projections, scores and values) of one forward."""
    return 2.0 * B * H * W * C * (1.25 * C), 2.0 * B * H * W * (H * W // 4) * (C // 8 + C // 2)


def _net_flops(arch, B):
    """One forward of G and of D on B images."""
    img, ch, gm, _, _, attn, _, _, _ = ARCHS[arch]
    g = 2.0 * B * img * img * 27 * gm[-1] * ch
    for i in range(len(gm) - 1):
        g += _g_flops(B, 4 << i, 4 << i, gm[i] * ch, gm[i + 1] * ch)
        if 8 << i == attn:
            g += sum(_attn_flops(B, attn, attn, gm[i + 1] * ch))
    d = 0.0
    for s in _d_specs(arch):
        d += _d_flops(B, s["H"], s["H"], s["cin"], s["cout"], s["down"], s["lsc"])
        if s["attn"]:
            d += sum(_attn_flops(B, attn, attn, s["cout"]))
    return g, d


def work(case):
    k = case["kind"]
    if k == "sn":
        n = case["rows"] * case["cols"]
        return {"bytes": 4.0 * (n + 2 * case["rows"] + case["cols"] + 1), "flops": 4.0 * n * case["iters"]}
    if k in ("gblock", "dblock", "attn", "gout"):
        B, M = case["B"], case["B"] * case["H"] * case["W"]
        e = 4 if case.get("f32") else 2
        if k == "gblock":
            n, nu = _count(_gblock_shapes(case["cin"], case["cout"], case["dc"]))
            act = e * M * (2 * cpad(case["cin"]) + 8 * cpad(case["cout"])) + 8 * B * case["dc"]
            flops = 3 * _g_flops(B, case["H"], case["W"], case["cin"], case["cout"])
        elif k == "dblock":
            n, nu = _count(_dblock_shapes(case["cin"], case["cout"], case["lsc"]))
            act = e * M * (2 * cpad(case["cin"]) + 2 * cpad(case["cout"]) // (4 if case["down"] else 1))
            flops = 3 * _d_flops(B, case["H"], case["W"], case["cin"], case["cout"], case["down"], case["lsc"])
        elif k == "attn":
            n, nu = _count(_attn_shapes(case["C"]))
            act = e * M * 4 * cpad(case["C"])
            proj, core = _attn_flops(B, case["H"], case["W"], case["C"])
            L = case["H"] * case["W"] // 4
            flops = 3 * proj + core + 2.0 * M * L * (3 * (case["C"] // 8) + 2 * (case["C"] // 2))
        else:
            n, nu = _count(_gout_shapes(case["C"]))
            act = M * (2 * e * cpad(case["C"]) + 4 * 3 * 2)
            flops = 3 * 2.0 * M * 27 * case["C"]
        return {"bytes": float(act + 8 * n + 8 * nu), "flops": flops}
    B, img = case["B"], ARCHS[case["arch"]][0]
    (gn, gu), (dn, du) = (_count(_net_shapes(case["arch"], w)) for w in (0, 1))
    g, d = _net_flops(case["arch"], B)
    pix = 12.0 * B * img * img
    if k == "g_sample":
        return {"bytes": 4.0 * gn + 8.0 * gu + pix, "flops": g}
    if k == "d_step":   # the optimiser reads and writes weights and moments, the gradient is read and written
        return {"bytes": 28.0 * dn + 8.0 * du + 2 * pix, "flops": 6 * d}
    n = case["n_D"]
    return {"bytes": 28.0 * (gn + n * dn) + 8.0 * (gu + n * du) + n * pix,
            "flops": n * (g + 6 * d) + 3 * g + 2 * d}


def tolerance(case):
    k = case["kind"]
    if k == "sn" or case.get("f32"):
        return {"rel": 1e-5, "max": 1e-3}   # fp32 sums: up to 6e-7 from float64
    # bf16 operands: 2e-3 (outputs) to 4e-2 (gradients, through ReLU decisions that
    # rounding turns) from float64; a ReLU input that a last bit moves across zero
    # turns one element by its own size, hence the wide "max"
    if k in ("gblock", "dblock", "attn"):
        return {"rel": 1e-2, "max": 0.99}
    if k == "gout":
        return {"rel": 7e-3, "max": 0.5}    # the bf16 dx: 1.7e-3 from float64
    return {"rel": 3e-2, "max": 0.99}       # whole networks: 1.9e-2 (images) from float64


# ------------------------------------------------------- 64-bit references
def _norm(t):
    return t / t.norm().clamp_min(SN_EPS)


def _sn(W, u, iters=1):
    """W / sigma (differentiable, u and v constant), and the new u, v, sigma."""
    A = W.reshape(W.shape[0], -1)
    with torch.no_grad():
        for _ in range(iters):
            v = _norm(A.t() @ u)
            u = _norm(A @ v)
    sigma = u @ (A @ v)
    return W / sigma, u, v, sigma


class _Net:
    """Named float64 parameters over flat buffers; normalised weights on request."""

    def __init__(self, shapes, P, u):
        self.flat = P.double().requires_grad_(True)
        self.u = u.double()
        self.w, self.uo = {}, {}
        o = uo = 0
        for name, shape, sn in shapes:
            k = math.prod(shape)
            self.w[name] = self.flat[o:o + k].view(shape)
            o += k
            if sn:
                self.uo[name] = (uo, shape[0])
                uo += shape[0]

    def sn(self, name):
        o, n = self.uo[name]
        W, u, _, _ = _sn(self.w[name], self.u[o:o + n].clone())
        self.u[o:o + n] = u
        return W


def _conv(x, W):
    """NHWC conv, stride 1, same padding, W [Cout][R][R][Cin], as one product per tap."""
    R, (B, H, Wd, _) = W.shape[1], x.shape
    if R == 1:
        return x @ W[:, 0, 0].t()
    xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    y = 0
    for r in range(3):
        for s in range(3):
            y = y + xp[:, r:r + H, s:s + Wd] @ W[:, r, s].t()
    return y


def _up2(x):
    B, H, W, C = x.shape
    return x[:, :, None, :, None].expand(B, H, 2, W, 2, C).reshape(B, 2 * H, 2 * W, C)


def _win(x):
    B, H, W, C = x.shape
    return x.reshape(B, H // 2, 2, W // 2, 2, C)


def _bn(x):
    m = x.mean((0, 1, 2))
    return (x - m) / ((x - m).square().mean((0, 1, 2)) + BN_EPS).sqrt()


def _gblock(n, p, x, cond):
    def cbn(t, i):
        g, b = cond @ n.sn(p + "bn%d.gain" % i).t(), cond @ n.sn(p + "bn%d.bias" % i).t()
        return ((1 + g)[:, None, None] * _bn(t) + b[:, None, None]).relu()
    h = _conv(_up2(cbn(x, 1)), n.sn(p + "conv1.w")) + n.w[p + "conv1.b"]
    y = _conv(cbn(h, 2), n.sn(p + "conv2.w")) + n.w[p + "conv2.b"]
    return y + _up2(_conv(x, n.sn(p + "sc.w")) + n.w[p + "sc.b"])


def _dblock(n, p, x, pre, down, lsc):
    h = _conv(x.relu() if pre else x, n.sn(p + "conv1.w")) + n.w[p + "conv1.b"]
    y = _conv(h.relu(), n.sn(p + "conv2.w")) + n.w[p + "conv2.b"]
    s = x
    if down:
        y, s = _win(y).mean((2, 4)), _win(s).mean((2, 4))
    return y + (_conv(s, n.sn(p + "sc.w")) + n.w[p + "sc.b"] if lsc else s)


def _attn(n, p, x):
    B, H, W, C = x.shape
    t = (x @ n.sn(p + "theta")[:, 0, 0].t()).reshape(B, H * W, -1)
    k = _win(x @ n.sn(p + "phi")[:, 0, 0].t()).amax((2, 4)).reshape(B, H * W // 4, -1)
    g = _win(x @ n.sn(p + "g")[:, 0, 0].t()).amax((2, 4)).reshape(B, H * W // 4, -1)
    o = torch.softmax(torch.bmm(t, k.transpose(1, 2).contiguous()), -1) @ g
    return x + n.w[p + "gamma"] * (o.reshape(B, H, W, -1) @ n.sn(p + "o")[:, 0, 0].t())


def _gout(n, x):
    a = (n.w["out_bn.gain"] * _bn(x) + n.w["out_bn.bias"]).relu()
    return torch.tanh(_conv(a, n.sn("out_conv.w")) + n.w["out_conv.b"])


def _padded(t):
    return torch.nn.functional.pad(t, (0, cpad(t.shape[-1]) - t.shape[-1]))


def _g_net(arch, P, u, z, y):
    _, ch, gm, _, _, attn, _, dz, _ = ARCHS[arch]
    n = _Net(_net_shapes(arch, 0), P, u)
    zs = z.double().split(dz // len(gm), 1)
    h = (zs[0] @ n.sn("linear.w").t() + n.w["linear.b"]).reshape(-1, 4, 4, gm[0] * ch)
    for i in range(len(gm) - 1):
        h = _gblock(n, "g%d." % i, h, torch.cat([n.w["shared"][y.long()], zs[i + 1]], 1))
        if 8 << i == attn:
            h = _attn(n, "attn.", h)
    return _gout(n, h), n.u


def _d_net(arch, P, u, x, y):
    n = _Net(_net_shapes(arch, 1), P, u)
    h = x.double()
    for j, s in enumerate(_d_specs(arch)):
        h = _dblock(n, "d%d." % j, h, s["pre"], s["down"], s["lsc"])
        if s["attn"]:
            h = _attn(n, "attn.", h)
    h = h.relu().sum((1, 2))
    return (h * (n.sn("head.w") + n.sn("embed")[y.long()])).sum(1) + n.w["head.b"], n.u


def exact(case, seed):
    k = case["kind"]
    if k == "train":
        return None   # minutes of float64 products
    d = _inputs(case, seed)
    if k == "sn":
        _, u, v, sigma = _sn(d["W"].double(), d["u"].double(), case["iters"])
        return {"u": u, "v": v, "sigma": sigma.reshape(1)}
    if k == "g_sample":
        with torch.no_grad():
            img, u = _g_net(case["arch"], d["GP"], d["Gu"], d["z"], d["y"])
        return {"img": img, "u": u}
    if k == "d_step":
        # the updated weights have no float64 value to hold to: the first Adam step with beta1 = 0
        # is lr * sign(gradient), whatever the gradient's size
        with torch.no_grad():
            out, u = _d_net(case["arch"], d["DP"], d["Du"], torch.cat([d["xr"], d["xf"]]), torch.cat([d["yr"], d["yf"]]))
            B = case["B"]
            loss = (1 - out[:B]).relu().mean() + (1 + out[B:]).relu().mean()
        return {"loss": loss.item(), "params": None, "u": u}
    cin = case["C"] if k in ("attn", "gout") else case["cin"]
    x = d["x"][..., :cin].double().requires_grad_(True)
    if k == "gblock":
        n = _Net(_gblock_shapes(cin, case["cout"], case["dc"]), d["P"], d["u"])
        cond = d["cond"].double().requires_grad_(True)
        y, dy = _gblock(n, "", x, cond), d["dy"][..., :case["cout"]]
    elif k == "dblock":
        n = _Net(_dblock_shapes(cin, case["cout"], case["lsc"]), d["P"], d["u"])
        y, dy = _dblock(n, "", x, case["pre"], case["down"], case["lsc"]), d["dy"][..., :case["cout"]]
    elif k == "attn":
        n = _Net(_attn_shapes(cin), d["P"], d["u"])
        y, dy = _attn(n, "", x), d["dy"][..., :cin]
    else:
        n = _Net(_gout_shapes(cin), d["P"], d["u"])
        y, dy = _gout(n, x), d["dimg"]
    y.backward(dy.double())
    r = {"y" if k != "gout" else "img": _padded(y.detach()) if k != "gout" else y.detach(), "u": n.u,
         "dx": _padded(x.grad), "grads": n.flat.grad}
    if k == "gblock":
        r["dcond"] = cond.grad
    return r
