"""The order of the sums that decisions hang on.

A ReLU (max-pool, hinge) input within rounding of zero turns with the last
bit of the sums before it, and one turned element moves a small block's
gradients by 1e-3 and a training iteration's later losses and SN vectors by
several percent.  So a rearrangement that is meant to save time only must
leave those sums' bits alone:
* an fp32 block's convolutions add an output's products one by one, tap by
  tap and channel by channel, whichever kernel its size selects, and its
  batch statistics have one chunking;
* in a network, G's activations, D's activations and D's gradients follow
  fixed rules on the sizes, not the launch plans.
The pins are digests of whole outputs at seeded inputs: a change here is a
change of the order of operations (or of a rule above), to be made knowingly
and with a new pin."""
import hashlib

import numpy as np
import pytest

from oracle import biggan as O
from oracle import blocks as OB
from paragan_2411_03999_amd import lib
from paragan_2411_03999_amd.synth import Stream, init_params, init_u

from .parity import SEEN, context, harvest, need_gpu
from .test_gpu_train_step import hparams, make_nets, run_train_step, step_inputs

pytestmark = pytest.mark.gpu


def digest(*tensors):
    h = hashlib.sha256()
    for t in tensors:
        h.update(np.ascontiguousarray(t.cpu().numpy()).tobytes())
    return h.hexdigest()[:16]


# ------------------------------------------------------------- fp32 blocks
def f32_dblock(torch, ctx, x, dy, p, u, cin, cout, down):
    """y and dx of the fp32 D block on x."""
    B, H, W, _ = x.shape
    d = lib.DBlockDesc(B, H, W, cin, cout, 1, int(down), 1, lib.F32, 1, 1e-12)
    ents, npar, nu = lib.paragan_dblock_layout(d)
    P, U = lib.flat_from_named(ents, npar, p), lib.u_from_named(ents, nu, u)
    saved, ws = (lib.workspace(n) for n in lib.paragan_dblock_sizes(d))
    Y, DX, G = torch.zeros_like(dy), torch.zeros_like(x), torch.zeros(npar, device="cuda")
    lib.paragan_dblock_fwd(ctx, d, P, U, x, Y, saved, ws)
    lib.paragan_dblock_bwd(ctx, d, P, x, saved, dy, DX, G, ws)
    torch.cuda.synchronize()
    return Y, DX


# the small-grid kernel (below 384 tiles of 64 x 64) against the tiled one on
# the same images: direct and pooled outputs, ragged channels
@pytest.mark.parametrize("down", [False, True])
def test_f32_image_is_the_same_bits_at_any_batch(down):
    torch = need_gpu()
    H = W = 16
    cin, cout, few, many = 40, 72, 2, 1024
    s = Stream(811)
    shapes = OB.dblock_param_shapes(cin, cout, True)
    p, u = init_params(shapes, s, weights="gaussian"), init_u(shapes, ["conv1.w", "conv2.w", "sc.w"], s)
    x = lib.to_device_nhwc(s.normal((few, H, W, cin)), lib.F32)
    k = 2 if down else 1
    dy = lib.to_device_nhwc(s.normal((few, H // k, W // k, cout)), lib.F32)
    seen = set(SEEN)
    out, names = [], []
    for n in (few, many):
        SEEN.clear()
        ctx = context()
        out.append(f32_dblock(torch, ctx, x.repeat(n // few, 1, 1, 1), dy.repeat(n // few, 1, 1, 1), p, u, cin, cout,
                              down))
        harvest(ctx)
        names.append(set(SEEN))
        seen |= SEEN
    SEEN.update(seen)
    assert any(m.startswith("k_conv_f32r") for m in names[0]) and not any("f32mfma" in m and "conv" in m for m in names[0])
    assert sum(m.startswith("k_conv_f32mfma") for m in names[1]) >= 2, sorted(names[1])
    for a, b in zip(*out):
        assert torch.equal(a, b[:few])
        assert torch.equal(a, b[-few:])


# (B, H, W, cin, cout, dc): digest of y
F32_PINS = {
    (4, 8, 8, 64, 64, 128): "590800dddcacf6e7",
    (8, 14, 11, 70, 50, 100): "1d7231f52a909a13",
}


@pytest.mark.parametrize("shape", list(F32_PINS))
def test_f32_gblock_forward_bits(shape):
    torch = need_gpu()
    B, H, W, cin, cout, dc = shape
    s = Stream(812)
    shapes = OB.gblock_param_shapes(cin, cout, dc)
    p, u = init_params(shapes, s, weights="gaussian"), init_u(shapes, OB.GBLOCK_SN, s)
    d = lib.GBlockDesc(B, H, W, cin, cout, dc, lib.F32, 1, 1e-5, 1e-12)
    ents, npar, nu = lib.paragan_gblock_layout(d)
    P, U = lib.flat_from_named(ents, npar, p), lib.u_from_named(ents, nu, u)
    X = lib.to_device_nhwc(s.normal((B, H, W, cin)), lib.F32)
    COND = torch.from_numpy(s.normal((B, dc)).astype(np.float32)).cuda()
    Y = lib.empty_nhwc(B, 2 * H, 2 * W, cout, lib.F32)
    saved, ws = (lib.workspace(n) for n in lib.paragan_gblock_sizes(d))
    ctx = context()
    lib.paragan_gblock_fwd(ctx, d, P, U, X, COND, Y, saved, ws)
    torch.cuda.synchronize()
    harvest(ctx)
    assert digest(Y) == F32_PINS[shape]


# ---------------------------------------------------------------- networks
# (arch, B, n_D): digests of a sample, and of an iteration's losses, D's
# parameters and both networks' SN vectors
NET_PINS = {
    ("biggan128", 8, 2): ("c9ac48b712c3b841", "6f449da94aab6cb1"),
    ("biggan512", 2, 1): ("cb63291edb0b7d8a", "770ba2ccecea7362"),
}


@pytest.mark.parametrize("key", list(NET_PINS))
def test_network_bits(key):
    torch = need_gpu()
    arch, B, n_D = key
    a = {"biggan128": O.biggan128, "biggan512": O.biggan512}[arch]()
    d, s, _, _, G, D = make_nets(torch, a, B, 813, hparams())
    inp, keep = step_inputs(torch, s, a, B, n_D)
    ctx = context()
    ws = lib.workspace(lib.paragan_train_step_ws_size(d))
    img = torch.empty((B, a.img, a.img, 3), dtype=torch.float32, device="cuda")
    ctx.check(lib.paragan_g_sample(ctx, d, G.clone(torch).state, keep[2 * n_D], keep[3 * n_D], img, ws))
    torch.cuda.synchronize()
    sample = digest(img)
    losses = torch.tensor(run_train_step(torch, d, G, D, inp, n_D, ws, ctx))
    harvest(ctx)
    got = (sample, digest(losses, D.P, D.U, G.U))
    print(key, got, flush=True)
    assert got == NET_PINS[key]
