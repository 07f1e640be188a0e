"""Parity of the launch forms that small problems take: convolutions whose K
loop is split over blocks, weight gradients planned in whole rounds of
blocks, the conditional-BN linear maps and the sub-pixel fold.  Sizes at the edges of their tiles: partial pixel
and channel tiles, uneven last splits, every gather and epilogue of a split
conv.  Same oracle and bars as the block tests."""
import pytest

from paragan_2411_03999_amd import lib

from . import parity
from .test_gpu_blocks import run_dblock, run_gblock

pytestmark = pytest.mark.gpu


def launched(part):
    return sorted(n for n in parity.SEEN if part in n)


# (kind, shape, the kernel instances that must have run split)
SPLIT = [
    # halo kernels at 16-wide rows: 192 channels (6 chunks) and 96
    ("g", dict(B=1, H=16, W=16, cin=192, cout=192, dc=20), ["k_conv_halo<192x128,false>/split",
                                                            "k_conv_halo<192x128,G_SUB,false>/split"]),
    ("g", dict(B=2, H=16, W=16, cin=96, cout=96, dc=20), ["k_conv_halo<96x512,false>/split"]),
    # ring kernels: 128-wide tiles with a partial channel tile (160 channels), ragged pixels
    ("g", dict(B=3, H=5, W=7, cin=136, cout=160, dc=20), ["k_conv_fwd<128x128,G_DIRECT,false>/split",
                                                          "k_conv_fwd<128x128,G_S2,false>/split"]),
    ("d", dict(B=3, H=10, W=6, cin=200, cout=136, preact=True, down=True, lsc=True),
     ["k_conv_fwd<128x128,G_S2,true>/split", "k_conv_fwd<128x128,G_DIRECT,true>/split"]),
    # identity skip, bf16 residual, one pixel past a 256-pixel tile
    ("d", dict(B=1, H=1, W=257, cin=256, cout=256, preact=True, down=False, lsc=False),
     ["k_conv_fwd<128x256,G_DIRECT,true>/split"]),
]


@pytest.mark.parametrize("kind,shape,names", SPLIT)
def test_split_conv(kind, shape, names):
    run = run_gblock if kind == "g" else run_dblock
    parity.SEEN.difference_update(names)
    run(dtype=lib.BF16, seed=700, weights="gaussian", **shape)
    for n in names:
        assert n in parity.SEEN, (n, launched("split"))


# Weight-gradient plans: row-tap tiles on a two-row image, a pixel range that
# ends inside a stage and inside the last split, fewer pixels than one split
@pytest.mark.parametrize("kind,shape", [
    ("d", dict(B=1, H=2, W=32, cin=64, cout=256, preact=True, down=False, lsc=True)),
    ("d", dict(B=2, H=33, W=31, cin=96, cout=192, preact=True, down=False, lsc=True)),
    ("g", dict(B=1, H=3, W=3, cin=64, cout=384, dc=20)),
])
def test_wgrad_plan(kind, shape):
    run = run_gblock if kind == "g" else run_dblock
    run(dtype=lib.BF16, seed=710, weights="gaussian", **shape)


# Conditional-BN maps: conditioning wider than one staged chunk and not a
# multiple of four, samples and channels past one tile, split sums over the
# channels; the sub-pixel fold with its splits over waves (960 source pixels)
@pytest.mark.parametrize("shape", [
    dict(B=17, H=2, W=3, cin=264, cout=40, dc=171),
    dict(B=33, H=1, W=2, cin=32, cout=72, dc=3),
    dict(B=3, H=16, W=20, cin=32, cout=40, dc=148),
])
@pytest.mark.parametrize("dtype", [lib.BF16, lib.F32])
def test_cbn_maps(shape, dtype):
    run_gblock(dtype=dtype, seed=720, weights="gaussian", **shape)
