"""The LDS-DMA conv tiles at every depth around their pipelines: fewer steps
than LDS stages, as many, one and two more, odd and even counts (a depth that
is no multiple of a tile's step goes to the register-staged tiles); rows and
channels that end inside a tile.

Inputs and weights are bf16 values, so every product is exact in float32; a
float32 sum of K of them in any order is within (K + 2) * 2^-24 * sum |w| |x|
of the exact one, plus the rounding of the bias addition."""

import numpy as np
import pytest

from harness import GpuWorkload, oracle_outputs
from test_gpu_layers import DMA_TILES, L, TILES, conv
from workloads.configs import ModelSpec, Workload

pytestmark = pytest.mark.gpu

DEPTHS = [8, 40, 64, 96, 128, 136, 192, 256, 264, 320, 384, 456]


@pytest.mark.parametrize("k", DEPTHS)
@pytest.mark.parametrize("tile", DMA_TILES, ids=lambda t: TILES[t])
def test_conv_dma_depths(tile, k):
    from paper_2201_07705_amd import gemel as G
    ms = [ModelSpec("m", "custom", [conv("c", -1, k, 72, 1, bias=True, out=True)], 3, (k, 11, 9))]
    wl = Workload("depth", 37, "bf16", ms, [], "normal")
    params = [wl.params(0)]
    fr = [wl.frames(0)]
    g = GpuWorkload(wl, params)
    try:
        g.ctx.set_option(G.OPT_CONV_TILE, tile)
        g.ctx.set_option(G.OPT_CONV_SPLITS, 1)
        got = g.run(fr, repeat=2)[0][0].astype(np.float64)
    finally:
        g.close()
    ref = oracle_outputs(wl, params, fr)[0][0]
    mag = [[{**p, "w": np.abs(p["w"]), "b": np.abs(p["b"])} for p in params[0]]]
    top = oracle_outputs(wl, mag, [np.abs(fr[0])])[0][0]
    assert np.all(np.abs(got - ref) <= (k + 4) * 2.0 ** -24 * top)


def outputs(layers, chw, frames, groups, tile, **opts):
    from paper_2201_07705_amd import gemel as G
    print("rows", chw, frames, "tile", TILES[tile], opts, flush=True)
    ms = [ModelSpec(f"m{i}", "custom", layers, n, chw) for i, n in enumerate(frames)]
    wl = Workload("rows", 41, "bf16", ms, groups, "normal")
    g = GpuWorkload(wl, [wl.params(0)] * len(ms))
    try:
        for k, v in dict(CONV_TILE=tile, CONV_SPLITS=1, **opts).items():
            g.ctx.set_option(getattr(G, "OPT_" + k), v)
        return g.run([wl.frames(i) for i in range(len(ms))])
    finally:
        g.close()


def same(a, b):
    for x, y in zip(a, b):
        for u, v in zip(x, y):
            assert np.isfinite(u).all() and np.array_equal(u, v)


# the 256 x 256 tile of depth 64 keeps its 256 rows where 224 need another turn of the 256 CUs: with 256
# channels from 57345 to 65536 rows (ragged and whole last tiles, a tile across two models); 224 rows below
# and, over two turns, above
ROWS = [((240, 239), [1]), ((256, 256), [1]), ((170, 171), [1, 1]), ((224, 256), [1]), ((250, 280), [1])]


@pytest.mark.parametrize("hw,frames", ROWS, ids=lambda v: "x".join(map(str, v)))
def test_rows_of_the_deep_256x256_tile(hw, frames):
    """Internal and NCHW outputs with a residual, bit for bit those of the
    128 x 128 tile: every tile sums the depth in the same order."""
    lay = [conv("a", -1, 64, 256, 1, bn=True, act="relu"),
           conv("b", -1, 64, 256, 3, 1, 1, bn=True, act="relu", res=0),
           L("p", "maxpool", 1, cin=256, cout=256, kh=3, kw=3, stride=3, out=True),
           conv("d", -1, 64, 256, 3, 1, 1, bn=True, act="leaky", res=0, res_mode="act_add", out=True)]
    groups = [[(m, l) for m in range(len(frames))] for l in (0, 1, 3)] if len(frames) > 1 else []
    a = outputs(lay, (64,) + hw, frames, groups, TILES.index("dma64_256x256"))
    same(a, outputs(lay, (64,) + hw, frames, groups, TILES.index("dma128x128")))


@pytest.mark.parametrize("hw,frames", [((240, 242), [1]), ((256, 256), [1]), ((170, 172), [1, 1]), ((250, 280), [1])],
                         ids=lambda v: "x".join(map(str, v)))
def test_pooled_rows_of_the_deep_256x256_tile(hw, frames):
    lay = [conv("a", -1, 64, 256, 3, 1, 1, bn=True, act="relu"),
           L("p", "maxpool", 0, cin=256, cout=256, kh=2, kw=2, stride=2, out=True)]
    groups = [[(m, 0) for m in range(len(frames))]] if len(frames) > 1 else []
    tile = TILES.index("dma64_256x256")
    a = outputs(lay, (64,) + hw, frames, groups, tile)
    same(a, outputs(lay, (64,) + hw, frames, groups, tile, FUSE_POOL=0))
    same(a, outputs(lay, (64,) + hw, frames, groups, TILES.index("dma128x128")))
