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
from test_gpu_layers import DMA_TILES, TILES, conv
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
