"""Input pack, output export, pooling and routing kernels at the edges of
their tiles: channel counts around 8 and 64, maps of one pixel, around 64
pixels and of several workgroups, ragged frame counts over two models. Pack,
upsample, max pool, concat and export move values without arithmetic, so
bf16-representable inputs come back exactly; the average pool sums in
float32 (a bf16 rounding, or (pixels + 2) * 2^-24 of the mean magnitude)."""

import numpy as np
import pytest
import torch

from harness import GpuWorkload, compare, oracle_outputs
from test_gpu_layers import L
from workloads.configs import ModelSpec, Workload

pytestmark = pytest.mark.gpu

MAPS = [(1, 1), (7, 7), (8, 8), (5, 13), (33, 40)]
CHANNELS = [3, 8, 9, 24, 64, 72, 200]


def run(layers, chw, frames, dtype):
    ms = [ModelSpec(f"m{i}", "custom", layers, n, chw) for i, n in enumerate(frames)]
    wl = Workload("layout", 23, dtype, ms, [], "normal")
    fr = [wl.frames(i) for i in range(len(ms))]
    g = GpuWorkload(wl)
    try:
        return fr, g.run(fr)
    finally:
        g.close()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("hw", MAPS, ids=lambda m: f"{m[0]}x{m[1]}")
@pytest.mark.parametrize("c", CHANNELS)
def test_moved_values_are_exact(c, hw, dtype):
    lay = [L("u", "upsample", -1, cin=c, cout=c, out=True),
           L("p", "maxpool", 0, cin=c, cout=c, kh=3, kw=3, stride=2, pad=1, out=True),
           L("q", "maxpool", 0, cin=c, cout=c, kh=2, kw=2, stride=2, out=True),
           L("r", "maxpool", 0, cin=c, cout=c, kh=2, kw=2, stride=1, pad=1, out=True)]
    if c % 8 == 0:
        lay.append(L("k", "concat", 2, src1=1, cin=c, cout=2 * c, out=True))
    fr, got = run(lay, (c,) + hw, [3, 1], dtype)
    for x, outs in zip(fr, got):
        up = x.repeat(2, 2).repeat(2, 3)
        assert np.array_equal(outs[0], up)

        def pool(k, s, p):
            z = np.pad(up, ((0, 0), (0, 0), (p, p), (p, p)), constant_values=-np.inf)
            v = np.lib.stride_tricks.sliding_window_view(z, (k, k), axis=(2, 3))
            return v[:, :, ::s, ::s].max((4, 5))

        assert np.array_equal(outs[1], pool(3, 2, 1))
        assert np.array_equal(outs[2], x)
        assert np.array_equal(outs[3], pool(2, 1, 1))
        if c % 8 == 0:
            assert np.array_equal(outs[4], np.concatenate([outs[2], outs[1]], 1))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("c,hw", [(8, (1, 1)), (32, (16, 16)), (40, (7, 7)), (136, (3, 50)), (2048, (7, 7))])
def test_average_pool(c, hw, dtype):
    lay = [L("a", "avgpool", -1, cin=c, cout=c, out=True)]
    fr, got = run(lay, (c,) + hw, [2, 5], dtype)
    for x, outs in zip(fr, got):
        ref = x.astype(np.float64).mean((2, 3), keepdims=True)
        mag = np.abs(x.astype(np.float64)).mean((2, 3), keepdims=True)
        bound = (hw[0] * hw[1] + 2) * 2.0 ** -24 * mag
        if dtype == "bf16":
            bound = bound + 2.0 ** -8 * (np.abs(ref) + bound)
        assert np.all(np.abs(outs[0] - ref) <= bound)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("c,hw", [(8, (1, 1)), (24, (1, 3)), (32, (16, 16)), (32, (17, 15)), (32, (37, 29)), (40, (7, 7)),
                                  (136, (8, 8)), (136, (5, 13)), (136, (3, 50)), (2048, (7, 7))])
def test_average_pool_order_of_sums(c, hw, dtype):
    """Group g of 4 adds pixels g, g + 4, ... one after the other in float32,
    then the groups are added in order: the result is exact to the bit."""
    fr, got = run([L("a", "avgpool", -1, cin=c, cout=c, out=True)], (c,) + hw, [2, 5], dtype)
    n = np.float32(hw[0] * hw[1])
    for x, outs in zip(fr, got):
        px = x.reshape(x.shape[0], c, -1)
        part = [np.zeros(px.shape[:2], np.float32) for _ in range(4)]
        for p in range(px.shape[2]):
            part[p % 4] = part[p % 4] + px[:, :, p]
        ref = (((part[0] + part[1]) + part[2]) + part[3]) * (np.float32(1) / n)
        if dtype == "bf16":
            ref = torch.from_numpy(ref).bfloat16().float().numpy()
        assert np.array_equal(outs[0].reshape(ref.shape), ref)


@pytest.mark.parametrize("models", [2, 18], ids=["two", "more-than-a-launch-holds"])
def test_pooling_and_routing_of_several_models_share_launches(models):
    """The same pooling, routing and output layers behind one launch run as
    one launch per kind, with the results of separate launches."""
    from paper_2201_07705_amd import gemel as G
    c, hw = 16, 10
    lay = [L("p", "maxpool", -1, cin=c, cout=c, kh=2, kw=2, stride=2, out=True),
           L("u", "upsample", 0, cin=c, cout=c),
           L("k", "concat", 1, src1=-1, cin=c, cout=2 * c, out=True),
           L("a", "avgpool", 2, cin=2 * c, cout=2 * c, out=True)]
    ms = [ModelSpec(f"m{i}", "custom", lay, 1 + i % 3, (c, hw, hw)) for i in range(models)]
    wl = Workload("share", 29, "bf16", ms, [], "normal")
    fr = [wl.frames(i) for i in range(models)]
    outs, launches = [], []
    for group in (1, 0):
        g = GpuWorkload(wl)
        try:
            g.ctx.set_option(G.OPT_GROUP_UNMERGED, group)
            outs.append(g.run(fr, repeat=3))
            launches.append(g.ctx.query(G.Q_LAUNCHES))
        finally:
            g.close()
    for a, b in zip(*outs):
        for x, y in zip(a, b):
            assert np.array_equal(x, y)
    packs = (models + 15) // 16
    assert launches[1] == packs + 7 * models
    assert launches[0] == packs + 7 * packs


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_max_pool_of_nan_and_infinities(dtype):
    """Out-of-range taps count as -Inf and NaN never wins: windows of -Inf or
    NaN alone give -Inf, at the border and inside, at each window size."""
    c, h, w = 8, 9, 7
    lay = [L(f"p{k}", "maxpool", -1, cin=c, cout=c, kh=k, kw=k, stride=s, pad=p, out=True)
           for k, s, p in ((2, 1, 1), (2, 2, 0), (3, 2, 1), (3, 1, 1), (5, 2, 2))]
    wl = Workload("nan", 19, dtype, [ModelSpec("m", "custom", lay, 2, (c, h, w))], [], "normal")
    x = wl.frames(0)
    x[:, 0] = -np.inf
    x[:, 1, 2:7, 1:6] = np.nan
    x[:, 2] = np.nan
    x[:, 3, ::2] = -np.inf
    x[:, 3, 1, 1] = np.nan
    x[:, 4, 3, 3] = np.inf
    g = GpuWorkload(wl)
    try:
        outs = g.run([x])[0]
    finally:
        g.close()
    for l, o in zip(lay, outs):
        k, p = l["kh"], l["pad"]
        z = np.pad(np.where(np.isnan(x), -np.inf, x), ((0, 0), (0, 0), (p, p), (p, p)), constant_values=-np.inf)
        v = np.lib.stride_tricks.sliding_window_view(z, (k, k), axis=(2, 3))
        assert np.array_equal(o, v[:, :, ::l["stride"], ::l["stride"]].max((4, 5)))


def cycle_workload(dtype="bf16"):
    """Two models that share two convs and run them in opposite order, with a
    pool behind the same one in both: launches that take both models' convs
    would wait for each other."""
    def conv(name, src, **kw):
        return L(name, "conv", src, cin=16, cout=16, kh=3, kw=3, pad=1, bias=True, act="relu", **kw)

    def pool(src, **kw):
        return L("p", "maxpool", src, cin=16, cout=16, kh=3, kw=3, stride=1, pad=1, **kw)

    a = [conv("x", -1), pool(0), conv("y", 1), pool(2, out=True)]
    b = [conv("y", -1), conv("x", 0), pool(1), pool(2, out=True)]
    ms = [ModelSpec("a", "custom", a, 2, (16, 12, 12)), ModelSpec("b", "custom", b, 3, (16, 12, 12))]
    return Workload("cycle", 43, dtype, ms, [[(0, 0), (1, 1)], [(0, 2), (1, 0)]], "normal")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_pool_behind_convs_shared_in_opposite_order(dtype):
    wl = cycle_workload(dtype)
    params = [wl.params(i) for i in range(2)]
    fr = [wl.frames(i) for i in range(2)]
    g = GpuWorkload(wl, params)
    try:
        got = g.run(fr, repeat=3)
    finally:
        g.close()
    compare(wl, got, oracle_outputs(wl, params, fr), tag=f"cycle-{dtype}", check_argmax=False)


def _large(layers, chw):
    """One frame of bf16 values on the device and its outputs."""
    import paper_2201_07705_amd as P
    print("large map", chw, flush=True)
    ctx = P.Context(0, "bf16")
    try:
        i = ctx.register_model(layers, [None] * len(layers), chw)
        x = torch.randint(-127, 128, (1,) + chw, dtype=torch.int8, device="cuda",
                          generator=torch.Generator("cuda").manual_seed(5)).float()
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        outs = ctx.infer([i], [x], stream=s)[0]
        s.synchronize()
        return x, outs
    finally:
        ctx.close()


@pytest.mark.parametrize("times", [1, 2])
def test_maps_of_2_30_pixels_and_2_31_items(times):
    """The largest frames upsampled: a map of 2^30 pixels pooled, averaged and
    exported, and one of 2^31 8-channel items exported."""
    torch.cuda.empty_cache()
    h, w = (16384, 16384) if times == 1 else (8192, 16384)
    lay = [L("u", "upsample", -1, cin=1, cout=1, out=True)]
    if times == 1:
        lay += [L("p", "maxpool", 0, cin=1, cout=1, kh=2, kw=2, stride=2, out=True),
                L("a", "avgpool", 0, cin=1, cout=1, out=True)]
    else:
        lay = [L("u0", "upsample", -1, cin=1, cout=1), L("u", "upsample", 0, cin=1, cout=1, out=True)]
    x, outs = _large(lay, (1, h, w))
    k = 2 * times
    up = outs[0].view(h, k, w, k)
    for dy in range(k):
        for dx in range(k):
            assert torch.equal(up[:, dy, :, dx], x[0, 0])
    if times == 1:
        assert torch.equal(outs[1], x)
        # symmetric whole numbers: sums of 2^28 of them wander by about 2^20,
        # well within the 2^24 up to which float32 sums are exact
        mean = x.sum(dtype=torch.float64) / 2 ** 28
        assert float(outs[2]) == float(mean.float().bfloat16())
    del x, outs, up
    torch.cuda.empty_cache()
