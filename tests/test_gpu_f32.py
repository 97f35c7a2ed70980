"""float32 convs and FC layers on the matrix-core kernel, at the sizes where
its choices change: one or two fragments per wave, the depth split over 1 to
16 waves of a workgroup (by the launch's rows, without a change of the
result's bits), depths that end inside a 16-deep chunk, 8 input channels (a
chunk of two taps), ragged rows and columns.

Bound: a float32 sum of K products in any order is within
(K + 2) * 2^-24 * sum |w| |x| of the exact one (each of the K products and
sums rounds once), plus one rounding of the scale and shift."""

import numpy as np
import pytest

from harness import GpuWorkload, oracle_outputs
from test_gpu_layers import L, conv
from workloads.configs import ModelSpec, Workload

pytestmark = pytest.mark.gpu

CASES = [
    # cin, cout, k, stride, pad, hw, frames
    (3, 16, 3, 1, 1, 32, 1),      # 2x1 fragments, chunks of two taps, K 72
    (16, 32, 3, 2, 1, 17, 1),     # odd map, stride 2
    (32, 40, 3, 1, 1, 16, 1),     # N ends inside a fragment pair
    (8, 8, 1, 1, 0, 5, 1),        # one chunk, half of it beyond K
    (24, 24, 1, 1, 0, 3, 1),      # M 9: 1x2 fragments; K 24
    (64, 64, 3, 1, 1, 56, 1),     # depth split over several waves
    (64, 64, 3, 1, 1, 56, 6),     # over two waves, 2x2 fragments
    (512, 512, 3, 1, 1, 7, 2),    # deepest split
    (256, 128, 1, 2, 0, 14, 3),
    (3, 64, 7, 2, 3, 61, 2),
]


def exact(models, in_chw, frames, tweak=None):
    ms = [ModelSpec(f"m{i}", "custom", lay, n, in_chw) for i, (lay, n) in enumerate(zip(models, frames))]
    wl = Workload("f32", 11, "f32", ms, [], "normal")
    params = [wl.params(i) for i in range(len(ms))]
    if tweak:
        tweak(params)
    fr = [wl.frames(i) for i in range(len(ms))]
    g = GpuWorkload(wl, params)
    try:
        got = g.run(fr)
    finally:
        g.close()
    return wl, params, fr, got


def check(wl, params, fr, got, K):
    ref = oracle_outputs(wl, params, fr)
    mag = [[{**p, "w": np.abs(p["w"]), "b": None if p["b"] is None else np.abs(p["b"])} if p else None for p in ps]
           for ps in params]
    top = oracle_outputs(wl, mag, [np.abs(f) for f in fr])
    for g, r, t in zip(got, ref, top):
        for a, b, m in zip(g, r, t):
            # the oracle returns float32: half an ulp of its own
            assert np.all(np.abs(a.astype(np.float64) - b) <= (K + 4) * 2.0 ** -24 * m + 1e-30)


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_conv_f32_bound(case):
    cin, cout, k, s, p, hw, n = case
    lay = [conv("c", -1, cin, cout, k, s, p, bias=True, out=True)]
    check(*exact([lay], (cin, hw, hw), [n]), cin * k * k)


@pytest.mark.parametrize("cin,cout,n", [(32, 10, 1), (512, 1000, 2), (2048, 80, 16), (4096, 64, 17), (40, 24, 70)])
def test_fc_f32_bound(cin, cout, n):
    lay = [L("f", "fc", -1, cin=cin, cout=cout, bias=True, out=True)]
    check(*exact([lay], (cin, 1, 1), [n]), cin)


def test_infinite_weight_outside_the_image_is_skipped():
    """An infinite weight at a corner tap reaches only the outputs whose tap
    lies inside the image; the others stay finite and exact."""
    def tweak(params):
        params[0][0]["w"][:, :, 0, 0] = np.inf
    lay = [conv("c", -1, 8, 16, 3, 1, 1, bias=True, out=True)]
    wl, params, fr, got = exact([lay], (8, 9, 9), [1], tweak)
    a = got[0][0]
    assert np.isfinite(a[:, :, 0, :]).all() and np.isfinite(a[:, :, :, 0]).all()
    assert not np.isfinite(a[:, :, 1:, 1:]).any()


# input channels and window: 18, 7, 21, 36, 4 and 3 chunks of 32 in 8, 2, 8, 16, 2 parts and one. With
# 2x2 fragments (from 2 frames of 55 x 55 on, whose rows end inside a workgroup's tiles) over 4, 2, 4, 4,
# 2 waves and one, over 8 where there are 8 parts and 2 frames; with 1x2 (one frame) over up to 8
DEPTHS = [(64, 3), (24, 3), (72, 3), (128, 3), (128, 1), (96, 1)]


@pytest.mark.parametrize("n", [12, 6, 4, 2, 1])
@pytest.mark.parametrize("cin,k", DEPTHS)
def test_conv_f32_bound_at_each_split(cin, k, n):
    lay = [conv("c", -1, cin, 64, k, 1, k // 2, bias=True, out=True)]
    check(*exact([lay], (cin, 55, 55), [n]), cin * k * k)


@pytest.mark.parametrize("cin,k", DEPTHS)
def test_f32_bits_do_not_depend_on_the_round(cin, k):
    """Twelve frames in one round, fewer at a time, and as two merged models:
    the same bits for every frame, through an internal layer with a residual,
    a strided one, an average pool and an FC layer."""
    lay = [conv("a", -1, cin, 64, k, 1, k // 2, bn=True, act="relu"),
           conv("b", 0, 64, 64, 3, 1, 1, bn=True, act="relu", res=0),
           conv("d", 1, 64, 128, 3, 2, 1, bn=True, act="leaky", out=True),
           L("p", "avgpool", 2, cin=128, cout=128),
           L("f", "fc", 3, cin=128, cout=40, bias=True, out=True)]
    ms = [ModelSpec(f"m{i}", "custom", lay, n, (cin, 55, 55)) for i, n in enumerate((5, 7))]
    wl = Workload("f32", 17, "f32", ms, [[(0, l), (1, l)] for l in range(5) if l != 3], "normal")
    params = [wl.params(0)] * 2
    fr = [wl.frames(i) for i in range(2)]
    g = GpuWorkload(wl, params)
    try:
        merged = g.run(fr)
        alone = [g.run(fr, order=[i])[i] for i in range(2)]
        x = np.concatenate(fr)
        whole = g.run([x, x], order=[0])[0]
        parts = [[np.concatenate(o) for o in zip(*(g.run([x[i:i + n]] * 2, order=[0])[0] for i in range(0, 12, n)))]
                 for n in (1, 2, 4, 6)]
    finally:
        g.close()
    for o, w in enumerate(whole):
        assert np.array_equal(np.concatenate([m[o] for m in merged]), w)
        assert np.array_equal(np.concatenate([m[o] for m in alone]), w)
        for p in parts:
            assert np.array_equal(p[o], w)
