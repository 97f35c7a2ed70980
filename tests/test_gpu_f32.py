"""float32 convs and FC layers on the matrix-core kernel, at the sizes where
its choices change: one or two fragments per wave, each split of the depth
over the waves of a workgroup, depths that end inside a 16-deep chunk, 8
input channels (a chunk of two taps), ragged rows and columns.

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
    (64, 64, 3, 1, 1, 56, 6),     # and not split
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
