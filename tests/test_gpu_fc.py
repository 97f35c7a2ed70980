"""bf16 FC layers of up to 64 frames at the edges of the streaming kernel's
choices: depths that end inside a ring step, one step, fewer steps than ring
buffers, many splits; neurons that end inside a wave or a workgroup; every
frame padding; two models (grouped) with ragged frame counts.

Inputs and weights are bf16 values, so every product is exact in float32; a
float32 sum of K of them in any order is within (K + 2) * 2^-24 * sum |w| |x|
of the exact one, plus the rounding of the bias addition."""

import numpy as np
import pytest

from harness import GpuWorkload, oracle_outputs
from test_gpu_layers import L
from workloads.configs import ModelSpec, Workload

pytestmark = pytest.mark.gpu

SIZES = [(8, 10), (120, 16), (128, 64), (264, 72), (1000, 1000), (4096, 24), (6272, 136)]
FRAMES = [(1,), (2,), (3, 1), (8,), (9,), (5, 16), (17,), (33,), (64,), (20, 40)]


def check(k, n, frames):
    lay = [L("f", "fc", -1, cin=k, cout=n, bias=True, out=True)]
    ms = [ModelSpec(f"m{i}", "custom", lay, f, (k, 1, 1)) for i, f in enumerate(frames)]
    wl = Workload("fc", 31, "bf16", ms, [], "normal")
    params = [wl.params(i) for i in range(len(ms))]
    fr = [wl.frames(i) for i in range(len(ms))]
    g = GpuWorkload(wl, params)
    try:
        got = g.run(fr, repeat=2)
    finally:
        g.close()
    ref = oracle_outputs(wl, params, fr)
    mag = [[{**p, "w": np.abs(p["w"]), "b": np.abs(p["b"])} for p in ps] for ps in params]
    top = oracle_outputs(wl, mag, [np.abs(f) for f in fr])
    for a, b, m in zip(got, ref, top):
        assert np.all(np.abs(a[0].astype(np.float64) - b[0]) <= (k + 4) * 2.0 ** -24 * m[0])


@pytest.mark.parametrize("frames", FRAMES, ids=lambda f: "-".join(map(str, f)))
@pytest.mark.parametrize("k,n", SIZES)
def test_fc_bf16_bound(k, n, frames):
    check(k, n, frames)


# the two forms of the input slice up to 16 frames: 14336 elements and the next run
@pytest.mark.parametrize("k,n,frames", [(1792, 40, (8,)), (1800, 40, (8,)), (2040, 72, (7, 2)), (896, 24, (13,)), (904, 24, (16,))])
def test_fc_input_slice_forms(k, n, frames):
    check(k, n, frames)
