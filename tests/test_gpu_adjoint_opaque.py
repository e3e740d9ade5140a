"""Table gradients of a thin haze in front of an opaque block, within one
stretch of the ray: what lies behind a sample must not enter its
transmittance, however dense it is.

Every sample falls on a voxel centre and the materials (a haze, and two dense
ones in random layers) lie on flat stretches of the table, so a' is the table's
opacity to 2^-22 whatever the interpolation does.  Relative tolerance of the
haze's colour gradients: 5 * 2^-22 ln 2 (a' of the haze, 5 in total) + 2^-24 /
0.16 (the opacity of one sample, 1 - 2^-0.2531)
+ 36 * 2^-25 (sums over 20 samples and 16 rays) + 8 * 2^-24 (products) < 4e-6;
of its opacity gradient, which subtracts the colour behind, 1e-5.
"""
import numpy as np
import pytest

import synth
from test_gpu_adjoint import _gpu_grads, _oracle_grads, dp  # noqa: F401

pytestmark = pytest.mark.gpu

HAZE, DEPTH = 20, 400


@pytest.mark.parametrize("dense", [3.7, 53.3, 307.7, 701.3, 1900.9])
def test_haze_in_front_of_an_opaque_block(dp, dense):  # noqa: F811
    rng = np.random.default_rng(67)
    scale = 1000.0
    tf = np.zeros((256, 4), dtype=np.float32)
    tf[:128] = (0.2, 0.3, 0.1, 0.2531 / (scale * np.log2(np.e)))
    tf[128:192] = (0.9, 0.7, 0.8, dense / (scale * np.log2(np.e)))
    tf[192:] = (0.9, 0.7, 0.8, 0.7321 * dense / (scale * np.log2(np.e)))
    field = np.empty((DEPTH, 4, 4), dtype=np.float32)
    field[:] = np.where(rng.random((DEPTH, 1, 1)) < 0.5, 150.5, 220.5) / 255.0
    field[:HAZE] = 50.5 / 255.0
    cam = dict(kind="orthographic", eye=(2.0, 2.0, -8.0), dir=(0.0, 0.0, 1.0), up=(0.0, 1.0, 0.0), view_height=4.0,
               width=4, height=4)
    targets = [rng.uniform(-12.0, -8.0, (4, 4, 4))]
    boxes = [((0, 0, 0), (4, 4, DEPTH))]
    args = (field, boxes, [cam], tf, targets, scale)
    _, ref, _ = _oracle_grads(*args, dt=1.0)
    _, got, _, _ = _gpu_grads(dp, *args, dt=1.0)
    assert np.all(np.isfinite(got))
    for e in (50, 51):
        rel = np.abs(got[e] - ref[e]) / np.abs(ref[e])
        print(f"dense a' {dense}: entry {e} relative error {rel}", flush=True)
        assert np.all(rel[:3] <= 4e-6) and rel[3] <= 1e-5
