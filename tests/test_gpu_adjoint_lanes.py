"""Adjoint edges of several lanes per ray, against the oracle's gradients.

A ray's samples are cut into four stretches, one lane each: rays of fewer
samples than lanes and of odd counts, bricks thinner than a step, tiles that
stick out of the ROI, many samples per cell, and stretches whose transmittance
is below the smallest float.

Tolerance: 1e-4 of the largest gradient of the group, plus what rounding does
to a sample's transmittance exp2(-a'): a' = scale dt log2(e) alpha(v), v being
a float32 interpolation of values in [0, 1] (error within 2^-22), so
d a' <= scale dt log2(e) max|d alpha / dv| 2^-22.
"""
import numpy as np
import pytest

import synth
from test_gpu_adjoint import _gpu_grads, _oracle_grads, dp  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", [0, 1], ids=["f32", "f16"])
@pytest.mark.parametrize("dims,nb,size,dt,scale", [
    ((9, 7, 5), 1, (13, 11), 2.0, 3.0),        # 0 to 6 samples a ray
    ((17, 13, 11), 6, (23, 9), 1.7, 3.0),      # bricks of 1 to 9 voxels: rays of 1 to 5 samples
    ((8, 8, 1), 1, (17, 17), 0.5, 3.0),        # one voxel thick
    ((12, 10, 9), 2, (9, 9), 0.07, 3.0),       # many samples per cell
    ((16, 16, 16), 2, (16, 16), 0.5, 1500.0),  # transmittance below 2^-126 within a stretch
])
def test_ray_stretches_match_oracle(dp, dims, nb, size, dt, scale, storage):  # noqa: F811
    rng = np.random.default_rng(61)
    field = synth.tile_field(rng, dims, n_blobs=4, noise=0.05)
    boxes = synth.kd_split(dims, nb, rng)
    cams = [synth.orbit_camera((0, 0, 0), dims, *size, az_deg=az, el_deg=el, radius_factor=1.6)
            for az, el in ((25.0, 15.0), (100.0, -50.0))]
    tf = synth.default_tf()
    targets = [rng.uniform(0, 1, (size[1], size[0], 4)) for _ in cams]
    _, gtf_ref, gvol_ref = _oracle_grads(field, boxes, cams, tf, targets, scale, dt, storage)
    _, gtf, gvol, _ = _gpu_grads(dp, field, boxes, cams, tf, targets, scale, 64, dt, storage)
    slope = 255.0 * np.max(np.abs(np.diff(np.asarray(tf, dtype=np.float64)[:, 3])))
    tol = 1e-4 + scale * dt * np.log2(np.e) * slope * 2.0 ** -22
    for got, ref in ((gtf, gtf_ref), (gvol, gvol_ref)):
        top = np.max(np.abs(ref))
        assert top > 0 and np.all(np.isfinite(got))
        assert np.max(np.abs(got - ref)) <= tol * top, (np.max(np.abs(got - ref)), tol * top)
