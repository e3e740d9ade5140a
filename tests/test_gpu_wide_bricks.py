"""Bricks on both sides of the 8 MiB a slice up to which corner rows are read
by 32-bit offsets (24-bit products); above it every walk takes 64-bit
addresses.  The far corner of thin bricks, so that the largest offsets are
read: the direct march against the staged one bit for bit and against the
oracle, gradients and shadowed ray-queue frames against the oracle."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_adjoint import _gpu_grads, _oracle_grads, dp  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BG = (0.1, 0.2, 0.3, 1.0)
# dims, storage: stored slices of 2048 x 1022 float32 (8,372,224 bytes), 2048 x 1026 (8,404,992),
# 2048 x 2047 float16 (8,384,512), 2048 x 2048 (8,388,608)
CASES = [((2046, 1020, 3), 0), ((2046, 1024, 3), 0), ((2041, 2045, 2), 1), ((2041, 2046, 2), 1)]
IDS = ["f32 rows", "f32 64-bit", "f16 rows", "f16 64-bit"]


def _field(dims, storage):
    f = np.random.default_rng(31).uniform(0.0, 1.0, dims[::-1]).astype(np.float32)
    return f.astype(np.float16).astype(np.float32) if storage else f      # what the bricks hold


def _corner(dims, w, h, az, el):
    lo = (dims[0] - 30, dims[1] - 24, 0)
    return synth.orbit_camera(lo, dims, w, h, az_deg=az, el_deg=el, radius_factor=1.1)


@pytest.mark.parametrize("dims,storage", CASES, ids=IDS)
def test_direct_march(dp, dims, storage):  # noqa: F811
    field = _field(dims, storage)
    print(f"wide bricks: direct {dims} storage {storage}", flush=True)
    for az, el in ((100.0, 4.0), (30.0, 25.0), (190.0, -60.0)):
        cam = _corner(dims, 47, 35, az, el)
        sc = synth.scene_from_field("wide", field, [((0, 0, 0), dims)], synth.default_tf(), cam, 0.4, 0.6)
        outs = []
        for path, config in ((dp.VR_PATH_DIRECT, None), (dp.VR_PATH_STAGED, (1, 16, 4)), (dp.VR_PATH_STAGED, (0, 16, 4))):
            r = dp.Renderer([(b.voxels, b.lo) for b in sc.bricks], sc.tf, sc.vrange, sc.opacity_scale, sc.step, 0.0,
                            storage=storage, path=path, march_config=config)
            try:
                r.set_camera(cam)
                r.reset_samples()
                img = r.render(BG)
                r.synchronize()
                outs.append((img.cpu().numpy().copy(), r.sample_counts()))
            finally:
                r.close()
        for img, counts in outs[1:]:
            assert np.array_equal(img, outs[0][0]) and np.array_equal(counts, outs[0][1])
        ref = oracle.render_scene(sc, cam, BG)[0]
        assert np.sum(outs[0][1]) > 0 and np.max(np.abs(outs[0][0] - np.asarray(ref).reshape(outs[0][0].shape))) <= 1e-5


@pytest.mark.parametrize("dims,storage", CASES, ids=IDS)
def test_gradients(dp, dims, storage):  # noqa: F811
    field = _field(dims, storage)
    print(f"wide bricks: gradients {dims} storage {storage}", flush=True)
    cams = [_corner(dims, 23, 17, 100.0, 6.0), _corner(dims, 23, 17, 30.0, 40.0)]
    targets = [np.random.default_rng(5).uniform(0, 1, (17, 23, 4)) for _ in cams]
    args = (field, [((0, 0, 0), dims)], cams, synth.default_tf(), targets, 0.8)
    _, gtf_ref, gvol_ref = _oracle_grads(*args, dt=0.4, storage=storage)
    _, gtf, gvol, _ = _gpu_grads(dp, *args, interval=64, dt=0.4, storage=storage)
    for got, ref in ((gtf, gtf_ref), (gvol, gvol_ref)):
        top = np.max(np.abs(ref))
        assert top > 0 and np.max(np.abs(got - ref)) <= 1e-4 * top


@pytest.mark.parametrize("dims,storage", CASES, ids=IDS)
def test_ray_queue_shadows(dp, dims, storage):  # noqa: F811
    field = _field(dims, storage)
    print(f"wide bricks: ray queues {dims} storage {storage}", flush=True)
    cam = _corner(dims, 31, 23, 140.0, 30.0)
    sc = synth.scene_from_field("wide", field, [((0, 0, 0), dims)], synth.default_tf(), cam, 0.5, 0.6)
    light, ambient = (0.9, 0.3, 0.15), 0.25
    r = dp.Renderer([(b.voxels, b.lo) for b in sc.bricks], sc.tf, sc.vrange, sc.opacity_scale, sc.step, 0.0,
                    storage=storage)
    try:
        r.set_camera(cam)
        assert r.rqc_plan() > 0
        got = r.render_rqc(light, ambient, BG)
        r.synchronize()
        got = got.cpu().numpy().astype(np.float64)
    finally:
        r.close()
    ref, _, _ = oracle.render_scene_shadowed(sc, light, ambient, bg=BG)
    assert np.max(np.abs(got - np.asarray(ref).reshape(got.shape))) <= 1e-5
