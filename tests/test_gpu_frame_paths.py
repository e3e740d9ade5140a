"""The default march of a frame, which takes the staged or the direct queue by
tiles, storage, step and voxels a pixel, against both chosen by hand: the same
bits and sample counts on either side of the rule, for cameras along each axis,
orthographic views, uneven spacing, ragged images and mixed storage."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CONFIG = {0: (1, 32, 4), 1: (0, 16, 4)}      # the staged defaults: float32 ring, float16 slab


def _ortho(dims, w, h, axis, sign):
    c = 0.5 * np.asarray(dims, dtype=np.float64)
    d = np.zeros(3)
    d[axis] = sign
    up = (0.0, 1.0, 0.0) if axis != 1 else (0.0, 0.0, 1.0)
    return dict(kind="orthographic", eye=tuple(c - 2.0 * max(dims) * d), dir=tuple(d), up=up,
                view_height=1.1 * max(dims), width=w, height=h)


@pytest.mark.parametrize("dims,nb,size,view,storage,spacing,step", [
    ((40, 36, 44), 3, (93, 71), ("orbit", 100.0, -12.0), (0,), (1.0, 1.0, 1.0), 0.5),   # few tiles, along x
    ((40, 36, 44), 3, (17, 15), ("orbit", 10.0, 70.0), (1,), (1.0, 1.0, 1.0), 1.0),     # few tiles, along y
    ((40, 36, 44), 4, (449, 447), ("orbit", 30.0, 20.0), (0, 1), (1.0, 1.0, 1.0), 0.5),  # both queues, one each way
    ((150, 140, 160), 5, (353, 349), ("orbit", 30.0, 20.0), (0,), (1.0, 1.0, 1.0), 0.25),   # float32, staged
    ((64, 48, 56), 4, (400, 401), ("ortho", 0, -1.0), (0,), (1.0, 0.5, 2.0), 0.5),
    ((64, 48, 56), 4, (300, 301), ("ortho", 2, 1.0), (1, 0), (0.5, 1.0, 1.0), 0.3),
])
def test_default_frame_equals_staged_and_direct(dims, nb, size, view, storage, spacing, step):
    import paper_2501_01628_amd as dp
    rng = np.random.default_rng(71)
    field = rng.uniform(0.0, 1.0, dims[::-1]).astype(np.float32)
    boxes = synth.kd_split(dims, nb, rng)
    world = tuple(n * s for n, s in zip(dims, spacing))
    cam = (synth.orbit_camera((0, 0, 0), world, *size, az_deg=view[1], el_deg=view[2], radius_factor=1.3)
           if view[0] == "orbit" else _ortho(world, *size, *view[1:]))
    outs = []
    for path, chosen in ((dp.VR_PATH_STAGED, False), (dp.VR_PATH_STAGED, True), (dp.VR_PATH_DIRECT, False)):
        r = dp.Renderer([], synth.default_tf(), (0.0, 1.0), 0.3, step, path=path)
        try:
            for k, (lo, hi) in enumerate(boxes):
                r.storage = storage[k % len(storage)]
                r.add_brick(synth.extract_brick(field, lo, hi), tuple(a * s for a, s in zip(lo, spacing)), spacing)
            if chosen:
                for st in (0, 1):
                    dp.vr_set_march_config(r.ctx, st, *CONFIG[st])
            r.set_camera(cam)
            r.reset_samples()
            img = r.render((0.1, 0.2, 0.3, 1.0))
            r.synchronize()
            outs.append((img.cpu().numpy().copy(), r.sample_counts()))
        finally:
            r.close()
    for img, counts in outs[1:]:
        assert np.array_equal(img, outs[0][0]) and np.array_equal(counts, outs[0][1])
    assert np.sum(outs[0][1]) > 0
