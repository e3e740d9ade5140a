"""Shadow rays of bricks whose pixels hold very different numbers of samples:
a flat brick and a long one behind a few pixels, so that those pixels hold far
more samples than the wavefronts that the mean pixel gives a tile (and take
several rounds), on few tiles and on many, against the oracle."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

BG = (0.1, 0.2, 0.3, 1.0)


@pytest.mark.parametrize("size,each", [((40, 40), 6.0), ((407, 399), 1.5)])       # 50 tiles, 2600 tiles
def test_long_brick_behind_a_flat_one(size, each):
    import paper_2501_01628_amd as dp
    rng = np.random.default_rng(29)
    dims, step = (32, 32, 90), 0.9
    field = rng.uniform(0.0, 1.0, dims[::-1]).astype(np.float32)
    boxes = [((0, 0, 0), (32, 32, 2)), ((13, 14, 2), (17, 18, 90))]
    cam = dict(kind="orthographic", eye=(16.0, 16.0, -5.0), dir=(0.02, 0.013, 1.0), up=(0.0, 1.0, 0.0),
               view_height=33.0, width=size[0], height=size[1])
    sc = synth.scene_from_field("split", field, boxes, synth.default_tf(), cam, step, 0.3)
    pix = np.stack(np.meshgrid(np.arange(size[0]), np.arange(size[1])), -1).reshape(-1, 2).astype(np.int32)
    if len(pix) > 2000:
        pix = pix[rng.choice(len(pix), 2000, replace=False)]
    light, ambient = (-0.3, 0.2, -1.0), 0.2
    r = dp.Renderer([(b.voxels, b.lo) for b in sc.bricks], sc.tf, sc.vrange, sc.opacity_scale, sc.step, 0.0)
    try:
        r.set_camera(cam)
        total = r.rqc_plan()
        rois = [roi[2] * roi[3] for roi in r.rois]
        # (a pixel of the long brick holds up to 97 samples)
        assert 0 < each * total / sum(rois) + 8 < 64
        img = r.render_rqc(light, ambient, BG)
        r.synchronize()
        img = img.cpu().numpy().astype(np.float64)
    finally:
        r.close()
    ref, _, cnt = oracle.render_scene_shadowed(sc, light, ambient, bg=BG, pixels=pix)
    assert np.max(np.abs(img[pix[:, 1], pix[:, 0]] - np.asarray(ref).reshape(-1, 4))) <= 1e-5
