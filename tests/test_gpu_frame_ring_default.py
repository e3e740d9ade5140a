"""The default frame of float32 bricks that the choice of the march leaves
staged (large bricks, more than two tiles per CU, more voxels a pixel than its
line), so that the default ring queue is the one that runs: the same bits and
sample counts as the ring by hand and as the direct march."""
import math

import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

STEP = 0.5


def _stays_staged(r, cam, boxes):
    """The rule's inputs, each brick beyond every line that would send it to
    the direct march."""
    tiles = sum(((w + 15) // 16) * ((h + 15) // 16) for _, _, w, h in r.rois)
    eye, target = np.asarray(cam["eye"]), np.asarray(cam["target"])
    f = (target - eye) / np.linalg.norm(target - eye)
    lines = []
    for lo, hi in boxes:
        size = 4.0 * np.prod([b - a + 2 for a, b in zip(lo, hi)])
        depth = float(np.dot(0.5 * (np.asarray(lo) + np.asarray(hi)) - eye, f))
        vpp = 2.0 * depth * math.tan(math.radians(cam["fovy_deg"]) / 2.0) / cam["height"]
        lines.append(vpp / min(math.sqrt(1.28 * STEP), 0.75 * (20.0e6 / size) ** 0.25))
        assert size > 8.0e6
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    return tiles > 2 * cus and min(lines) > 1.0


@pytest.mark.parametrize("az,el", [(30.0, 20.0), (100.0, -12.0), (185.0, 60.0)])
def test_default_is_the_ring(az, el):
    import paper_2501_01628_amd as dp
    dims, size = (300, 220, 200), (463, 345)
    rng = np.random.default_rng(73)
    field = rng.uniform(0.0, 1.0, dims[::-1]).astype(np.float32)
    boxes = [((0, 0, 0), (150, 220, 96)), ((150, 0, 0), (300, 220, 104)), ((0, 0, 96), (150, 220, 200)),
             ((150, 0, 104), (300, 220, 200))]
    cam = synth.orbit_camera((0, 0, 0), dims, *size, az_deg=az, el_deg=el, radius_factor=1.4)
    outs = []
    for path, config in ((dp.VR_PATH_STAGED, None), (dp.VR_PATH_STAGED, (1, 32, 4)), (dp.VR_PATH_DIRECT, None)):
        r = dp.Renderer([(synth.extract_brick(field, lo, hi), lo) for lo, hi in boxes], synth.default_tf(), (0.0, 1.0),
                        0.05, STEP, path=path, march_config=config)
        try:
            r.set_camera(cam)
            assert _stays_staged(r, cam, boxes)
            r.reset_samples()
            img = r.render((0.1, 0.2, 0.3, 1.0))
            r.synchronize()
            outs.append((img.cpu().numpy().copy(), r.sample_counts()))
        finally:
            r.close()
    for img, counts in outs[1:]:
        assert np.array_equal(img, outs[0][0]) and np.array_equal(counts, outs[0][1])
    assert np.sum(outs[0][1]) > 0
