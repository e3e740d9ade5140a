"""Shadow rays at the ends of their range: a mesh part that they reach after
more than 2^31 samples, and a light whose direction has a component too small
to have a reciprocal."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BG = (0.1, 0.2, 0.3, 1.0)


def _two_parts(shift):
    """A cube of 3^3 cells in view, and one like it `shift` along x, out of view."""
    import paper_2501_01628_amd as dp
    rng = np.random.default_rng(5)
    v, t = synth.tet_mesh((3, 3, 3), jitter=0.125, rng=rng)
    v = np.round(np.asarray(v) * 64.0) / 64.0            # exact after the shift
    vals = synth.tet_field(v, rng, (3, 3, 3))
    cam = dict(kind="orthographic", eye=(1.5, 1.5, -4.0), dir=(0.0, 0.0, 1.0), up=(0.0, 1.0, 0.0), view_height=3.5,
               width=24, height=24)
    r = dp.TetRenderer([(v, t), (v + np.array([shift, 0.0, 0.0]), t)], synth.hidden_tf(11), (0.02, 0.95), 1.5,
                       2.0 ** -7)
    try:
        for k in (0, 1):
            r.set_values(k, vals)
        r.set_camera(cam)
        total = r.shadow_plan()
        r.samples.zero_()
        img = r.render_shadowed((1.0, 0.0, 0.0), 0.2, BG, count=True)
        r.synchronize()
        return img.cpu().numpy().copy(), total, int(r.samples.item())
    finally:
        r.close()


def test_part_beyond_two_to_the_31_shadow_samples():
    """The far part shades as the near one does: moved by 3 * 2^23 (3 * 2^30
    steps of 2^-7), its samples move by whole steps, and the sample points
    round at 2^-28."""
    near, total, held = _two_parts(8.0)
    far, total_far, held_far = _two_parts(8.0 + 3.0 * 2.0 ** 23)
    assert total_far == total > 0 and held > total
    assert abs(held_far - held) <= 1e-3 * held            # points on faces may round to either side
    assert np.max(np.abs(far - near)) <= 1e-5


def test_light_component_without_a_reciprocal():
    """A direction component of 1e-310 moves no sample, so the image is that
    of a zero component: also for samples exactly on a brick's lower face,
    whose distance to it is zero."""
    import paper_2501_01628_amd as dp
    dims = (8, 8, 8)
    rng = np.random.default_rng(7)
    field = rng.uniform(0.0, 1.0, dims).astype(np.float32)
    boxes = [((0, 0, 0), (8, 4, 8)), ((0, 4, 0), (8, 8, 8))]
    # the middle row of pixels sees exactly y = 4
    cam = dict(kind="orthographic", eye=(4.0, 4.0, -16.0), dir=(0.0, 0.0, 1.0), up=(0.0, 1.0, 0.0), view_height=9.0,
               width=9, height=9)
    sc = synth.scene_from_field("light", field, boxes, synth.default_tf(), cam, 0.5, 1.5)
    imgs = []
    for light in ((1.0, 0.0, 0.0), (1.0, 1e-310, 0.0)):
        r = dp.Renderer([(b.voxels, b.lo) for b in sc.bricks], sc.tf, sc.vrange, sc.opacity_scale, sc.step, 0.0)
        try:
            r.set_camera(cam)
            r.rqc_plan()
            out = r.render_rqc(light, 0.1, BG)
            r.synchronize()
            imgs.append(out.cpu().numpy().copy())
        finally:
            r.close()
    assert np.max(np.abs(imgs[1] - imgs[0])) <= 1e-6
