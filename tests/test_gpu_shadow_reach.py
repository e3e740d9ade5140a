"""Shadow rays at the ends of their range: a mesh part that they reach after
more than 2^31 samples."""
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
