"""Shadow rays of a mesh whose pixels hold very different numbers of samples:
one layer of cells across the view and a long column behind a few pixels, so
that those pixels hold far more samples than the wavefronts that the mean
pixel gives a tile (and take several rounds), against the oracle."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

BG = (0.1, 0.0, 0.2, 0.5)


@pytest.mark.parametrize("size", [(24, 24), (61, 43)])
def test_column_behind_a_layer(size):
    import paper_2501_01628_amd as dp
    rng = np.random.default_rng(23)
    cells, dt = (40, 6, 6), 0.45
    v, t = synth.tet_mesh(cells)
    c = np.floor(v[t].mean(1)).astype(int)
    t = t[(c[:, 0] == 0) | ((c[:, 1] == 2) & (c[:, 2] == 3))]
    used, inv = np.unique(t, return_inverse=True)
    v, t = v[used], inv.reshape(-1, 4).astype(np.int32)
    vals = synth.tet_field(v, rng, cells)
    cam = dict(kind="orthographic", eye=(-2.0, 3.013, 2.987), dir=(1.0, 0.0, 0.0), up=(0.0, 1.0, 0.0),
               view_height=6.3, width=size[0], height=size[1])
    tf, vr, scale, light, ambient = synth.hidden_tf(11), (0.02, 0.95), 0.4, (-1.0, 0.02, 0.01), 0.2
    r = dp.TetRenderer([(v, t)], tf, vr, scale, dt, max_runs=4)
    try:
        r.set_values(0, vals)
        r.set_camera(cam)
        total = r.shadow_plan()
        # (a pixel of the column holds 88 samples; 6 wavefronts a sample of the mean pixel are fewer)
        assert 0 < 6.0 * total / (size[0] * size[1]) + 4 < 80
        r.samples.zero_()
        img = r.render_shadowed(light, ambient, BG, count=True).cpu().numpy().astype(np.float64)
        r.synchronize()
        held = int(r.samples.item())
    finally:
        r.close()
    ref, cnt = oracle.render_tets_shadowed(cam, [(v, vals, t)], tf, vr, scale, dt, light, ambient, BG)
    assert total == int(cnt[0]) and held == int(cnt[0] + cnt[2])
    assert np.max(np.abs(img - np.asarray(ref).reshape(img.shape))) <= 1e-5
