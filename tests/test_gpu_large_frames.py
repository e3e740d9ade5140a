"""The largest image the camera takes, 32768 x 32768: more 8 x 8 tiles than one
launch holds workgroups for.  A sample of pixels (the corners and random ones)
against the oracle."""
import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SIZE = 32768
BG = (0.1, 0.2, 0.3, 1.0)
LIGHT, AMBIENT = (0.3, 1.0, -0.4), 0.25


@pytest.fixture(autouse=True)
def _room():
    if not torch.cuda.is_available() or torch.cuda.mem_get_info()[0] < 120 << 30:
        pytest.skip("needs 120 GB of free device memory")
    yield
    torch.cuda.empty_cache()


def _pixels():
    rng = np.random.default_rng(3)
    far = SIZE - 1
    return np.concatenate([[(0, 0), (far, 0), (0, far), (far, far)],
                           rng.integers(0, SIZE, (300, 2))]).astype(np.int32)


def _at(frame, pix):
    x, y = (torch.from_numpy(pix[:, c].astype(np.int64)).cuda() for c in (0, 1))
    return frame.view(SIZE, SIZE, 4)[y, x].double().cpu().numpy()


def test_ray_queue_shadows():
    import paper_2501_01628_amd as dp
    dims = (5, 4, 4)
    field = np.random.default_rng(9).uniform(0.0, 1.0, dims[::-1]).astype(np.float32)
    cam = synth.inside_camera((0, 0, 0), dims, SIZE, SIZE)
    sc = synth.scene_from_field("large", field, [((0, 0, 0), dims)], synth.default_tf(), cam, 1.5, 0.5)
    pix = _pixels()
    print("rqc at 32768 x 32768", flush=True)
    r = dp.Renderer([(b.voxels, b.lo) for b in sc.bricks], sc.tf, sc.vrange, sc.opacity_scale, sc.step, 0.0)
    try:
        r.set_camera(cam)
        assert r.rqc_plan() > SIZE * SIZE // 2
        r.render_rqc(LIGHT, AMBIENT, BG)
        r.synchronize()
        got = _at(r.frame, pix)
    finally:
        r.close()
        del r
    ref, _, _ = oracle.render_scene_shadowed(sc, LIGHT, AMBIENT, bg=BG, pixels=pix)
    assert np.max(np.abs(got - np.asarray(ref).reshape(got.shape))) <= 1e-5


def test_tetrahedral_parts_with_and_without_shadows():
    import paper_2501_01628_amd as dp
    cells = (2, 2, 2)
    rng = np.random.default_rng(13)
    v, t = synth.tet_mesh(cells, jitter=0.1, rng=rng)
    vals = synth.tet_field(v, rng, cells)
    cam = synth.inside_camera((0, 0, 0), cells, SIZE, SIZE)
    pix = _pixels()
    tf, vr, scale, dt = synth.hidden_tf(11), (0.02, 0.95), 0.7, 0.45
    print("tets at 32768 x 32768", flush=True)
    r = dp.TetRenderer([(v, t)], tf, vr, scale, dt, max_runs=1)
    try:
        r.set_values(0, vals)
        r.set_camera(cam)
        r.render(BG)
        r.synchronize()
        plain = _at(r.frame, pix)
        assert r.shadow_plan() > SIZE * SIZE // 2
        r.render_shadowed(LIGHT, AMBIENT, BG)
        r.synchronize()
        shadowed = _at(r.frame, pix)
    finally:
        r.close()
        del r
    ref, _ = oracle.render_tets(cam, [(v, vals, t)], tf, vr, scale, dt, BG, pixels=pix)
    assert np.max(np.abs(plain - np.asarray(ref).reshape(plain.shape))) <= 1e-5
    ref, _ = oracle.render_tets_shadowed(cam, [(v, vals, t)], tf, vr, scale, dt, LIGHT, AMBIENT, BG, pixels=pix)
    assert np.max(np.abs(shadowed - np.asarray(ref).reshape(shadowed.shape))) <= 1e-5
