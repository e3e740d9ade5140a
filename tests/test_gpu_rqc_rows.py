"""Ray-queue cycling's brick reads at their edges: ragged tiles, one-voxel
bricks, lights along an axis, and float16 rows, against the oracle."""
import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BG = (0.1, 0.2, 0.3, 1.0)


@pytest.mark.parametrize("dims,boxes,size,light,storage", [
    ((9, 7, 11), [((0, 0, 0), (1, 7, 11)), ((1, 0, 0), (9, 7, 11))], (9, 7), (1.0, 0.0, 0.0), 0),
    ((8, 8, 8), [((0, 0, 0), (8, 8, 1)), ((0, 0, 1), (8, 3, 8)), ((0, 3, 1), (8, 8, 8))], (31, 17), (0.2, -1.0, 0.3), 1),
    ((33, 5, 6), [((0, 0, 0), (33, 5, 6))], (64, 8), (-0.4, 0.1, -1.0), 0)])
def test_shadowed_bricks_at_their_edges(dims, boxes, size, light, storage):
    import paper_2501_01628_amd as dp
    rng = np.random.default_rng(sum(dims))
    field = rng.uniform(0.0, 1.0, dims[::-1]).astype(np.float32)
    if storage:
        field = field.astype(np.float16).astype(np.float32)     # what the bricks hold
    cam = synth.orbit_camera((0, 0, 0), dims, *size, az_deg=40.0, el_deg=25.0, radius_factor=1.4)
    sc = synth.scene_from_field("rows", field, boxes, synth.default_tf(), cam, 0.4, 1.5)
    print(f"rqc rows: {dims}, {len(boxes)} bricks, {size}, light {light}, storage {storage}", flush=True)
    r = dp.Renderer([(b.voxels, b.lo) for b in sc.bricks], sc.tf, sc.vrange, sc.opacity_scale, sc.step, 0.0,
                    storage=storage)
    try:
        r.set_camera(cam)
        r.rqc_plan()
        out = r.render_rqc(light, 0.25, BG)
        r.synchronize()
        got = out.cpu().numpy().astype(np.float64)
    finally:
        r.close()
    ref, _, _ = oracle.render_scene_shadowed(sc, light, 0.25, bg=BG)
    assert np.max(np.abs(got - np.asarray(ref).reshape(got.shape))) <= 1e-5
