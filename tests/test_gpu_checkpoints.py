"""What the checkpointed forward stores: the transmittance in front of every
interval-th owned sample of a ray, against the product of exp2(-a') in float64.

Every sample falls on a voxel centre, so a' is the table's opacity at the
voxel's value to 2^-22 (float32 table arithmetic).  Tolerance, relative: 2^-22 ln
2 of the ray's total a' (at most 30) + 2 roundings a sample (128 samples):
30 * 1.7e-7 + 256 * 6e-8 < 2.1e-5."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 2.1e-5


@pytest.mark.parametrize("storage", [0, 1], ids=["f32", "f16"])
@pytest.mark.parametrize("interval", [1, 3, 32, 64])
@pytest.mark.parametrize("many", [False, True], ids=["one call a partial", "one call"])
def test_stored_transmittance(interval, many, storage):
    import paper_2501_01628_amd as dp
    rng = np.random.default_rng(37)
    dims, w, h = (5, 4, 128), 5, 4
    scale = 0.6
    field = rng.uniform(0.0, 1.0, dims[::-1]).astype(np.float32)
    if storage:
        field = field.astype(np.float16).astype(np.float32)
    boxes = [((0, 0, 0), (5, 4, 60)), ((0, 0, 60), (5, 4, 128))]
    # one pixel a voxel column, samples at the voxels' centres
    cam = dict(kind="orthographic", eye=(2.5, 2.0, -3.0), dir=(0.0, 0.0, 1.0), up=(0.0, 1.0, 0.0), view_height=4.0,
               width=w, height=h)
    tf = synth.default_tf()
    r = dp.Renderer([(synth.extract_brick(field, lo, hi), lo) for lo, hi in boxes], tf, (0.0, 1.0), scale, 1.0, 0.0,
                    storage=storage)
    try:
        r.set_camera(cam)
        sizes = [dp.vr_checkpoint_size(r.ctx, b, p, interval) for b, p in zip(r.bricks, r.partials)]
        bufs = [torch.full((n // 4,), float("nan"), device="cuda") for n in sizes]
        print(f"checkpoints: interval {interval}, many {many}, storage {storage}", flush=True)
        if many:
            need = dp.vr_checkpointed_workspace_size(len(boxes))
            ws = torch.empty(need // 4 + 64, device="cuda")
            dp.vr_render_partials_checkpointed(r.ctx, r.bricks, r.partials, interval, list(zip(bufs, sizes)),
                                               ws.data_ptr() + (-ws.data_ptr()) % 256, need)
        else:
            for b, p, ck, n in zip(r.bricks, r.partials, bufs, sizes):
                dp.vr_render_partial_checkpointed(r.ctx, b, p, interval, ck, n)
        r.synchronize()
        got = [b.cpu().numpy().astype(np.float64) for b in bufs]
        rois = list(r.rois)
    finally:
        r.close()
    alpha = np.asarray(tf, dtype=np.float64)[:, 3] * scale * np.log2(np.e)
    for (lo, hi), roi, ck in zip(boxes, rois, got):
        ck = ck.reshape(roi[3], roi[2], -1)
        n = hi[2] - lo[2]
        for y in range(h):
            for x in range(w):
                # image right is camera r = dir x up = -x; image up is +y
                col = field[lo[2]:hi[2], h - 1 - y, w - 1 - x].astype(np.float64)
                a = np.interp(col * 255.0, np.arange(256), alpha)
                T = np.exp2(-np.concatenate([[0.0], np.cumsum(a)]))[0:n:interval]
                have = ck[y - roi[1], x - roi[0], :len(T)]
                assert np.max(np.abs(have - T) / T) <= TOL, (x, y)
