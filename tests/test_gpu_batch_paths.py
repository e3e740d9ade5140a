"""A batch whose groups march directly by the rule, against the same batch with
staged configurations chosen by hand, tuned, and tuned from its cache file: the
same bits, with mixed storage and several release groups."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _images(br):
    for f in br.frames:
        f.fill_(-1.0)
    torch.cuda.synchronize()
    br.launch()
    br.synchronize()
    return [f.cpu().numpy().copy() for f in br.frames]


@pytest.mark.parametrize("dims,size,storage,groups", [
    ((24, 20, 28), (61, 47), (0,), 1),           # direct: few tiles
    ((40, 36, 44), (320, 300), (0, 1), 2),       # float32 direct, float16 staged (fine pixels)
    ((40, 36, 44), (33, 31), (1,), 2),           # float16 direct
])
def test_batch_paths_give_the_same_bits(dims, size, storage, groups, tmp_path, monkeypatch):
    import paper_2501_01628_amd as dp
    rng = np.random.default_rng(83)
    field = rng.uniform(0.0, 1.0, dims[::-1]).astype(np.float32)
    boxes = synth.kd_split(dims, 4, rng)
    cams = [synth.orbit_camera((0, 0, 0), dims, *size, az_deg=az, el_deg=15.0, radius_factor=1.3) for az in (30, 95)]
    out = []
    for chosen in (None, (0, 16, 4), (1, 32, 8)):
        br = dp.BatchRenderer(0.5)
        try:
            if chosen:
                for st in (0, 1):
                    dp.vr_set_march_config(br.ctx, st, *chosen)
            br.add_tf(synth.default_tf(), (0.0, 1.0), 0.3)
            ids = [br.add_brick(synth.extract_brick(field, lo, hi), lo, storage[k % len(storage)])
                   for k, (lo, hi) in enumerate(boxes)]
            for c in [br.add_camera(c) for c in cams]:
                br.add_frame(c, ids, 0, (0.1, 0.2, 0.3, 1.0))
            br.build()
            if groups > 1:
                dp.vr_batch_set_groups(br.batch, groups)
            out.append(_images(br))
            if chosen is None:
                monkeypatch.setenv("DPVR_AUTOTUNE_CACHE", str(tmp_path / "tune.txt"))
                assert br.autotune(reps=2) > 0.0
                out.append(_images(br))
                assert br.autotune(reps=2) == -1.0
                out.append(_images(br))
        finally:
            br.close()
    for imgs in out[1:]:
        for a, b in zip(out[0], imgs):
            assert np.array_equal(a, b)
    assert all(np.isfinite(a).all() for a in out[0])
