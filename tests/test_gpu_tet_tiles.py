"""Tetrahedral frames whose tiles go to a wavefront each (many tiles, or fewer
with few samples across a part): a sample of pixels against the oracle, plain
and shadowed, and every held sample counted once."""
import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BG = (0.1, 0.0, 0.2, 0.5)
LIGHT, AMBIENT = (1.0, 0.4, -0.2), 0.3


@pytest.mark.parametrize("locator", [0, 1], ids=["grid", "bvh"])
@pytest.mark.parametrize("name,cells,nparts,dt,size", [
    ("few samples across", (4, 4, 4), 1, 0.9, (1003, 807)),      # 12,726 tiles, a mean chord of 3 samples
    ("many tiles", (5, 4, 3), 4, 0.27, (1211, 973)),             # four parts over most of 152 x 122 tiles
])
def test_sampled_pixels(name, cells, nparts, dt, size, locator):
    import paper_2501_01628_amd as dp
    rng = np.random.default_rng(len(name))
    v, t = synth.tet_mesh(cells, jitter=0.15, rng=rng)
    vals = synth.tet_field(v, rng, cells)
    parts = synth.tet_partitions(v, t, nparts, rng, rough=nparts > 1)
    cam = synth.inside_camera((0, 0, 0), cells, *size) if nparts > 1 else synth.orbit_camera(
        (0, 0, 0), cells, *size, az_deg=35.0, el_deg=15.0, radius_factor=0.9)
    tf, vr, scale = synth.hidden_tf(11), (0.02, 0.95), 0.7
    pix = np.stack([rng.integers(0, size[0], 500), rng.integers(0, size[1], 500)], 1).astype(np.int32)
    pix[:2] = [(0, 0), (size[0] - 1, size[1] - 1)]
    print(f"tet tiles: {name}, locator {locator}", flush=True)
    r = dp.TetRenderer([(pv, pt) for pv, pt, _ in parts], tf, vr, scale, dt, max_runs=16, locator=locator)
    try:
        for k, (_, _, used) in enumerate(parts):
            r.set_values(k, vals[used])
        r.set_camera(cam)
        r.samples.zero_()
        plain = r.render(BG, count=True).cpu().numpy().astype(np.float64)
        r.synchronize()
        held = int(r.samples.item())
        total = r.shadow_plan()
        shadowed = r.render_shadowed(LIGHT, AMBIENT, BG).cpu().numpy().astype(np.float64)
        r.synchronize()
    finally:
        r.close()
    assert held == total > 0
    tparts = [(pv, vals[used], pt) for pv, pt, used in parts]
    for got, ref in ((plain, oracle.render_tets(cam, tparts, tf, vr, scale, dt, BG, pixels=pix)[0]),
                     (shadowed, oracle.render_tets_shadowed(cam, tparts, tf, vr, scale, dt, LIGHT, AMBIENT, BG,
                                                            pixels=pix)[0])):
        assert np.max(np.abs(got[pix[:, 1], pix[:, 0]] - np.asarray(ref).reshape(-1, 4))) <= 1e-5
