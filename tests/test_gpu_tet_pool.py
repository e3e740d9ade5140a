"""Tiles of the tetrahedral march with more runs than its LDS pool holds: a
mesh cut into thin layers along the view, two parts taking them in turn, so
that every ray crosses each part in 20 runs.  Images, held counts and the
error for too few run slots, against the oracle, with and without shadows."""
import os
import re

import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BG = (0.1, 0.0, 0.2, 0.5)
LAYERS, DT = 40, 0.3
LIGHT, AMBIENT = (1.0, 0.4, -0.2), 0.3
TF, VR, SCALE = synth.hidden_tf(11), (0.02, 0.95), 0.2


def _layers():
    rng = np.random.default_rng(17)
    cells = (2, 2, LAYERS)
    v, t = synth.tet_mesh(cells)
    vals = synth.tet_field(v, rng, cells)
    z = np.floor(v[t].mean(1)[:, 2]).astype(int)
    parts = []
    for p in (0, 1):
        used, inv = np.unique(t[z % 2 == p], return_inverse=True)
        parts.append((v[used], inv.reshape(-1, 4).astype(np.int32), vals[used]))
    # (the middle of the cells' faces: no ray lies in a face)
    cam = dict(kind="orthographic", eye=(1.013, 0.987, -1.0), dir=(0.0, 0.0, 1.0), up=(0.0, 1.0, 0.0),
               view_height=1.6, width=16, height=16)
    return parts, cam


def _runs_per_ray():
    zs = -1.0 + (np.arange(int((LAYERS + 2) / DT)) + 0.5) * DT
    layer = np.floor(zs[(zs > 0) & (zs < LAYERS)]).astype(int)
    return int(np.sum(np.diff(np.concatenate([[1], layer % 2 == 0])) == 1)) + int(layer[0] % 2 == 0)


@pytest.fixture(scope="module")
def case():
    return _layers()


def _renderer(case, max_runs, locator=None):
    import paper_2501_01628_amd as dp
    parts, cam = case
    r = dp.TetRenderer([(v, t) for v, t, _ in parts], TF, VR, SCALE, DT, max_runs=max_runs, locator=locator)
    for k, (_, _, vals) in enumerate(parts):
        r.set_values(k, vals)
    r.set_camera(cam)
    r.samples.zero_()
    return dp, r


def test_the_case_overfills_the_pool():
    src = open(os.path.join(ROOT, "paper_2501_01628_amd", "csrc", "tets.hip")).read()
    pool = int(re.search(r"constexpr int kPool = (\d+);", src).group(1))
    assert 64 * _runs_per_ray() > pool and _runs_per_ray() <= 32


@pytest.mark.parametrize("locator", [0, 1], ids=["grid", "bvh"])
def test_plain(case, locator):
    dp, r = _renderer(case, 32, locator)
    try:
        print("tet pool: plain", flush=True)
        img = r.render(BG, count=True)
        r.synchronize()
        img, held = img.cpu().numpy().astype(np.float64), int(r.samples.item())
    finally:
        r.close()
    ref, cnt = oracle.render_tets(case[1], [(v, f, t) for v, t, f in case[0]], TF, VR, SCALE, DT, BG)
    assert cnt[1] == 0 and held == int(cnt[0])
    assert np.max(np.abs(img - ref)) <= 1e-5


def test_shadowed(case):
    dp, r = _renderer(case, 32)
    try:
        print("tet pool: shadowed", flush=True)
        total = r.shadow_plan()
        img = r.render_shadowed(LIGHT, AMBIENT, BG, count=True)
        r.synchronize()
        img, held = img.cpu().numpy().astype(np.float64), int(r.samples.item())
    finally:
        r.close()
    ref, cnt = oracle.render_tets_shadowed(case[1], [(v, f, t) for v, t, f in case[0]], TF, VR, SCALE, DT, LIGHT,
                                           AMBIENT, BG)
    assert cnt[1] == 0 and total == int(cnt[0]) and held == int(cnt[0] + cnt[2])
    assert np.max(np.abs(img - ref)) <= 1e-5


def test_too_few_run_slots(case):
    dp, r = _renderer(case, 5)
    try:
        print("tet pool: five run slots", flush=True)
        r.render(BG)
        with pytest.raises(dp.VRError):
            r.synchronize()
    finally:
        r.close()
