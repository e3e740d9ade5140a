"""The tetrahedral march's search at its edges, against the oracle: long empty
stretches inside a part's box (skipped by the cells' distances), tiles with
more runs than the LDS pool holds, planes that float32 leaves undecided (a
mesh far from the origin), rays of one or two samples, and a vertex value that
is not finite."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

TOL = 1e-5      # per channel, the float32 bar of the frame


def _render(parts, vals, cam, dt, scale, max_runs):
    import paper_2501_01628_amd as dp
    tf, vr = synth.hidden_tf(11), (0.02, 0.95)
    r = dp.TetRenderer([(pv, pt) for pv, pt, _ in parts], tf, vr, scale, dt, max_runs=max_runs)
    try:
        for k, (_, _, used) in enumerate(parts):
            r.set_values(k, vals[used])
        r.set_camera(cam)
        r.samples.zero_()
        img = r.render((0.1, 0.0, 0.2, 0.5), count=True)
        r.synchronize()
        img, held = img.cpu().numpy().astype(np.float64), int(r.samples.item())
    finally:
        r.close()
    ref, cnt = oracle.render_tets(cam, [(pv, vals[used], pt) for pv, pt, used in parts], tf, vr, scale, dt,
                                  (0.1, 0.0, 0.2, 0.5))
    return img, held, ref, cnt


def _two_ends(v, t, length):
    """Part 0: both ends of the box, part 1: the middle."""
    x = v[t].mean(1)[:, 0]
    ends = (x < 2.0) | (x > length - 2.0)
    parts = []
    for sel in (ends, ~ends):
        used, inv = np.unique(t[sel], return_inverse=True)
        parts.append((v[used], inv.reshape(-1, 4).astype(np.int32), used))
    return parts


@pytest.mark.parametrize("name,cells,dt,shift,size", [
    ("gap", (14, 3, 3), 0.05, 0.0, (37, 21)), ("gap_coarse", (30, 2, 2), 0.9, 0.0, (24, 24)),
    ("pool", (6, 5, 5), 0.04, 0.0, (17, 19)), ("far_from_origin", (5, 4, 6), 0.21, 3.0e5, (23, 17)),
    ("few_samples", (3, 3, 3), 2.5, 0.0, (16, 9))])
def test_search_edges(name, cells, dt, shift, size):
    rng = np.random.default_rng(len(name))
    v, t = synth.tet_mesh(cells, jitter=0.15, rng=rng)
    vals = synth.tet_field(v, rng, cells)
    parts = _two_ends(v, t, cells[0]) if name.startswith("gap") else synth.tet_partitions(
        v, t, 3, rng, rough=name == "pool")
    lo = np.full(3, shift)
    parts = [(np.asarray(pv) + lo, pt, used) for pv, pt, used in parts]
    cam = synth.orbit_camera(lo, lo + np.asarray(cells), *size, az_deg=75.0, el_deg=12.0, radius_factor=1.2)
    print(f"tet search: {name}, {len(t)} tetrahedra, {size}, dt {dt}", flush=True)
    img, held, ref, cnt = _render(parts, vals, cam, dt, 0.7, 32)
    assert cnt[1] == 0 and held == int(cnt[0])
    assert np.max(np.abs(img - ref)) <= TOL


def test_value_that_is_not_finite():
    cells = (4, 4, 4)
    rng = np.random.default_rng(3)
    v, t = synth.tet_mesh(cells, jitter=0.1, rng=rng)
    vals = synth.tet_field(v, rng, cells)
    vals[len(vals) // 2] = np.inf          # classified as the table's last entry around that vertex
    cam = synth.orbit_camera((0, 0, 0), cells, 40, 30, az_deg=20.0, el_deg=30.0, radius_factor=1.3)
    print("tet search: infinite vertex value", flush=True)
    img, held, ref, cnt = _render([(v, t, np.arange(len(v)))], vals, cam, 0.3, 0.7, 8)
    assert held == int(cnt[0]) and np.isfinite(img).all()
    assert np.max(np.abs(img - ref)) <= TOL
