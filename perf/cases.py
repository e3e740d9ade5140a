"""Performance cases of the renderer's public entry points.

``listed()`` names the cases, ``draw(rng)`` gives more of the same ranges,
``prepare(case, seed)`` makes what a program holds before the call (bricks,
meshes, transfer function, camera, buffers), ``run(state)`` is one pass
through the public API, ``work(case)`` the bytes and operations the pass
cannot do without, and ``exact(case, seed)`` the same outputs computed in
float64 with plain torch, without the library.

Five kinds of work:
  frame   sort-last frame of a bricked volume (``Renderer.render``), with
          ``update`` preceded by the ingest of a new time step on every brick
  batch   bricks x time steps x cameras as one unit (``BatchRenderer``)
  grad    gradient step: forward + backward of an L2 image loss with respect
          to the transfer function and all voxels (``DiffRenderer``)
  rqc     ray-queue cycling with shadow rays (``Renderer.render_rqc``)
  tets    tetrahedral parts (``TetRenderer``), optionally with shadow rays
"""
import math

import numpy as np
import torch

import paper_2501_01628_amd as dp

DEV = "cuda"
BG = (0.1, 0.2, 0.3, 1.0)
LIGHT = (0.8, 1.0, -0.4)
AMBIENT = 0.3
CHUNK = 4_000_000          # ray samples evaluated together by exact()


# ------------------------------------------------------------------- the cases
def listed():
    return [
        # a thumbnail or a linked small view: launches and latency count
        dict(name="frame_small", kind="frame", nx=64, ny=64, nz=64, bricks=2, width=256, height=256, storage="f32",
             step=0.5, opacity=1.0, az=30.0, el=20.0, blobs=8, shock=False, noise=0.02, update=False),
        # an ordinary window on a ragged sub-volume, seen nearly along x as an orbit passes there
        dict(name="frame_ragged", kind="frame", nx=211, ny=149, nz=173, bricks=5, width=641, height=479,
             storage="f32", step=0.5, opacity=0.3, az=100.0, el=-12.0, blobs=24, shock=True, noise=0.0, update=False),
        # the benchmark frame: a large volume in 16 uneven bricks at full HD
        dict(name="frame_large", kind="frame", nx=1024, ny=1024, nz=512, bricks=16, width=1920, height=1080,
             storage="f32", step=0.5, opacity=0.05, az=30.0, el=20.0, blobs=64, shock=True, noise=0.0, update=False),
        # half-precision bricks, fine step, 4K image: the most samples per frame
        dict(name="frame_f16_4k", kind="frame", nx=1024, ny=512, nz=512, bricks=32, width=3840, height=2160,
             storage="f16", step=0.25, opacity=0.05, az=30.0, el=20.0, blobs=64, shock=True, noise=0.05,
             update=False),
        # playback of a simulation whose new time step is on the device: ingest of every brick, then the frame
        dict(name="frame_newstep", kind="frame", nx=384, ny=384, nz=256, bricks=8, width=1920, height=1080,
             storage="f32", step=0.5, opacity=0.1, az=30.0, el=20.0, blobs=48, shock=True, noise=0.0, update=True),
        # an image database: many small partials in one launch
        dict(name="batch", kind="batch", lo=48, hi=160, bricks=8, steps=3, cams=4, size=512, storage="f32", step=0.5,
             opacity=0.1, blobs=64),
        # transfer-function and volume fitting against eight views
        dict(name="grad_views", kind="grad", nx=128, ny=128, nz=128, bricks=1, width=512, height=512, crop=1.0,
             views=8, storage="f32", step=0.5, opacity=1.0, az=0.0, el=20.0, blobs=8, shock=False, interval=64),
        # fitting a larger bricked half-precision volume to the middle of one fine view
        dict(name="grad_bricks_f16", kind="grad", nx=512, ny=256, nz=256, bricks=16, width=384, height=384, crop=0.36,
             views=1, storage="f16", step=0.25, opacity=0.05, az=30.0, el=20.0, blobs=32, shock=True, interval=64),
        # shadows across bricks: every sample's ray toward the light visits every brick
        dict(name="rqc_shadows", kind="rqc", nx=96, ny=96, nz=96, bricks=6, width=384, height=384, step=0.5,
             opacity=0.25, az=30.0, el=20.0, blobs=8, shock=True),
        # an unstructured mesh in uneven non-convex parts
        dict(name="tets", kind="tets", cx=80, cy=64, cz=64, parts=8, width=1280, height=720, step=0.5, opacity=0.05,
             az=30.0, el=20.0, blobs=8, shadow=False),
        # a small odd mesh in a small view
        dict(name="tets_odd", kind="tets", cx=17, cy=13, cz=11, parts=3, width=317, height=241, step=0.31,
             opacity=0.4, az=205.0, el=-33.0, blobs=4, shadow=False),
        # the same kind of mesh with one directional light
        dict(name="tets_shadow", kind="tets", cx=40, cy=32, cz=32, parts=4, width=384, height=384, step=0.5,
             opacity=0.1, az=30.0, el=20.0, blobs=6, shadow=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    az, el = round(rng.uniform(0.0, 360.0), 1), round(rng.uniform(-50.0, 50.0), 1)
    kind = rng.choice(["frame", "frame", "frame", "batch", "grad", "grad", "rqc", "tets", "tets", "tets_shadow"])
    view = dict(az=az, el=el)
    if kind == "frame":
        f16 = rng.random() < 0.4
        # the finer step is drawn with smaller volumes: no drawn frame takes more samples than the listed 4K one
        step = rng.choice([0.5, 0.5, 0.25]) if f16 else 0.5
        top = 700 if step == 0.25 else 900
        w = _log(rng, 200, 2400)
        return dict(kind="frame", nx=_log(rng, 40, top), ny=_log(rng, 40, top), nz=_log(rng, 40, 512),
                    bricks=rng.randint(1, 24), width=w, height=max(64, int(w * rng.uniform(0.5, 0.8))),
                    storage="f16" if f16 else "f32", step=step, opacity=rng.choice([0.05, 0.1, 0.3, 1.0]),
                    blobs=rng.randint(8, 64), shock=rng.random() < 0.6, noise=rng.choice([0.0, 0.02, 0.05]),
                    update=rng.random() < 0.3, **view)
    if kind == "batch":
        lo = _log(rng, 24, 64)
        return dict(kind="batch", lo=lo, hi=lo + _log(rng, 8, 96), bricks=rng.randint(2, 10), steps=rng.randint(1, 4),
                    cams=rng.randint(1, 4), size=_log(rng, 160, 600), storage=rng.choice(["f32", "f16"]), step=0.5,
                    opacity=0.1, blobs=rng.randint(16, 64))
    if kind == "grad":
        w = _log(rng, 96, 512)
        return dict(kind="grad", nx=_log(rng, 40, 200), ny=_log(rng, 40, 200), nz=_log(rng, 40, 200),
                    bricks=rng.randint(1, 8), width=w, height=max(64, int(w * rng.uniform(0.7, 1.0))),
                    crop=rng.choice([1.0, 0.5]), views=rng.randint(1, 4), storage=rng.choice(["f32", "f16"]), step=0.5,
                    opacity=rng.choice([0.1, 0.3, 1.0]), blobs=rng.randint(8, 24), shock=rng.random() < 0.5,
                    interval=rng.choice([64, 64, 32, 16]), **view)
    if kind == "rqc":
        w = _log(rng, 96, 360)
        return dict(kind="rqc", nx=_log(rng, 32, 96), ny=_log(rng, 32, 96), nz=_log(rng, 32, 96),
                    bricks=rng.randint(2, 6), width=w, height=max(64, int(w * rng.uniform(0.7, 1.0))), step=0.5,
                    opacity=rng.choice([0.1, 0.25, 0.5]), blobs=rng.randint(4, 12), shock=rng.random() < 0.5, **view)
    shadow = kind == "tets_shadow"
    top = 32 if shadow else 64
    w = _log(rng, 120, 320 if shadow else 1280)
    return dict(kind="tets", cx=_log(rng, 8, top), cy=_log(rng, 8, top), cz=_log(rng, 8, top),
                parts=rng.randint(1, 6 if shadow else 10), width=w, height=max(64, int(w * rng.uniform(0.55, 0.9))),
                step=rng.choice([0.5, 0.37]), opacity=rng.choice([0.05, 0.1, 0.4]), blobs=rng.randint(3, 8),
                shadow=shadow, **view)


# ---------------------------------------------------------------- seeded inputs
def _table():
    x = np.array([0.0, 0.2, 0.4, 0.6, 0.8, 1.0])
    rgba = np.array([[0, 0, .5, 0], [0, .5, 1, 0], [0, 1, .5, .2], [1, 1, 0, .5], [1, .5, 0, .8], [1, 0, 0, 1.0]])
    g = np.arange(256) / 255.0
    return np.stack([np.interp(g, x, rgba[:, c]) for c in range(4)], 1).astype(np.float32)


def _orbit(dims, width, height, az, el, crop=1.0):
    """Perspective view of the box [0, dims] from twice its longest edge;
    crop < 1 narrows the field of view to the middle of the image."""
    c = 0.5 * np.asarray(dims, dtype=np.float64)
    r, a, e = 2.0 * float(max(dims)), math.radians(az), math.radians(el)
    off = r * np.array([math.cos(e) * math.sin(a), math.sin(e), math.cos(e) * math.cos(a)])
    fovy = math.degrees(2.0 * math.atan(crop * math.tan(math.radians(22.5))))
    return dict(kind="perspective", eye=tuple(float(v) for v in c + off), target=tuple(float(v) for v in c),
                up=(0.0, 1.0, 0.0), fovy_deg=fovy, width=int(width), height=int(height))


def _uniform(gen, lo, hi, *shape):
    return lo + (hi - lo) * torch.rand(*shape, generator=gen, dtype=torch.float64)


def _axis(n, off, centres, sigmas):
    x = torch.arange(n, dtype=torch.float64) + 0.5 + off
    return torch.exp(-(x[None, :] - centres[:, None]) ** 2 / (2.0 * sigmas[:, None] ** 2)).to(torch.float32).to(DEV)


def _blobs(shape, off, centres, sigmas, amps):
    """Sum of Gaussian blobs at the voxel centres of a grid of ``shape``
    (nx, ny, nz) whose first voxel has index ``off``."""
    nx, ny, nz = shape
    ax = [_axis(n, o, centres[:, a].contiguous(), sigmas) for a, (n, o) in enumerate(zip(shape, off))]
    yx = (ax[1][:, :, None] * ax[0][:, None, :]).reshape(len(amps), ny * nx)
    z = (ax[2] * amps.to(torch.float32).to(DEV)[:, None]).t().contiguous()
    return torch.mm(z, yx).view(nz, ny, nx)


def _sigma(dims):
    m = float(min(dims))
    return (4.0, 12.0) if m >= 48 else (max(1.0, m / 16.0), max(2.0, m / 5.0))


def _field(case, dims, gen, seed):
    """(nz, ny, nx) float32 field in [0, 1]: Gaussian blobs, optionally a
    tanh front and smooth noise."""
    nx, ny, nz = dims
    size = torch.tensor(dims, dtype=torch.float64)
    n = int(case["blobs"])
    v = _blobs(dims, (0, 0, 0), _uniform(gen, 0.0, 1.0, n, 3) * size, _uniform(gen, *_sigma(dims), n),
               _uniform(gen, 0.3, 1.0, n))
    if case.get("shock"):
        nrm = torch.randn(3, generator=gen, dtype=torch.float64)
        nrm = (nrm / nrm.norm()).tolist()
        p0 = (0.5 * size + _uniform(gen, -0.25, 0.25, 3) * size).tolist()
        ax = [((torch.arange(m, device=DEV, dtype=torch.float32) + 0.5 - p0[a]) * nrm[a]) for a, m in enumerate(dims)]
        yx = ax[1][:, None] + ax[0][None, :]
        for z in range(nz):
            v[z] += 0.3 * (1.0 - torch.tanh((yx + ax[2][z]) * 0.25))
    if case.get("noise"):
        g = torch.Generator(device=DEV)
        g.manual_seed(int(seed) + 77)
        low = torch.rand((1, 1, max(2, nz // 16), max(2, ny // 16), max(2, nx // 16)), device=DEV, generator=g)
        v += float(case["noise"]) * (torch.nn.functional.interpolate(low, size=(nz, ny, nx), mode="trilinear")[0, 0]
                                     - 0.5)
    return v.clamp_(0.0, 1.0)


def _boxes(dims, n, gen):
    """Uneven kd decomposition: the largest leaf is cut across its longest axis."""
    leaves = [((0, 0, 0), tuple(dims))]
    while len(leaves) < n:
        i = max(range(len(leaves)), key=lambda k: (math.prod(h - l for l, h in zip(*leaves[k])), -k))
        lo, hi = leaves[i]
        ext = [h - l for l, h in zip(lo, hi)]
        a = max(range(3), key=lambda k: (ext[k], -k))
        cut = lo[a] + min(max(int(round(float(_uniform(gen, 0.35, 0.65, 1)) * ext[a])), 1), ext[a] - 1)
        h0, l1 = list(hi), list(lo)
        h0[a] = l1[a] = cut
        leaves[i] = (lo, tuple(h0))
        leaves.append((tuple(l1), hi))
    return leaves


def _padded(field):
    """The field with one layer of edge copies on every face."""
    return torch.nn.functional.pad(field[None, None], (1,) * 6, mode="replicate")[0, 0]


def _scene(case, seed):
    gen = torch.Generator()
    gen.manual_seed(int(seed))
    dims = (case["nx"], case["ny"], case["nz"])
    field = _field(case, dims, gen, seed)
    return dims, field, _boxes(dims, case["bricks"], gen)


def _batch_scene(case, seed):
    """Bricks in the slots of a 4 x 2 x 2 grid, each time step a field of
    blobs moving through it; ghosts come from the analytic field."""
    gen = torch.Generator()
    gen.manual_seed(int(seed))
    ext = torch.randint(case["lo"], case["hi"] + 1, (case["bricks"], 3), generator=gen).tolist()
    pitch = case["hi"] + 16
    dims = (4 * pitch, 2 * pitch, 2 * pitch)
    n = case["blobs"]
    cen = _uniform(gen, 0.0, 1.0, n, 3) * torch.tensor(dims, dtype=torch.float64)
    sig, amp = _uniform(gen, 4.0, 12.0, n) * case["hi"] / 160.0, _uniform(gen, 0.3, 1.0, n)
    vel = _uniform(gen, -4.0, 4.0, n, 3)
    steps = []
    for t in range(case["steps"]):
        bricks = []
        for b, e in enumerate(ext):
            lo = tuple(pitch * s for s in (b % 4, (b // 4) % 2, (b // 8) % 2))
            vox = _blobs([v + 2 for v in e], [v - 1 for v in lo], cen + t * vel, sig, amp).clamp_(0.0, 1.0)
            bricks.append((vox, lo))
        steps.append(bricks)
    cams = [_orbit(dims, case["size"], case["size"], 30.0 + 90.0 * c, 20.0) for c in range(case["cams"])]
    return steps, cams


# the six tetrahedra of a cube around its main diagonal, as corner offsets
_KUHN = [[(0, 0, 0)] + [tuple(int(a in p[:m]) for a in range(3)) for m in (1, 2, 3)]
         for p in ((0, 1, 2), (0, 2, 1), (1, 0, 2), (1, 2, 0), (2, 0, 1), (2, 1, 0))]


def _mesh(case, seed):
    """Vertices (V, 3) float64 of the lattice (interior ones moved by up to
    0.15 per axis), tetrahedra (cubes, 6, 4) and float32 vertex values."""
    gen = torch.Generator()
    gen.manual_seed(int(seed))
    cells = (case["cx"], case["cy"], case["cz"])
    n = torch.tensor(cells)
    v = torch.cartesian_prod(*[torch.arange(c + 1, dtype=torch.float64) for c in cells]).to(DEV)
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) + 5)
    jit = (torch.rand(v.shape, device=DEV, generator=g, dtype=torch.float64) * 2.0 - 1.0) * 0.15
    inner = ((v > 0) & (v < n.to(DEV))).all(1)
    v[inner] += jit[inner]
    c = torch.cartesian_prod(*[torch.arange(m) for m in cells]).to(DEV)
    s = ((cells[1] + 1) * (cells[2] + 1), cells[2] + 1, 1)
    base = c[:, 0] * s[0] + c[:, 1] * s[1] + c[:, 2]
    offs = torch.tensor([[o[0] * s[0] + o[1] * s[1] + o[2] for o in t] for t in _KUHN], device=DEV)
    tets = base[:, None, None] + offs[None]
    size = n.to(torch.float64)
    m = max(cells)
    val = torch.zeros(len(v), dtype=torch.float64, device=DEV)
    for _ in range(case["blobs"]):
        p = (_uniform(gen, 0.0, 1.0, 3) * size).to(DEV)
        sg, am = float(_uniform(gen, m / 10, m / 4, 1)), float(_uniform(gen, 0.3, 1.0, 1))
        val += am * torch.exp(-((v - p) ** 2).sum(1) / (2.0 * sg * sg))
    return cells, v, tets, val.clamp(0.0, 1.0).to(torch.float32), gen


def _mesh_parts(case, cells, v, tets, gen):
    """Uneven non-convex parts: nearest seed under a weighted distance plus
    three plane waves per part.  [(vertices, tets, used)] with local numbering."""
    flat = tets.reshape(-1, 4)
    cen = v[flat].mean(1)
    m = float(max(cells))
    best = torch.full((len(flat),), math.inf, dtype=torch.float64, device=DEV)
    owner = torch.zeros(len(flat), dtype=torch.int64, device=DEV)
    for p in range(case["parts"]):
        seed = (_uniform(gen, 0.0, 1.0, 3) * torch.tensor(cells, dtype=torch.float64)).to(DEV)
        d = (cen - seed).norm(dim=1) / float(_uniform(gen, 0.5, 2.0, 1))
        for _ in range(3):
            k = torch.randn(3, generator=gen, dtype=torch.float64)
            k = (k / k.norm() * (6.0 * math.pi / m)).to(DEV)
            d += m / 24.0 * (1.0 + torch.sin((cen * k).sum(1) + float(_uniform(gen, 0.0, 2.0 * math.pi, 1))))
        near = d < best
        best = torch.where(near, d, best)
        owner[near] = p
    parts = []
    for p in range(case["parts"]):
        used, inv = torch.unique(flat[owner == p], return_inverse=True)
        parts.append((v[used].cpu().numpy(), inv.to(torch.int32).cpu().numpy().reshape(-1, 4), used))
    return parts


# ---------------------------------------------------------------- prepare and run
class _Owned:
    """Closes a renderer when the program drops it."""

    def __init__(self, r):
        self.r = r

    def __del__(self):
        try:
            self.r.close()
        except Exception:
            pass


def _storage(case):
    return dp.VR_F16 if case.get("storage") == "f16" else dp.VR_F32


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("frame", "rqc"):
        dims, field, boxes = _scene(case, seed)
        full = _padded(field)
        bricks = [(full[lo[2]:hi[2] + 2, lo[1]:hi[1] + 2, lo[0]:hi[0] + 2].contiguous(), lo) for lo, hi in boxes]
        r = dp.Renderer(bricks, _table(), (0.0, 1.0), case["opacity"], case["step"], storage=_storage(case))
        r.set_camera(_orbit(dims, case["width"], case["height"], case["az"], case["el"]))
        if kind == "rqc":
            r.rqc_plan()
            return dict(kind=kind, own=_Owned(r))
        r.synchronize()
        return dict(kind=kind, own=_Owned(r), new=[b for b, _ in bricks] if case["update"] else None)
    if kind == "batch":
        steps, cams = _batch_scene(case, seed)
        r = dp.BatchRenderer(case["step"])
        r.add_tf(_table(), (0.0, 1.0), case["opacity"])
        ids = [[r.add_brick(vox, lo, _storage(case)) for vox, lo in bricks] for bricks in steps]
        cam_ids = [r.add_camera(c) for c in cams]
        for bricks in ids:
            for c in cam_ids:
                r.add_frame(c, bricks, 0, BG)
        r.build()
        return dict(kind=kind, own=_Owned(r))
    if kind == "grad":
        dims, field, boxes = _scene(case, seed)
        dr = dp.DiffRenderer(dims, boxes, (0.0, 1.0), case["opacity"], case["step"], case["interval"],
                             storage=_storage(case))
        cams, targets = _grad_views(case, dims, seed)
        return dict(kind=kind, own=_Owned(dr), tf=torch.tensor(_table(), device=DEV, requires_grad=True),
                    vol=field.requires_grad_(True), cams=cams, targets=targets)
    cells, v, tets, val, gen = _mesh(case, seed)
    parts = _mesh_parts(case, cells, v, tets, gen)
    r = dp.TetRenderer([(pv, pt) for pv, pt, _ in parts], _table(), (0.0, 1.0), case["opacity"], case["step"],
                       max_runs=32)
    for k, (_, _, used) in enumerate(parts):
        r.set_values(k, val[used])
    r.set_camera(_orbit(cells, case["width"], case["height"], case["az"], case["el"]))
    if case["shadow"]:
        r.shadow_plan()
    return dict(kind=kind, own=_Owned(r), shadow=case["shadow"])


def _grad_views(case, dims, seed):
    cams = [_orbit(dims, case["width"], case["height"], case["az"] + 360.0 / case["views"] * k, case["el"],
                   case["crop"]) for k in range(case["views"])]
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) + 9)
    return cams, [torch.rand((c["height"], c["width"], 4), device=DEV, generator=g) for c in cams]


def run(state):
    kind, r = state["kind"], state["own"].r
    if kind == "frame":
        if state["new"] is not None:
            for k, vox in enumerate(state["new"]):
                r.set_data(k, vox)
        return r.render(BG)
    if kind == "batch":
        r.launch()
        return r.frames
    if kind == "rqc":
        return r.render_rqc(LIGHT, AMBIENT, BG)
    if kind == "grad":
        tf, vol = state["tf"], state["vol"]
        tf.grad = vol.grad = None
        frames = [r.render(tf, vol, cam, BG) for cam in state["cams"]]
        loss = sum(((f - t) ** 2).sum() for f, t in zip(frames, state["targets"]))
        loss.backward()
        return dict(frames=[f.detach() for f in frames], tf=tf.grad, vol=vol.grad)
    if state["shadow"]:
        return r.render_shadowed(LIGHT, AMBIENT, BG)
    return r.render(BG)


# ------------------------------------------------------------------------- work
def _chords(cam, lo, hi):
    """(mean over the image of the length of a pixel's ray inside the box) x
    pixels, from a coarse grid of pixels; (covered pixels) likewise."""
    n = 96
    px, py = np.meshgrid((np.arange(n) + 0.5) / n * cam["width"] - 0.5, (np.arange(n) + 0.5) / n * cam["height"] - 0.5)
    o, d = _rays_np(cam, px.ravel(), py.ravel())
    d = np.where(d == 0.0, 1e-300, d)
    with np.errstate(over="ignore"):
        a, b = (np.asarray(lo, float) - o) / d, (np.asarray(hi, float) - o) / d
    t = np.maximum(np.maximum(a, b).min(1) - np.maximum(np.minimum(a, b).max(1), 0.0), 0.0)
    s = cam["width"] * cam["height"] / float(n * n)
    return float(t.sum()) * s, float((t > 0).sum()) * s


def _rays_np(cam, px, py):
    eye, tgt, up = (np.asarray(cam[k], float) for k in ("eye", "target", "up"))
    f = (tgt - eye) / np.linalg.norm(tgt - eye)
    r = np.cross(f, up)
    r /= np.linalg.norm(r)
    u = np.cross(r, f)
    W, H, k = cam["width"], cam["height"], math.tan(math.radians(cam["fovy_deg"]) / 2.0)
    x, y = ((2.0 * (px + 0.5)) / W - 1.0) * (k * W / H), (1.0 - (2.0 * (py + 0.5)) / H) * k
    d = f + x[:, None] * r + y[:, None] * u
    return eye, d / np.linalg.norm(d, axis=1, keepdims=True)


def _shadow_samples(dims, dt):
    """Mean number of shadow samples of a point of the box."""
    p = np.random.default_rng(0).random((4096, 3)) * np.asarray(dims, float)
    l = np.asarray(LIGHT) / np.linalg.norm(LIGHT)
    t = np.where(l > 0, (np.asarray(dims, float) - p) / l, -p / l).min(1)
    return float(t.mean()) / dt


# operations of a sample: position 6, trilinear 21, table 10, exponential 1, accumulation 8
SAMPLE_OPS = 46


def work(case):
    kind = case["kind"]
    if kind == "batch":
        # extents are drawn; their mean stands for them
        e = 0.5 * (case["lo"] + case["hi"])
        pitch = case["hi"] + 16
        dims = (4 * pitch, 2 * pitch, 2 * pitch)
        samples = 0.0
        for c in range(case["cams"]):
            cam = _orbit(dims, case["size"], case["size"], 30.0 + 90.0 * c, 20.0)
            for b in range(case["bricks"]):
                lo = np.array([pitch * s for s in (b % 4, (b // 4) % 2, (b // 8) % 2)], float)
                samples += _chords(cam, lo, lo + e)[0] / case["step"]
        samples *= case["steps"]
        vox = case["steps"] * case["bricks"] * (e + 2) ** 3
        frames = case["steps"] * case["cams"] * case["size"] ** 2
        return dict(bytes=vox * (2 if case["storage"] == "f16" else 4) + 16 * frames, flops=SAMPLE_OPS * samples)
    if kind == "tets":
        cells = (case["cx"], case["cy"], case["cz"])
        cam = _orbit(cells, case["width"], case["height"], case["az"], case["el"])
        samples = _chords(cam, (0, 0, 0), cells)[0] / case["step"]
        if case["shadow"]:
            samples *= 1.0 + _shadow_samples(cells, case["step"])
        nt = 6 * math.prod(cells)
        # position 8, four sub-volumes 24, value 11, then table, exponential and accumulation
        return dict(bytes=nt * 16 + math.prod(c + 1 for c in cells) * 28 + 16 * case["width"] * case["height"],
                    flops=62.0 * samples)
    dims = (case["nx"], case["ny"], case["nz"])
    size = 2 if case.get("storage") == "f16" else 4
    vox = math.prod(dims)
    if kind == "grad":
        samples = 0.0
        for k in range(case["views"]):
            cam = _orbit(dims, case["width"], case["height"], case["az"] + 360.0 / case["views"] * k, case["el"],
                         case["crop"])
            samples += _chords(cam, (0, 0, 0), dims)[0] / case["step"]
        # forward, the walk back (the sample again, the recurrences and the products) and 8 corner sums
        frames = case["views"] * case["width"] * case["height"]
        return dict(bytes=vox * (4 + size + 4) + 48 * frames, flops=(2 * SAMPLE_OPS + 75) * samples)
    cam = _orbit(dims, case["width"], case["height"], case["az"], case["el"])
    samples, covered = _chords(cam, (0, 0, 0), dims)
    samples /= case["step"]
    frame = 16 * case["width"] * case["height"]
    if kind == "rqc":
        return dict(bytes=4 * vox + frame, flops=SAMPLE_OPS * samples * (1.0 + _shadow_samples(dims, case["step"])))
    # the ingest reads the new step and writes the bricks, the frame reads them
    return dict(bytes=vox * (size + (4 + size if case["update"] else 0)) + frame, flops=SAMPLE_OPS * samples)


# ------------------------------------------------------------- float64 reference
def _rays(cam):
    """Origin and unit directions (pixels, 3) in float64, row 0 at the top."""
    px = np.tile(np.arange(cam["width"], dtype=np.float64), cam["height"])
    py = np.repeat(np.arange(cam["height"], dtype=np.float64), cam["width"])
    o, d = _rays_np(cam, px, py)
    return torch.as_tensor(o, device=DEV), torch.as_tensor(d, device=DEV)


def _span(o, d, lo, hi, dt):
    """First sample index and number of samples that cover the box, per ray
    (o: (3,) or (n, 3)); a sample is at (k + 1/2) dt."""
    a, b = (lo - o) / d, (hi - o) / d
    tin = torch.minimum(a, b).nan_to_num(nan=-math.inf).amax(-1).clamp(min=0.0)
    tout = torch.maximum(a, b).nan_to_num(nan=math.inf).amin(-1)
    k0 = (torch.floor(tin / dt - 0.5) - 1.0).clamp(min=0.0)
    n = torch.ceil(tout / dt - 0.5) + 2.0 - k0
    return k0, torch.where(tout >= tin, n, torch.zeros_like(n)).clamp(min=0.0)


class _Grid:
    """A ghost-padded voxel box, its owned box [lo, hi) and trilinear samples of it."""

    def __init__(self, vox, lo):
        self.vox = vox.reshape(-1)
        self.n = [s - 2 for s in reversed(vox.shape)]
        self.lo = torch.tensor([float(v) for v in lo], dtype=torch.float64, device=DEV)
        self.hi = self.lo + torch.tensor([float(v) for v in self.n], dtype=torch.float64, device=DEV)

    def sample(self, p):
        """(values, owned) at the points p = (x, y, z) tensors."""
        inside = torch.ones_like(p[0], dtype=torch.bool)
        i, f = [], []
        for a in range(3):
            inside &= (p[a] >= self.lo[a]) & (p[a] < self.hi[a])
            s = p[a] - self.lo[a] + 0.5
            j = torch.floor(s).clamp(0, self.n[a])
            i.append(j.to(torch.int64))
            f.append(s - j)
        sx, sxy = self.n[0] + 2, (self.n[0] + 2) * (self.n[1] + 2)
        base = (i[2] * sxy + i[1] * sx + i[0]).reshape(-1)

        def at(o):
            return self.vox.index_select(0, base + o).view(p[0].shape)

        rows = [torch.lerp(at(o), at(o + 1), f[0]) for o in (0, sx, sxy, sxy + sx)]
        return torch.lerp(torch.lerp(rows[0], rows[1], f[1]), torch.lerp(rows[2], rows[3], f[1]), f[2]), inside


def _rgba(table, v):
    """Table rows interpolated at v (range [0, 1]); a table of 256 R rows is R
    copies (spreads the gradient's sums over them)."""
    s = (v * 255.0).clamp(0.0, 255.0)
    seg = torch.floor(s.detach()).clamp(max=254.0)
    phi = (s - seg).unsqueeze(-1)
    idx = seg.to(torch.int64).reshape(-1)
    if len(table) > 256:
        idx = idx + 256 * (torch.arange(len(idx), device=DEV) % (len(table) // 256))
    a, b = table.index_select(0, idx), table.index_select(0, idx + 1)
    a, b = a.view(*v.shape, 4), b.view(*v.shape, 4)
    return a + phi * (b - a)


def _weights(sigma_dt, inside):
    """Front-to-back weights T_k alpha_k along the last axis and 1 - T_end."""
    x = torch.where(inside, sigma_dt, torch.zeros_like(sigma_dt))
    c = torch.cumsum(x, -1)
    return torch.exp(x - c) * -torch.expm1(-x), -torch.expm1(-c[..., -1])


def _chunks(n):
    """Runs [a, b) of rays, in order, of about CHUNK samples each (n: samples per ray)."""
    counts = n.cpu().numpy()
    a = 0
    while a < len(counts):
        b = min(len(counts), a + 65536)
        while b - a > 64 and (b - a) * counts[a:b].max() > CHUNK:
            b = a + (b - a) // 2
        if counts[a:b].max() > 0:
            yield a, b, int(counts[a:b].max())
        a = b


def _points(o, d, k0, K, dt):
    t = (k0[:, None] + torch.arange(K, dtype=torch.float64, device=DEV)[None, :] + 0.5) * dt
    oo = o if o.dim() == 1 else o.t()[..., None]
    return t, [oo[a] + t * d[:, a, None] for a in range(3)]


def _frame64(case, cam, bricks, table, shade=None):
    """The frame (H, W, 4): bricks' partial images in depth order over BG.
    ``shade(points, owned)``: factors of the emitted colour."""
    dt, bg = float(case["step"]), torch.tensor(BG, dtype=torch.float64, device=DEV)
    o, d = _rays(cam)
    parts = []
    for grid in bricks:
        k0, n = _span(o, d, grid.lo, grid.hi, dt)
        C = torch.zeros(len(d), 4, dtype=torch.float64, device=DEV)
        key = torch.full((len(d),), math.inf, dtype=torch.float64, device=DEV)
        for a, b, K in _chunks(n):
            t, p = _points(o, d[a:b], k0[a:b], K, dt)
            v, inside = grid.sample(p)
            c = _rgba(table, v)
            w, A = _weights(c[..., 3] * (case["opacity"] * dt), inside)
            rgb = c[..., :3] if shade is None else c[..., :3] * shade(p, inside)[..., None]
            C[a:b, :3] = (w[..., None] * rgb).sum(1)
            C[a:b, 3] = A
            key[a:b] = torch.where(inside, t, torch.full_like(t, math.inf)).amin(1)
        parts.append((key, C))
    keys, order = torch.stack([k for k, _ in parts]).sort(dim=0, stable=True)
    out = torch.zeros(len(d), 4, dtype=torch.float64, device=DEV)
    everyone = torch.stack([c for _, c in parts])
    for q in range(len(parts)):
        out = out + (1.0 - out[:, 3:]) * everyone.gather(0, order[q][None, :, None].expand(1, -1, 4))[0]
    out = out + (1.0 - out[:, 3:]) * bg
    return out.view(cam["height"], cam["width"], 4)


def _stored(case, vox):
    """The voxel values as the bricks hold them, in float64."""
    return vox.to(torch.float16).double() if case.get("storage") == "f16" else vox.double()


def _shadow64(case, grid, table):
    """Transmittance factors a0 + (1 - a0) S of the points of a ray block."""
    dt = float(case["step"])
    l = torch.tensor(LIGHT, dtype=torch.float64, device=DEV)
    l = l / l.norm()

    def shade(p, inside):
        q = torch.stack([x[inside] for x in p], 1)
        S = torch.ones(len(q), dtype=torch.float64, device=DEV)
        k0, n = _span(q, l.expand_as(q), grid.lo, grid.hi, dt)
        order = torch.argsort(n)
        for a, b, K in _chunks(n[order]):
            sel = order[a:b]
            _, pts = _points(q[sel], l.expand(len(sel), 3), k0[sel], K, dt)
            v, own = grid.sample(pts)
            x = _rgba(table, v)[..., 3] * (case["opacity"] * dt)
            S[sel] = torch.exp(-torch.where(own, x, torch.zeros_like(x)).sum(1))
        f = torch.ones_like(p[0])
        f[inside] = AMBIENT + (1.0 - AMBIENT) * S
        return f

    return shade


class _Mesh64:
    """Point location by trying the tetrahedra of the cubes around a point
    (a vertex moves by 0.15 at most, so 27 cubes hold every candidate)."""

    def __init__(self, cells, v, tets, val):
        self.cells = torch.tensor(cells, dtype=torch.float64, device=DEV)
        self.dims = cells
        x = v[tets.reshape(-1, 4)]
        self.inv = torch.linalg.inv((x[:, 1:] - x[:, :1]).transpose(1, 2)).reshape(-1, 9)
        self.v0, self.val = x[:, 0].contiguous(), val.double()[tets.reshape(-1, 4)]
        self.lo, self.hi = torch.zeros(3, dtype=torch.float64, device=DEV), self.cells
        self.near = sorted(((i, j, k) for i in (-1, 0, 1) for j in (-1, 0, 1) for k in (-1, 0, 1)),
                           key=lambda o: sum(abs(a) for a in o))

    def sample(self, p):
        inside = torch.ones_like(p[0], dtype=torch.bool)
        for a in range(3):
            inside &= (p[a] >= 0.0) & (p[a] < self.cells[a])
        q = torch.stack([x[inside] for x in p], 1)
        val = torch.zeros(len(q), dtype=torch.float64, device=DEV)
        todo = torch.arange(len(q), device=DEV)
        cell = q.floor().to(torch.int64)
        for off in self.near:
            if not len(todo):
                break
            c = cell[todo] + torch.tensor(off, device=DEV)
            ok = ((c >= 0) & (c < self.cells.to(torch.int64))).all(1)
            sel, c = todo[ok], c[ok]
            base = 6 * ((c[:, 0] * self.dims[1] + c[:, 1]) * self.dims[2] + c[:, 2])
            found = torch.zeros(len(sel), dtype=torch.bool, device=DEV)
            for t in range(6):
                e = base + t
                x, m = q[sel] - self.v0[e], self.inv[e]
                lam = [(m[:, 3 * r:3 * r + 3] * x).sum(1) for r in range(3)]
                l0 = 1.0 - lam[0] - lam[1] - lam[2]
                hit = (torch.minimum(torch.minimum(lam[0], lam[1]), torch.minimum(lam[2], l0)) >= -1e-12) & ~found
                w = self.val[e]
                s = l0 * w[:, 0] + lam[0] * w[:, 1] + lam[1] * w[:, 2] + lam[2] * w[:, 3]
                val[sel] = torch.where(hit, s, val[sel])
                found |= hit
            done = torch.zeros(len(q), dtype=torch.bool, device=DEV)
            done[sel[found]] = True
            todo = todo[~done[todo]]
        out = torch.zeros_like(p[0])
        out[inside] = val
        return out, inside


def _grad64(case, seed):
    dims, field, _ = _scene(case, seed)
    dt, bg = float(case["step"]), torch.tensor(BG, dtype=torch.float64, device=DEV)
    cams, targets = _grad_views(case, dims, seed)
    vol = _stored(case, field).requires_grad_(True)
    tf = torch.tensor(_table(), device=DEV).double().requires_grad_(True)
    padded = _padded(vol)
    leaf = padded.detach().requires_grad_(True)
    copies = tf.repeat(1024, 1)
    tleaf = copies.detach().requires_grad_(True)
    grid = _Grid(leaf, (0, 0, 0))
    frames = []
    for cam, target in zip(cams, targets):
        o, d = _rays(cam)
        k0, n = _span(o, d, grid.lo, grid.hi, dt)
        out = bg.expand(len(d), 4).clone()
        want = target.double().view(-1, 4)
        for a, b, K in _chunks(2 * n):
            grid.vox = leaf.view(-1)
            _, p = _points(o, d[a:b], k0[a:b], (K + 1) // 2, dt)
            v, inside = grid.sample(p)
            c = _rgba(tleaf, v)
            w, A = _weights(c[..., 3] * (case["opacity"] * dt), inside)
            C = torch.cat([(w[..., None] * c[..., :3]).sum(1), A[:, None]], 1)
            f = C + (1.0 - C[:, 3:]) * bg
            ((f - want[a:b]) ** 2).sum().backward()
            out[a:b] = f.detach()
        frames.append(out.view(cam["height"], cam["width"], 4))
    torch.autograd.backward([padded, copies], [leaf.grad, tleaf.grad])
    return dict(frames=frames, tf=tf.grad, vol=vol.grad)


def exact(case, seed):
    kind = case["kind"]
    if kind == "grad":
        return _grad64(case, seed)
    with torch.no_grad():
        table = torch.tensor(_table(), device=DEV).double()
        if kind == "batch":
            steps, cams = _batch_scene(case, seed)
            return [_frame64(case, cam, [_Grid(_stored(case, vox), lo) for vox, lo in bricks], table)
                    for bricks in steps for cam in cams]
        if kind == "tets":
            cells, v, tets, val, _ = _mesh(case, seed)
            mesh = _Mesh64(cells, v, tets, val)
            cam = _orbit(cells, case["width"], case["height"], case["az"], case["el"])
            return _frame64(case, cam, [mesh], table, _shadow64(case, mesh, table) if case["shadow"] else None)
        # the frame does not depend on how the volume is split: one brick
        dims, field, _ = _scene(case, seed)
        grid = _Grid(_padded(_stored(case, field)), (0, 0, 0))
        cam = _orbit(dims, case["width"], case["height"], case["az"], case["el"])
        return _frame64(case, cam, [grid], table, _shadow64(case, grid, table) if kind == "rqc" else None)
