"""Stored voxels of both ingest kernels, element by element: rows of every
remainder of a unit of four, sources that are not 16-byte aligned, pad columns,
and edge replication at each side of the global grid."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", [0, 1], ids=["f32", "f16"])
@pytest.mark.parametrize("nx", [1, 2, 3, 4, 5, 6, 7, 8, 13, 131])
def test_stored_voxels(nx, storage):
    import paper_2501_01628_amd as dp
    rng = np.random.default_rng(nx)
    dims, gdims, lo = (nx, 3, 2), (nx + 3, 4, 4), (2, 0, 2)
    snx, sny, snz = (n + 2 for n in dims)
    pitch = (snx + 7) // 8 * 8
    ctx = dp.vr_context_create(0)
    try:
        nbytes = dp.vr_brick_workspace_size(dims, 1, storage)
        buf = torch.full((nbytes + 256,), 0xAB, dtype=torch.uint8, device="cuda")
        off = -buf.data_ptr() % 256
        b = dp.vr_brick_create(ctx, dims, 1, (0.0, 0.0, 0.0), (1.0, 1.0, 1.0), storage, buf.data_ptr() + off, nbytes)
        dt = np.float16 if storage else np.float32
        n = pitch * sny * snz * np.dtype(dt).itemsize

        def stored():
            torch.cuda.synchronize()
            return buf[off:off + n].cpu().numpy().view(dt).reshape(snz, sny, pitch)

        vox = rng.normal(size=(snz, sny, snx)).astype(np.float32)
        src = torch.empty(vox.size + 1, device="cuda")
        src[1:] = torch.tensor(vox.reshape(-1))      # 4 bytes past an aligned address
        torch.cuda.synchronize()
        dp.vr_brick_set_data(b, src.data_ptr() + 4, ctx)
        want = np.pad(vox, ((0, 0), (0, 0), (0, pitch - snx))).astype(dt)
        assert np.array_equal(stored(), want)

        vol = rng.normal(size=gdims[::-1]).astype(np.float32)
        dev = torch.tensor(vol, device="cuda")
        torch.cuda.synchronize()
        dp.vr_brick_set_data_global(b, dev, gdims, lo, ctx)
        idx = [np.clip(np.arange(s) + o - 1, 0, g - 1) for s, o, g in zip((snx, sny, snz), lo, gdims)]
        want = np.pad(vol[np.ix_(idx[2], idx[1], idx[0])], ((0, 0), (0, 0), (0, pitch - snx))).astype(dt)
        assert np.array_equal(stored(), want)
        dp.vr_brick_release(b)
    finally:
        dp.vr_context_release(ctx)
