"""The generic per-pixel tile at the edges of its lane and candidate split.

Anchors go four or eight to a workgroup (one or two to a wavefront), candidates
go 32 or 64 to a round and six rounds to a group of smoothed-R loads, and the
first lag transform takes its (kx, l_y) items 32 or 64 at a time: the sizes
below leave remainders of one or all but one in each of these, and cover grids
of one row, one column and the largest allowed.  Bars as in test_gpu_parity.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_1408_3526_amd import scenes  # noqa: E402
from test_gpu_parity import _cfg, check_rs, check_velocity_and_output, run_gpu  # noqa: E402

M8, M9, M16 = (8, 8, 4), (9, 9, 5), (16, 16, 8)


@pytest.mark.parametrize("M,H,W,nx,ny,tile", [
    (M8, 9, 1, 9, 9, 3), (M8, 11, 7, 1, 33, 4), (M8, 6, 9, 33, 1, 32), (M8, 5, 17, 33, 33, 2), (M8, 3, 8, 11, 3, 1),
    (M9, 10, 1, 17, 17, 4), (M9, 11, 3, 1, 33, 32), (M9, 4, 5, 33, 1, 1), (M9, 5, 9, 33, 33, 3), (M9, 3, 4, 13, 5, 2),
    (M16, 17, 1, 22, 5, 4), (M16, 18, 3, 1, 33, 32), (M16, 4, 5, 33, 2, 1), (M16, 5, 7, 33, 33, 3), (M16, 3, 4, 13, 5, 2),
])
def test_generic_tile_remainders(orc, M, H, W, nx, ny, tile):
    rng = np.random.default_rng(1000 * H + 10 * W + nx)
    T = M[2] + 3
    fr = scenes.gaussian_field(rng, 2 * H + 16, 2 * W + 16, 10.0)[:H, :W] + 100.0
    fr = np.stack([np.roll(fr, (t, -t), (0, 1)) + rng.normal(size=(H, W)) for t in range(T)]).astype(np.float32)
    gx = ((np.arange(nx) - (nx - 1) / 2) * 0.25).astype(np.float32)
    gy = ((np.arange(ny) - (ny - 1) / 2) * 0.25).astype(np.float32)
    g = run_gpu(fr, M, gx, gy, tile_rows=tile, kernel_variant=1)
    r = orc.run(_cfg(orc, H, W, M, gx, gy), fr, want_rs=True)
    check_rs(g, r)
    check_velocity_and_output(g, r, fr, nx, gx, gy)


@pytest.mark.parametrize("M,H,W,tile", [(M8, 70, 21, 64), (M8, 75, 30, 70), (M8, 9, 21, 1), (M9, 70, 19, 64),
                                        (M9, 9, 21, 1), (M9, 34, 18, 33), (M16, 70, 17, 64), (M16, 41, 37, 8)])
def test_rows_computed_in_tiles_equal_the_row_kernel(M, H, W, tile):
    """Tiles that compute their own row spectra (single streams) against the row
    kernel's (the batch uses it for every stream), bit for bit: tiles beyond the
    32 rows staged at a time, columns past the frame, non-finite samples."""
    from paper_1408_3526_amd import binding
    rng = np.random.default_rng(H + W)
    fr = (rng.normal(size=(10, H, W)) * 10 + 100).astype(np.float32)
    fr[2, H // 2, W // 3] = np.nan
    fr[5, 0, 0] = np.inf
    fr[5, H - 1, W - 1] = -np.inf
    g = scenes.grid(-2, 2, 0.5)
    f = binding.Filter(H, W, *M, g, g, tile_rows=tile, kernel_variant=1)
    b = binding.Batch([dict(H=H, W=W, M=M, gx=g, gy=g)], tile_rows=tile, kernel_variant=1)
    dev = torch.from_numpy(fr).cuda()
    for t in range(len(fr)):
        f.push_frame(dev[t])
        b.push([dev[t]])
        out, vxy, idx = b.output(0)
        assert torch.equal(f.output(), out), t
        assert torch.equal(f.velocity()[1], idx), t
    assert f.nonfinite_count() == 3
    f.close()
    b.close()


@pytest.mark.parametrize("M", [M8, M9])
def test_no_delay_reads_the_frame_being_stored(orc, M):
    """Output delay 0 in time: the delayed sample is the current frame's, whose
    delay-ring slot the same launch is storing (a non-finite sample reads as 0)."""
    H, W, T = 12, 14, 8
    rng = np.random.default_rng(3)
    fr = (rng.normal(size=(T, H, W)) * 5 + 50).astype(np.float32)
    fr[4, 3, 2] = np.nan
    g = scenes.grid(-1, 1, 0.5)
    r = run_gpu(fr, M, g, g, delay=(2, 3, 0), tile_rows=1)
    o = orc.run(_cfg(orc, H, W, M, g, g, dx=2, dy=3, dt=0), fr, want_rs=True)
    check_rs(r, o)
    check_velocity_and_output(r, o, np.where(np.isfinite(fr), fr, 0), len(g), g, g)
    assert r["nonfinite"] == 1


@pytest.mark.parametrize("M,nx,ny", [(M8, 9, 7), (M9, 13, 11), (M16, 13, 11)])
def test_best_candidate_where_r_overflows(M, nx, ny):
    """Samples whose power overflows FP32 in some anchors: the index is the first
    of the largest smoothed R, values that are not numbers left out, and 0 where
    there is no other."""
    from paper_1408_3526_amd import binding
    H, W, T = 13, 23, 5
    rng = np.random.default_rng(nx)
    fr = rng.normal(size=(T, H, W)) * 10.0 ** np.linspace(16, 20, W)
    fr[:, :3] = 0.0
    gx, gy = (((np.arange(n) - n // 2) * 0.25).astype(np.float32) for n in (nx, ny))
    f = binding.Filter(H, W, *M, gx, gy, tile_rows=4, kernel_variant=1)
    dev = torch.from_numpy(fr.astype(np.float32)).cuda()
    seen = set()
    for t in range(T):
        f.push_frame(dev[t])
        rs = f.smoothed_r().cpu().numpy()
        idx = f.velocity()[1].cpu().numpy()
        for y in range(H):
            for x in range(W):
                r = rs[y, x]
                ok = r[~np.isnan(r)]
                want = int(np.argmax(r == ok.max())) if ok.size else 0
                assert idx[y, x] == want, (t, y, x)
                seen.add("none" if not ok.size else "least" if np.isneginf(ok.max()) else "inf" if np.isinf(ok.max()) else "finite")
    assert "finite" in seen and len(seen) > 1
    f.close()
