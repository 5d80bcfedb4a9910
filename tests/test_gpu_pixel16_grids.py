"""The 16x16x8 wave-per-anchor kernel at the edges of its candidate layout.

Stage C takes two candidates per lane up to 18 columns of the grid and one
beyond; stage B takes l_y in groups of seven; rounds and groups are left
partly filled by the sizes below (a single row, a single column, the largest
grid).  Search results against the oracle with the bars of test_gpu_parity;
frame pairs and the ring against single pushes; the refined velocity against
the parabola through the kernel's own smoothed R.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_1408_3526_amd import binding, scenes  # noqa: E402
from test_gpu_parity import _cfg, check_rs, check_velocity_and_output, run_gpu  # noqa: E402

M = (16, 16, 8)
GRIDS = [(1, 1), (1, 21), (21, 1), (2, 7), (3, 8), (9, 14), (17, 15), (18, 21), (19, 21), (21, 21), (20, 4)]


def _check(g, r, fr, nx, gx, gy):
    check_rs(g, r)
    if g["rs"].shape[-1] > 1:
        check_velocity_and_output(g, r, fr, nx, gx, gy)
    else:                                        # one candidate: no runner-up to compare with
        assert not g["idx"].any()
        rms = np.sqrt(np.mean(fr.astype(np.float64) ** 2, axis=(1, 2)))
        assert np.all(np.abs(g["out"] - r["out"]).max(axis=(1, 2)) <= 1e-3 * rms)


def _frames(nx, ny, H=19, W=6, T=11):
    rng = np.random.default_rng(100 * nx + ny)
    fr = scenes.gaussian_field(rng, 2 * H + 24, 2 * W + 24, 10.0)[:H, :W] + 100.0
    fr = np.stack([np.roll(fr, (t, -t), (0, 1)) + rng.normal(size=(H, W)) for t in range(T)]).astype(np.float32)
    gx = ((np.arange(nx) - (nx - 1) / 2) * 0.25).astype(np.float32)
    gy = ((np.arange(ny) - (ny - 1) / 2) * 0.25).astype(np.float32)
    return fr, gx, gy


@pytest.mark.parametrize("nx,ny", GRIDS)
def test_search_grids(orc, nx, ny):
    fr, gx, gy = _frames(nx, ny)
    T, H, W = fr.shape
    g = run_gpu(fr, M, gx, gy, tile_rows=5, kernel_variant=2)
    r = orc.run(_cfg(orc, H, W, M, gx, gy), fr, want_rs=True)
    _check(g, r, fr, nx, gx, gy)


@pytest.mark.parametrize("nx,ny", GRIDS)
def test_pairs_and_ring_grids(orc, nx, ny):
    fr, gx, gy = _frames(nx, ny)
    T, H, W = fr.shape
    dev = torch.from_numpy(fr).cuda()
    a, b = (binding.Filter(H, W, *M, gx, gy, tile_rows=5) for _ in range(2))
    outs = [torch.empty(H, W, device="cuda") for _ in range(T)]
    for t in range(T):
        a.push_frame(dev[t])
    b.push_frames(list(dev), outs)
    assert torch.equal(a.output(), outs[-1]) and torch.equal(a.output(), b.output())
    assert torch.equal(a.smoothed_r(), b.smoothed_r())
    assert torch.equal(a.velocity()[1], b.velocity()[1])
    ring = run_gpu(fr, M, gx, gy, tile_rows=5, temporal=binding.TEMPORAL_RING)
    r = orc.run(_cfg(orc, H, W, M, gx, gy), fr, want_rs=True)
    _check(ring, r, fr, nx, gx, gy)
    a.close()
    b.close()


@pytest.mark.parametrize("nx,ny", GRIDS)
def test_refined_grids(nx, ny):
    fr, gx, gy = _frames(nx, ny)
    T, H, W = fr.shape
    dev = torch.from_numpy(fr).cuda()
    f = binding.Filter(H, W, *M, gx, gy, tile_rows=5, velocity_mode=binding.VEL_REFINED)
    for t in range(T):
        f.push_frame(dev[t])
    vxy, idx = (v.cpu().numpy().astype(np.float64) for v in f.velocity())
    rs = f.smoothed_r().cpu().numpy().astype(np.float64)
    f.close()
    idx = idx.astype(np.int64)
    assert np.array_equal(idx, rs.argmax(-1))
    for axis, g, i, n, step in ((0, gx, idx % nx, nx, 1), (1, gy, idx // nx, ny, nx)):
        inner = (i > 0) & (i < n - 1)
        assert np.array_equal(vxy[..., axis][~inner], g[i[~inner]].astype(np.float64))
        if not inner.any():
            continue
        r0, r1, r2 = (np.take_along_axis(rs, np.clip(idx + q * step, 0, nx * ny - 1)[..., None], -1)[..., 0] for q in (-1, 0, 1))
        den = r0 - 2 * r1 + r2
        # FP32 differences of neighbouring R: 1e-3 of a grid step where the peak
        # curves by at least 1e-3 of its value (each R is rounded to 6e-8 of it)
        well = inner & (-den >= 1e-3 * np.abs(r1))
        v = g[i] - 0.5 * 0.25 * (r2 - r0) / np.where(den == 0, 1, den)
        assert np.abs(vxy[..., axis] - v)[well].max(initial=0) <= 1e-3 * 0.25


@pytest.mark.parametrize("step,shift", [(1.0, 0.0), (0.5, 8.0), (0.25, -3.75), (0.3, 0.0), (1.0, 100.0)])
def test_pairs_and_ring_lattice_steps(orc, step, shift):
    """The chosen velocity in lattice steps: single frames read them from a
    table, pairs and the ring form them from the grid (all lattice scales, a
    grid off the lattice, velocities beyond one turn of the table)."""
    fr, _, _ = _frames(9, 5)
    gx = ((np.arange(9) - 4) * step + shift).astype(np.float32)
    gy = ((np.arange(5) - 2) * step - shift).astype(np.float32)
    T, H, W = fr.shape
    dev = torch.from_numpy(fr).cuda()
    a, b = (binding.Filter(H, W, *M, gx, gy, tile_rows=5) for _ in range(2))
    outs = [torch.empty(H, W, device="cuda") for _ in range(T)]
    for t in range(T):
        a.push_frame(dev[t])
    b.push_frames(list(dev), outs)
    assert torch.equal(a.output(), outs[-1])
    assert torch.equal(a.velocity()[0], b.velocity()[0])
    ring = run_gpu(fr, M, gx, gy, tile_rows=5, temporal=binding.TEMPORAL_RING)
    _check(ring, orc.run(_cfg(orc, H, W, M, gx, gy), fr, want_rs=True), fr, 9, gx, gy)
    a.close()
    b.close()
