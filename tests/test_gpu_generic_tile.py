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
