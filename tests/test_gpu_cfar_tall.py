"""CFAR on images at and beyond the height whose tiles of 4 rows a launch can take
(65536 rows of workgroups)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from test_gpu_cfar import check  # noqa: E402


@pytest.mark.parametrize("H", [262140, 262141, 262145, 300001])
@pytest.mark.parametrize("W,guard,train", [(1, 0, 1), (3, 1, 2)])
def test_cfar_tall(H, W, guard, train):
    rng = np.random.default_rng(H + W)
    x = rng.normal(size=(H, W)) * 2.0 + 0.3
    x[rng.integers(0, H, 400), rng.integers(0, W, 400)] += 15.0
    check(x, guard, train, 3.0)
