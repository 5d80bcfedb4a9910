"""rmdf_mlp_grads against the layer-by-layer entry points it stands for
(rmdf_mlp_gemm_nt, rmdf_mlp_head, rmdf_mlp_transpose, rmdf_mlp_colsum)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import mlp  # noqa: E402
from test_gpu_learned import _bf, _trainer_with  # noqa: E402


@pytest.mark.parametrize("n", [8, 32, 40, 56, 4104])
def test_an_overflowed_activation_in_the_last_row(n):
    """One activation of the last sample overflows.  Its sums are infinite, as that
    sample alone makes them; a tile's rows past the batch add nothing."""
    W1, W2 = np.zeros((mlp.N_H1, mlp.N_IN)), np.zeros((mlp.N_H2, mlp.N_H1))
    W1[:, 0] = 1.0                               # H1 = x0
    W2[np.arange(mlp.N_H2), np.arange(mlp.N_H2)] = 1.0
    W2[5, 5] = 4.0                               # H2 = x0, the sixth 4 x0
    W3 = np.full((3, mlp.N_H2), 2.0 ** -10)
    X = np.zeros((n, mlp.N_IN))
    X[:, 0] = 1.0
    X[-1, 0] = 2.0 ** 127
    tr = _trainer_with([W1, np.zeros(mlp.N_H1), W2, np.zeros(mlp.N_H2), W3, np.zeros(3)], n)
    tr.grads(_bf(X), torch.zeros(n, 2, device="cuda"))
    g = {k: v.cpu().numpy() for k, v in tr.g.items()}
    # o = (inf, inf, inf): the velocity errors' gradients are infinite in the last
    # row, the confidence's is its sigmoid's 1 / n
    assert np.isposinf(g["W3"][:2]).all() and np.isposinf(g["W3"][2, 5])
    assert np.isfinite(np.delete(g["W3"][2], 5)).all()
    assert np.isposinf(g["b3"][:2]).all() and np.isfinite(g["b3"][2])
    assert np.isposinf(g["b2"]).all()
