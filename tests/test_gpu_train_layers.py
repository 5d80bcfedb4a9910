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


def test_batches_of_another_shape_are_refused():
    """Operands that the kernels would read or write out of range, or take for
    something else, are refused on the host before any launch."""
    from paper_1408_3526_amd import binding as b
    from mlp_cases import random_params
    rng = np.random.default_rng(2)
    n = 64
    tr = _trainer_with(random_params(rng), n)
    X, lab = _bf(rng.normal(size=(n, mlp.N_IN))), torch.zeros(n, 2, device="cuda")
    tr.grads(X, lab)
    want = {k: v.clone() for k, v in tr.g.items()}
    wide = torch.zeros(n, 2 * mlp.N_IN, dtype=torch.bfloat16, device="cuda")
    flat = torch.zeros(n * mlp.N_IN, dtype=torch.bfloat16, device="cuda")
    for bad in (X[:, :1144].contiguous(), wide, flat, wide[:, :mlp.N_IN], wide[:, ::2], X.float(), X.half(), X.cpu()):
        with pytest.raises((TypeError, ValueError)):
            tr.grads(bad, lab)
    for bad in (lab[:n - 1], torch.zeros(n, device="cuda"), torch.zeros(n, 4, device="cuda")[:, :2], lab.double(), lab.cpu()):
        with pytest.raises((TypeError, ValueError)):
            tr.grads(X, bad)
    p, bf, buf = tr.p, tr.bf, tr.buf

    def call(**other):
        a = dict(W1=bf["W1"], b1=p["b1"], W2=bf["W2"], b2=p["b2"], W3=p["W3"], b3=p["b3"], loss=buf["loss"],
                 work=buf["work"], grads=tr.g)
        a.update(other)
        b.mlp_grads(X, lab, a["W1"], a["b1"], a["W2"], a["b2"], a["W3"], a["b3"], tr.wv, tr.half_step, a["grads"],
                    a["loss"], a["work"])
    for k in ("W1", "W2"):
        for bad in (p[k], bf[k][:-1], bf[k].t(), bf[k].cpu()):
            with pytest.raises((TypeError, ValueError)):
                call(**{k: bad})
    for k in ("b1", "b2", "W3", "b3"):
        for bad in (p[k][:-1], p[k].double(), p[k].cpu()):
            with pytest.raises((TypeError, ValueError)):
                call(**{k: bad})
    for k in tr.g:
        for bad in (tr.g[k][:-1], tr.g[k].double(), tr.g[k].cpu()):
            with pytest.raises((TypeError, ValueError)):
                call(grads=dict(tr.g, **{k: bad}))
    for bad in (buf["loss"].double(), buf["loss"].cpu()):
        with pytest.raises((TypeError, ValueError)):
            call(loss=bad)
    for bad in (buf["work"].view(torch.float32), buf["work"].cpu()):
        with pytest.raises((TypeError, ValueError)):
            call(work=bad)
    # nothing was launched, and more labels than samples are taken as before
    assert all(torch.equal(tr.g[k], want[k]) for k in want)
    tr.grads(X, torch.zeros(2 * n, 2, device="cuda"))
    assert all(torch.equal(tr.g[k], want[k]) for k in want)


@pytest.mark.parametrize("off", [1, 4, 7])
def test_features_at_any_address(off):
    """Contiguous features that begin at an address no multiple of 16 bytes."""
    from mlp_cases import random_params
    rng = np.random.default_rng(off)
    n = 40
    tr = _trainer_with(random_params(rng), n)
    X, lab = _bf(rng.normal(size=(n, mlp.N_IN))), torch.from_numpy(rng.normal(size=(n, 2)).astype(np.float32)).cuda()
    loss = tr.grads(X, lab).clone()
    want = {k: v.clone() for k, v in tr.g.items()}
    flat = torch.empty(off + n * mlp.N_IN, dtype=torch.bfloat16, device="cuda")
    view = flat[off:].view(n, mlp.N_IN)
    view.copy_(X)
    assert view.data_ptr() % 16 == 2 * off
    assert torch.equal(tr.grads(view, lab), loss)
    assert all(torch.equal(tr.g[k], want[k]) for k in want)
