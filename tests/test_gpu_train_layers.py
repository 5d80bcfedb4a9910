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


def layer_by_layer(tr, X, lab):
    """Loss, gradients and the BF16 intermediates H1, dH2, dH1 of one batch, a call
    per layer; the head adds its sums to what its outputs hold."""
    b, n = tr.b, X.shape[0]
    bf = dict(dtype=torch.bfloat16, device="cuda")
    g = {k: torch.zeros_like(v) for k, v in tr.g.items()}
    loss = torch.zeros(1, device="cuda")
    H1, H2, dH2, dH1 = (torch.empty(n, m, **bf) for m in (mlp.N_H1, mlp.N_H2, mlp.N_H2, mlp.N_H1))

    def t(x):
        out = torch.empty(x.shape[1], x.shape[0], **bf)
        b.mlp_transpose(x, out)
        return out
    tr.forward(X, H1, H2)
    b.mlp_head(H2, tr.p["W3"], tr.p["b3"], lab, tr.wv, tr.half_step, dH2, g["W3"], g["b3"], loss)
    b.mlp_gemm_nt(t(dH2), t(H1), out_f32=g["W2"])                  # dW2 = dH2^T H1
    b.mlp_colsum(dH2, g["b2"])
    b.mlp_gemm_nt(dH2, t(tr.bf["W2"]), epi=2, aux=H1, out_bf16=dH1)   # dH1 = dH2 W2 where H1 > 0
    b.mlp_gemm_nt(t(dH1), t(X), out_f32=g["W1"])                   # dW1 = dH1^T X
    b.mlp_colsum(dH1, g["b1"])
    return loss, g, (H1, dH2, dH1)


@pytest.mark.parametrize("n", [8, 24, 64, 72, 200, 1096])
def test_the_layers_one_by_one(n):
    """The layer-by-layer calls inside the intervals derived for FP32 accumulation
    in any order, and their BF16 intermediates the bits that the three launches
    leave in their scratch (H1, dH2, dH1, each section on 256 bytes)."""
    from mlp_cases import random_params
    rng = np.random.default_rng(300 + n)
    X = mlp.bf16_round(rng.normal(size=(n, mlp.N_IN)))
    params = random_params(rng)
    O = mlp.forward(X, params)[-1]
    lab = np.float32(O[:, :2] + rng.choice([-1, 1], (n, 2)) * rng.choice([0.1, 0.5], (n, 1)))
    tr = _trainer_with(params, n)
    Xd, labd = _bf(X), torch.from_numpy(lab).cuda()
    loss, g, layers = layer_by_layer(tr, Xd, labd)
    (lm, lr), want = mlp.grads_iv(X, lab, params, wv=tr.wv, half_step=tr.half_step)
    assert mlp.within(float(loss.item()), lm, lr)
    for k, (mid, rad) in want.items():
        assert mlp.within(g[k].cpu().numpy().astype(np.float64), mid, rad).all(), k
    tr.grads(Xd, labd)
    at = 0
    for name, t in zip(("H1", "dH2", "dH1"), layers):
        nb = t.numel() * 2
        got = tr.buf["work"][at:at + nb].view(torch.int16)
        assert torch.equal(got, t.reshape(-1).view(torch.int16)), name
        at += (nb + 255) // 256 * 256
    if n > 64:
        return
    # the head's sums are added to what is there (one wavefront: one addition)
    H2, d = (torch.empty(n, mlp.N_H2, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    tr.forward(Xd, layers[0], H2)
    more = [torch.full_like(x, 3.0) for x in (g["W3"], g["b3"], loss)]
    tr.b.mlp_head(H2, tr.p["W3"], tr.p["b3"], labd, tr.wv, tr.half_step, d, *more)
    for x, y in zip(more, (g["W3"], g["b3"], loss)):
        assert torch.equal(x, 3.0 + y)


def test_a_trainer_without_batches():
    """A Trainer made for its weights alone."""
    from paper_1408_3526_amd import learned
    tr = learned.Trainer(seed=3, batch=0)
    assert tr.blob().size == mlp.N_H1 * mlp.N_IN + mlp.N_H1 + mlp.N_H2 * mlp.N_H1 + mlp.N_H2 + 3 * mlp.N_H2 + 3
