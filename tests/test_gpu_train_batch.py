"""rmdf_mlp_grads at the edges of its split: tiles of 32 samples, steps of 64,
at most 16 chunks of the batch (a partly filled last tile, step and chunk, one
of each, and more than one step per chunk).  On integer data every FP32 sum is
exact in any order, so the gradients equal the FP64 reference bit for bit; on
random data every element lies inside the interval derived for FP32
accumulation in any order with BF16 rounding of the stored activations."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import mlp  # noqa: E402
from mlp_cases import exactness_premise, integer_case, random_params  # noqa: E402
from test_gpu_learned import _bf, _trainer_with  # noqa: E402

KEYS = ("W1", "b1", "W2", "b2", "W3", "b3")


@pytest.mark.parametrize("n", [8, 32, 64, 128, 1024, 2048])
def test_exact_on_integer_data(n):
    X, lab, params = integer_case(seed=n, n=n)
    assert exactness_premise(X, lab, params, n) < 1.0
    tr = _trainer_with(params, n)
    tr.grads(_bf(X), torch.from_numpy(np.asarray(lab, np.float32)).cuda())
    torch.cuda.synchronize()
    _, rg = mlp.loss_and_grads(X, lab, params, wv=tr.wv, half_step=tr.half_step, bf16=True)
    for k, G in zip(KEYS, rg):
        assert np.array_equal(tr.g[k].cpu().numpy().astype(np.float64), G), k


@pytest.mark.parametrize("n,batch", [(8, 8), (24, 64), (40, 40), (72, 72), (1096, 1096)])
def test_random_data_within_bounds(n, batch):
    rng = np.random.default_rng(n)
    X = mlp.bf16_round(rng.normal(size=(n, mlp.N_IN)))
    params = random_params(rng)
    O = mlp.forward(X, params)[-1]
    lab = np.float32(O[:, :2] + rng.choice([-1, 1], (n, 2)) * rng.choice([0.1, 0.5], (n, 1)))
    tr = _trainer_with(params, batch)
    loss = tr.grads(_bf(X), torch.from_numpy(lab).cuda())
    (lm, lr), g = mlp.grads_iv(X, lab, params, wv=tr.wv, half_step=tr.half_step)
    assert mlp.within(float(loss.item()), lm, lr)
    for k, (mid, rad) in g.items():
        assert mlp.within(tr.g[k].cpu().numpy().astype(np.float64), mid, rad).all(), k


def test_refused_batches():
    from paper_1408_3526_amd import binding as b
    rng = np.random.default_rng(1)
    tr = _trainer_with(random_params(rng), 64)
    X, lab = _bf(rng.normal(size=(12, mlp.N_IN))), torch.zeros(12, 2, device="cuda")
    with pytest.raises(b.RmdfError):            # not a multiple of 8
        tr.grads(X, lab)
    tr.buf["work"] = tr.buf["work"][:256]
    with pytest.raises(b.RmdfError):            # scratch too small
        tr.grads(_bf(rng.normal(size=(64, mlp.N_IN))), torch.zeros(64, 2, device="cuda"))
