"""The tiles of the bf16 products with steps of 64 k (wide16_kernel) where they can go wrong: a partial k step in every product, ragged
last tiles, k slices, logits far from zero, labels outside the classes, patterns whose rows are not 16-byte aligned; and the 256 x 256
tile with steps of 32 k, for such patterns where no copy of them fits into the workspace.

Bar: relative L2 1e-2 per tensor, as for every bf16 gradient: H, the output delta and the hidden delta are rounded to bf16
(2^-9 relative each, so about 3.4e-3 where the three do not average out); three of 3203 classes lost would be 3e-2.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1911_05181_amd as ulsnn
import synth_inputs as si

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = 1e-2


def _rel(a, b):
    return np.linalg.norm(a.cpu().numpy().astype(np.float64) - b) / np.linalg.norm(b)


def _np(t):
    return None if t is None else t.float().numpy()


def _dev(t):
    return None if t is None else t.to(DEV)


@pytest.mark.parametrize("n_in,n_hid,n_out,batch,dense", [
    (1030, 1100, 1500, 9000, False),    # all five products on these tiles; k = 1030, 1100, 1500, 9000: all with a remainder
    (1030, 1100, 1500, 4097, True),
    (1088, 1088, 1536, 8192, False),    # no remainder anywhere
    (300, 1300, 2051, 8191, False),     # both backward products of the output layer, remainders 3 and 63
    (400, 480, 3203, 16384, False),     # hidden delta in k slices
    (400, 480, 3203, 2047, False),      # the 128 x 128 tile for hidden delta and dW2, both in k slices
    (1024, 520, 1003, 5001, True),      # ... and for hidden and output layer
    (72, 1000, 40, 6001, True),         # a product shorter than a step
])
def test_gradient(n_in, n_hid, n_out, batch, dense):
    shape = si.MlpShape(n_in, n_hid, n_out, True)
    W1, W2, _, _ = si.mlp_weights(shape, 3)
    b1, b2 = si.random_biases(shape, 3, 0.2)
    X, y = si.mlp_patterns(shape, 3, 0, batch)
    W1, W2, X = W1.bfloat16(), W2.bfloat16(), X.bfloat16()
    weights = (_dev(W1), _dev(W2), _dev(X))
    if dense:
        t = torch.tanh(torch.randn(batch, n_out, generator=torch.Generator().manual_seed(3)))
        ref = oracle.mlp_grad_mse(_np(W1), _np(W2), _np(X), _np(t), _np(b1), _np(b2))
        call = lambda: ulsnn.mlp_grad_mse(*weights, _dev(t), _dev(b1), _dev(b2))
    else:
        y[[0, 5, batch - 1]] = torch.tensor([-1, n_out, 2 ** 30], dtype=y.dtype)      # no class: no gradient
        y[1:5] = torch.tensor([0, n_out - 1, 63, 64], dtype=y.dtype)
        ref = oracle.mlp_grad(_np(W1), _np(W2), _np(X), y.numpy(), _np(b1), _np(b2))
        call = lambda: ulsnn.mlp_grad(*weights, _dev(y), _dev(b1), _dev(b2))
    res, again = call(), call()
    torch.cuda.synchronize()
    errors = {name: _rel(getattr(res, name), getattr(ref, name)) for name in ("dW1", "dW2", "db1", "db2")}
    errors["loss"] = abs(res.loss.item() - ref.loss) / abs(ref.loss)
    print(n_in, n_hid, n_out, batch, {k: f"{e:.1e}" for k, e in errors.items()})
    assert max(errors.values()) <= TOL, errors
    for name in ("dW1", "dW2", "db1", "db2", "loss"):
        assert torch.equal(getattr(res, name), getattr(again, name)), name


def test_far_logits_and_a_partial_step():
    """All logits -128 (exact in bf16): exp(-log sum exp) overflows, so classes beyond the last must not form a delta."""
    shape = si.MlpShape(300, 1300, 2051, True)
    W1, W2, b1, _ = si.mlp_weights(shape, 3)
    X, y = si.mlp_patterns(shape, 3, 0, 8191)
    W1, W2, X, b2 = W1.bfloat16(), torch.zeros_like(W2).bfloat16(), X.bfloat16(), torch.full((2051,), -128.0)
    ref = oracle.mlp_grad(_np(W1), _np(W2), _np(X), y.numpy(), _np(b1), _np(b2))
    res = ulsnn.mlp_grad(_dev(W1), _dev(W2), _dev(X), _dev(y), _dev(b1), _dev(b2))
    torch.cuda.synchronize()
    assert not res.dW1.any() and not res.db1.any()
    assert _rel(res.dW2, ref.dW2) <= TOL and _rel(res.db2, ref.db2) <= TOL


@pytest.mark.parametrize("n_in,n_hid,n_out,batch", [
    (785, 251, 10, 45001),      # hidden layer and dW1, the latter in k slices; 785 = 3 * 256 + 17, 45001 = 32 * 1406 + 9
    (6001, 1500, 10, 5700),     # dW1 in one slice
    (785, 251, 40, 70001),      # two passes over the patterns: the second adds to the first's dW1
    (1017, 72, 10, 45001),      # a narrow hidden layer: 64 x 64 tiles of it, 128 x 128 of dW1
    (1017, 34, 31, 68383),      # 64 x 64 tiles of both, dW1 in 64 slices; the second pass is copied
])
def test_unaligned_patterns_that_are_not_copied(n_in, n_hid, n_out, batch):
    """Rows of an odd number of bf16 elements, too many for an aligned copy (it would have to fit into half of the slices' region
    of the workspace, 64 MB here)."""
    assert min(batch, 65536) * (n_in + 7) * 2 > 64 << 20
    g = torch.Generator(device=DEV).manual_seed(3)
    W1 = (torch.randn(n_in, n_hid, generator=g, device=DEV) / n_in ** 0.5).bfloat16()
    W2 = (torch.randn(n_hid, n_out, generator=g, device=DEV) / n_hid ** 0.5).bfloat16()
    X = torch.randn(batch, n_in, generator=g, device=DEV).bfloat16()
    y = torch.randint(0, n_out, (batch,), generator=g, device=DEV, dtype=torch.int32)
    res, again = ulsnn.mlp_grad(W1, W2, X, y), ulsnn.mlp_grad(W1, W2, X, y)
    H = torch.tanh(X.double() @ W1.double())
    L = torch.log_softmax(H @ W2.double(), 1)
    D = L.exp()
    D[torch.arange(batch, device=DEV), y.long()] -= 1
    dA = (D @ W2.double().t().contiguous()) * (1 - H * H)
    for got, want in ((res.dW1, X.double().t().contiguous() @ dA), (res.dW2, H.t().contiguous() @ D)):
        assert (got.double() - want).norm() <= TOL * want.norm()
    loss = -L[torch.arange(batch, device=DEV), y.long()].sum()
    assert abs(res.loss.double() - loss) <= TOL * loss
    assert torch.equal(ulsnn.mlp_loss(W1, W2, X, y), res.loss)
    assert torch.equal(res.dW1, again.dW1) and torch.equal(res.dW2, again.dW2)
