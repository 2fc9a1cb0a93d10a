"""The output stages around the widths where they change: remainders of 4, 64, 64 * 4 and 1024
columns, the widest row held in registers and the first beyond; a number of patterns that is no multiple of the rows of a workgroup; ignored
labels; biases so large that a softmax saturates.  Against 64 bits: relative 2-norm 1e-5, loss 1e-6 per pattern."""
import pytest
import torch

import paper_1911_05181_amd as ulsnn
import synth_inputs as si

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("n_out", [1, 3, 13, 63, 64, 65, 254, 255, 256, 257, 1023, 1024, 1025, 4095, 4096, 4097])
def test_output_stage(n_out, dense):
    n_in, n_hid, batch = 7, 70, 21
    net = si.MlpShape(n_in, n_hid, n_out, True)
    W1, W2, _, _ = si.mlp_weights(net, 8, device=DEV)
    b1, b2 = si.random_biases(net, 8, device=DEV)
    X, y = si.mlp_patterns(net, 8, 0, batch, device=DEV)
    T = si.mlp_targets(net, 8, 0, batch, device=DEV)
    y[1], y[2], y[3], y[20] = n_out - 1, -1, n_out, 0
    b2[n_out - 1] = 60.0                                   # the last column takes nearly all of the softmax
    w2 = W2.double()
    H = torch.tanh(X.double() @ W1.double() + b1.double())
    Z = H @ w2 + b2.double()
    if dense:
        Y = torch.tanh(Z)
        D = Y - T.double()
        loss, D = D.square().sum(), 2 * D * (1 - Y * Y)
        res = ulsnn.mlp_grad_mse(W1, W2, X, T, b1, b2)
        only = ulsnn.mlp_mse(W1, W2, X, T, b1, b2)
    else:
        live = (y >= 0) & (y < n_out)
        L = torch.log_softmax(Z, 1)
        at = torch.arange(batch, device=DEV)[live]
        loss, D = -L[at, y[live].long()].sum(), L.exp()
        D[at, y[live].long()] -= 1
        D[~live] = 0
        res = ulsnn.mlp_grad(W1, W2, X, y, b1, b2)
        only = ulsnn.mlp_loss(W1, W2, X, y, b1, b2)
    assert torch.equal(only, res.loss)
    assert abs(res.loss.double().item() - loss.item()) <= 1e-6 * (abs(loss.item()) + batch)
    for got, want in ((res.db2, D.sum(0)), (res.dW2, H.t().contiguous() @ D)):
        assert (got.double() - want).norm() <= 1e-5 * want.norm()          # (a single class: both are zero)


@pytest.mark.parametrize("n_in,n_hid,n_out,batch", [(33, 200, 40, 1986), (402, 64, 100, 300), (333, 70, 33, 1000), (65, 20, 40, 127), (9, 20, 40, 128), (777, 3, 5, 400)])
@pytest.mark.parametrize("dense", [False, True])
def test_bf16_patterns_with_unaligned_rows(n_in, n_hid, n_out, batch, dense):
    """Rows of X that are not 16-byte aligned are copied into aligned ones, by a gradient from 128 rows on and by an error
    alone above 64 columns, where the workspace holds them (not for the last shape, much wider than its hidden layer).  The
    copy changes no sum: the loss is the same bits either way.  bf16 operands: 1e-2."""
    net = si.MlpShape(n_in, n_hid, n_out, True)
    W1, W2, _, _ = si.mlp_weights(net, 9, device=DEV)
    b1, b2 = si.random_biases(net, 9, device=DEV)
    X, y = si.mlp_patterns(net, 9, 0, batch, device=DEV)
    T = si.mlp_targets(net, 9, 0, batch, device=DEV)
    W1, W2, X = (t.to(torch.bfloat16) for t in (W1, W2, X))
    w2, x = W2.double(), X.double()
    H = torch.tanh(x @ W1.double() + b1.double())
    Z = H @ w2 + b2.double()
    if dense:
        Y = torch.tanh(Z)
        D = 2 * (Y - T.double()) * (1 - Y * Y)
    else:
        D = torch.softmax(Z, 1)
        D[torch.arange(batch, device=DEV), y.long()] -= 1
    dA = (D @ w2.t().contiguous()) * (1 - H * H)
    res = (ulsnn.mlp_grad_mse if dense else ulsnn.mlp_grad)(W1, W2, X, T if dense else y, b1, b2)
    for got, want in ((res.dW1, x.t().contiguous() @ dA), (res.dW2, H.t().contiguous() @ D)):
        assert ((got.double() - want).norm() / want.norm()).item() <= 1e-2
    only = (ulsnn.mlp_mse if dense else ulsnn.mlp_loss)(W1, W2, X, T if dense else y, b1, b2)
    assert torch.equal(only, res.loss)
