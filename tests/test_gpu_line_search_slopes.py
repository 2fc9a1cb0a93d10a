"""The slopes of a group of steps from one stacked product, at the limits of its workspace: all eight steps of a group at
once, two at a time, and none (the subset is the whole batch of a wide output layer: gradients instead).  The bracket is
decided by the slopes' signs alone, so it must be the oracle's."""
import numpy as np
import pytest
import torch

import oracle
import paper_1911_05181_amd as ulsnn
import synth_inputs as si
from oracle import ref_cg

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("shape,batch,bracket", [((33, 17, 5), 130, 40), ((100, 130, 259), 700, 65), ((40, 30, 300), 500, 500),
                                                 ((20, 8, 1500), 600, 600)])
@pytest.mark.parametrize("alpha0", [1e-5, 1e-3])
@pytest.mark.parametrize("ignored", [False, True])
def test_bracket_is_the_oracles(shape, batch, bracket, alpha0, ignored):
    net = si.MlpShape(*shape, False)
    W1, W2, _, _ = si.mlp_weights(net, 6)
    X, y = si.mlp_patterns(net, 6, 0, batch)
    if ignored:
        y = y.clone()
        y[::7] = -1
        y[3::11] = net.n_out
    g = oracle.mlp_grad(W1.numpy(), W2.numpy(), X.numpy(), y.numpy())
    d1, d2 = (torch.from_numpy((-v).astype(np.float32)) for v in (g.dW1, g.dW2))
    want, _, _ = ref_cg.mlp_line_search(W1.numpy(), W2.numpy(), d1.numpy(), d2.numpy(), X.numpy(), y.numpy(), bracket, alpha0, 25)
    res = ulsnn.mlp_line_search(W1.to(DEV), W2.to(DEV), d1.to(DEV), d2.to(DEV), X.to(DEV), y.to(DEV), bracket, alpha0, 25)
    assert res.bracket_lo == np.float32(want.lo) and res.bracket_hi == np.float32(want.hi)
    assert res.gradient_evaluations == want.gradient_evaluations
    assert abs(res.loss0 - want.loss0) <= 1e-5 * want.loss0 and abs(res.loss - want.loss) <= 1e-5 * want.loss


@pytest.mark.parametrize("n_out", [5, 9, 65])
def test_a_class_whose_logits_are_minus_infinity(n_out):
    """The last class's logits overflow to -inf at every step: its probability is 0, and the slopes are those of the other
    classes.  It is the only column of its lane's vector (n_out = 4 q + 1), where nothing else sets a maximum."""
    n_in, n_hid, batch = 12, 40, 64
    net, whole = si.MlpShape(n_in, n_hid, n_out - 1, False), si.MlpShape(n_in, n_hid, n_out, False)
    W1, W2, _, _ = si.mlp_weights(whole, 6)
    X, y = si.mlp_patterns(net, 6, 0, batch)
    W1, X = W1.abs(), X.abs()                                                # H > 0 everywhere
    g = oracle.mlp_grad(W1.numpy(), W2[:, :-1].contiguous().numpy(), X.numpy(), y.numpy())
    d1 = torch.zeros_like(W1)                                                # the direction leaves H alone
    d2 = torch.zeros_like(W2)
    d2[:, :-1] = torch.from_numpy((-g.dW2).astype(np.float32))
    want, _, _ = ref_cg.mlp_line_search(W1.numpy(), W2[:, :-1].contiguous().numpy(), d1.numpy(), d2[:, :-1].contiguous().numpy(),
                                        X.numpy(), y.numpy(), batch, 1e-4, 25)
    W2 = W2.clone()
    W2[:, -1] = -3.0e38
    res = ulsnn.mlp_line_search(W1.to(DEV), W2.to(DEV), d1.to(DEV), d2.to(DEV), X.to(DEV), y.to(DEV), batch, 1e-4, 25)
    assert res.bracket_lo == np.float32(want.lo) and res.bracket_hi == np.float32(want.hi)
    assert res.gradient_evaluations == want.gradient_evaluations
    assert abs(res.loss - want.loss) <= 1e-5 * want.loss
