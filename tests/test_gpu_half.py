"""The two-term f16 split behind ulsnn_sgemm (gemm_half.hpp): every tile on ragged edges in every layout, operands outside
the range of f16, and its error beside the fp32 instruction's.

Bars: integers (|values| <= 8: one f16 term, partial sums below 2^24) bit for bit; real values against 64 bits, element by
element 1e-5 of the sum of absolute terms, as for every gradient (a lost term of an element shows as 2^-12 or more of it)."""
import itertools

import pytest
import torch

import paper_1911_05181_amd as ulsnn

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# k of at least 128 goes through the f16 terms; with a partial last step of 32
TILES = {"256x256": (3841, 3203, 141), "256x128": (1000, 4353, 301), "128x128w8": (700, 3203, 301), "128x128": (1921, 4353, 141),
         "128x64": (1000, 1729, 521), "64x128": (1921, 890, 521), "64x64": (300, 4353, 521)}


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _stored(X, transposed, pad):
    X = X.t() if transposed else X
    W = torch.full((X.shape[0], X.shape[1] + pad), float("nan"), device=DEV)
    W[:, :X.shape[1]] = X
    return W


def _sgemm(ta, tb, A, B, pad=0):
    (m, k), n = A.shape, B.shape[1]
    a, b = _stored(A, ta == "T", pad), _stored(B, tb == "T", pad)
    C = torch.full((m, n + pad), float("nan"), device=DEV)
    ulsnn.sgemm(ta, tb, m, n, k, 1.0, a, a.shape[1], b, b.shape[1], 0.0, C, n + pad)
    assert torch.isnan(C[:, n:]).all()
    return C[:, :n]


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("ta,tb", list(itertools.product("NT", "NT")))
def test_integers_on_ragged_edges(tile, ta, tb):
    m, n, k = TILES[tile]
    assert ulsnn.sgemm_describe_plan("N", "N", m, n, k).startswith(f"tile={tile} ")
    g = _gen(1)
    A, B = (torch.randint(-8, 9, s, generator=g, device=DEV).float() for s in ((m, k), (k, n)))
    assert torch.equal(_sgemm(ta, tb, A, B, 3).double(), A.double() @ B.double())


def _operands(kind, m, n, k):
    g = _gen(2)
    A, B = torch.randn(m, k, generator=g, device=DEV), torch.randn(k, n, generator=g, device=DEV)
    if kind == "single small elements":           # rows and columns whose only element is 2^-23 and 2^-45 of the others
        for at, e in ((5, -23), (m // 2, -45)):
            A[at], A[at, 7 * at % k] = 0, 1.3 * 2.0 ** e
        B[:, n - 2] = 0
        B[k - 1, n - 2] = 1.7 * 2.0 ** -23
    elif kind == "scaled against each other":     # A D and D^-1 B with powers of two: the same products
        d = 2.0 ** torch.randint(-25, 26, (k,), generator=g, device=DEV).float()
        A, B = A * d, B / d[:, None]
    elif kind == "mildly scaled":
        d = 2.0 ** torch.randint(-8, 9, (k,), generator=g, device=DEV).float()
        A, B = A * d, B / d[:, None]
    elif kind == "zeros first":                   # nothing to take a scale from in the first step
        A[:, :70], B[:35] = 0, 0
    elif kind == "large elements":                # beyond f16 for the scale of the others, in the last step and alone
        A[:, k - 3] *= 1e7
        B[k - 3] *= 1e-7
        A[m - 1, 40], B[60, n - 1] = 3e8, -2e9
    elif kind == "scaled rows":
        A *= 10.0 ** torch.linspace(-9, 9, m, device=DEV)[:, None]
    elif kind == "tiny and huge":
        A, B = A * 2.0 ** -120, B * 2.0 ** 100
    return A, B


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("kind", ["normal", "single small elements", "scaled against each other", "mildly scaled", "zeros first",
                                  "large elements", "scaled rows", "tiny and huge"])
def test_operands_of_any_range(tile, kind):
    m, n, k = TILES[tile]
    A, B = _operands(kind, m, n, k)
    got = _sgemm("N", "N", A, B).double()
    A, B = A.double(), B.double()
    err, terms = (got - A @ B).abs(), A.abs() @ B.abs()
    assert (err <= 1e-5 * terms).all(), float((err / terms).nan_to_num().max())


@pytest.mark.parametrize("tile", TILES)
def test_infinities_and_nan(tile):
    m, n, k = TILES[tile]
    A, B = _operands("normal", m, n, k)
    A[3, k - 1], B[40, n - 5] = float("inf"), float("nan")
    got, want = _sgemm("N", "N", A, B).double(), A.double() @ B.double()
    assert torch.equal(torch.isnan(got), torch.isnan(want)) and torch.equal(got.isinf(), want.isinf())
    fine = torch.isfinite(want)
    assert ((got - want).abs()[fine] <= 1e-5 * (A.abs().double() @ B.abs().double())[fine]).all()


@pytest.mark.parametrize("kind", ["normal", "one sign", "tanh and deltas"])
@pytest.mark.parametrize("k", [128, 480, 3203])
def test_error_beside_the_fp32_instructions(k, kind):
    """The 2-norm of the error against 64 bits, beside that of v_mfma_f32_32x32x2_f32 on the same operands."""
    m = n = 1024
    g = _gen(k)
    A, B = torch.randn(m, k, generator=g, device=DEV), torch.randn(k, n, generator=g, device=DEV)
    if kind == "one sign":
        A, B = A.abs(), B.abs()
    elif kind == "tanh and deltas":
        A, B = torch.tanh(A), torch.softmax(B, 1)
        B[torch.arange(k, device=DEV), torch.randint(0, n, (k,), generator=g, device=DEV)] -= 1
    want = A.double() @ B.double()
    C = torch.empty(m, n, device=DEV)
    ulsnn.sgemm_planned(1, 1, "N", "N", m, n, k, 1.0, A, k, B, n, 0.0, C, n)
    here, instruction = ((x.double() - want).norm() / want.norm() for x in (_sgemm("T", "N", A, B), C))
    print(f"{kind}, k = {k}: {here.item():.2e}, fp32 instruction {instruction.item():.2e}")
    assert here <= instruction


def test_gradient_of_confident_patterns():
    """Probabilities over 40 orders of magnitude: most steps of both products of the deltas leave the range of f16."""
    n_in, n_hid, n_out, batch = 300, 400, 900, 2500
    g = _gen(5)
    W1 = torch.randn(n_in, n_hid, generator=g, device=DEV) / n_in ** 0.5
    W2 = 4.0 * torch.randn(n_hid, n_out, generator=g, device=DEV) / n_hid ** 0.5 * 5.0
    X, y = torch.randn(batch, n_in, generator=g, device=DEV), torch.randint(0, n_out, (batch,), generator=g, device=DEV, dtype=torch.int32)
    res = ulsnn.mlp_grad(W1, W2, X, y)
    H = torch.tanh(X.double() @ W1.double())
    D = torch.softmax(H @ W2.double(), 1)
    D[torch.arange(batch, device=DEV), y.long()] -= 1
    dA = (D @ W2.double().t().contiguous()) * (1 - H * H)
    for got, want in ((res.dW2, H.t().contiguous() @ D), (res.dW1, X.double().t().contiguous() @ dA)):
        assert (got.double() - want).norm() <= 1e-5 * want.norm()
