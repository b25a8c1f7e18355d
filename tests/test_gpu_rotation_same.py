"""A token's codes and scale do not depend on which kernel rotates it: the rotation by strips (csrc/rotate_terms.hip) against the
kernels it stands in for, bit by bit.  A pair is led past it by columns of zeros: R2 in the corner of a larger identity, which
adds exact zeros to every sum."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_00422_amd import binding as B
    B.load()


def _tokens(g, M, K, x):
    """Every third token with one channel 1e8 above the others: nothing averages the error of its one large product out."""
    X = torch.randn(M, K, device=DEV, generator=g)
    X[::3, 5] = 1e8
    return X.to(torch.bfloat16) if x == "bf16" else X


def _rotate(X, R1, R2, bits, asym=False):
    from paper_2605_00422_amd import binding as B
    M, n1, n2 = X.shape
    layer = B.pack_weights(torch.ones(16, n1 * n2, device=DEV), R1, R2, None, None, n1, n2, asym=asym)
    act = B.Activations(layer, M)
    B.rotate_quant(layer, X.reshape(M, n1 * n2).contiguous(), act, bits)
    torch.cuda.synchronize()
    return act.q.view(M, n1, n2), act.scale


# bf16 tokens against rows of odd length (of n1 above 128: longer than 128), fp32 tokens against rows of 100.  (80 tokens: past
# those that are split)
@pytest.mark.parametrize("x,M,n1,n2,wide", [
    ("bf16", 9, 32, 16, 17), ("bf16", 600, 32, 46, 47), ("bf16", 30, 64, 80, 81), ("bf16", 600, 64, 80, 81),
    ("bf16", 80, 128, 64, 65), ("bf16", 80, 128, 86, 87), ("bf16", 300, 128, 86, 87), ("bf16", 700, 96, 96, 97),
    ("bf16", 120, 160, 112, 132), ("bf16", 300, 160, 112, 132),
    ("f32", 5, 16, 32, 100), ("f32", 40, 48, 64, 100), ("f32", 300, 64, 80, 100), ("f32", 20, 128, 86, 100),
    ("f32", 600, 128, 96, 100), ("f32", 17, 8, 12, 100)])
@pytest.mark.parametrize("asym", [False, True])
def test_the_kernels_it_stands_in_for(x, M, n1, n2, wide, asym):
    g = torch.Generator(device=DEV)
    g.manual_seed(M + n1 * n2)
    R1, R2 = (torch.linalg.qr(torch.randn(n, n, device=DEV, generator=g))[0].contiguous() for n in (n1, n2))
    X = _tokens(g, M, n1 * n2, x).view(M, n1, n2)
    Xw, R2w = torch.zeros(M, n1, wide, device=DEV, dtype=X.dtype), torch.eye(wide, device=DEV)
    Xw[:, :, :n2], R2w[:n2, :n2] = X, R2
    bits = 7 if asym else 8
    q, s = _rotate(X, R1, R2, bits, asym)
    qw, sw = _rotate(Xw, R1, R2w, bits, asym)
    assert torch.equal(s, sw)
    assert torch.equal(q, qw[:, :, :n2])


@pytest.mark.parametrize("M,n1,n2", [(256, 128, 64), (257, 128, 64), (511, 128, 64), (300, 96, 148)])
def test_another_number_of_tokens(M, n1, n2):
    """The tokens of a call with a token or two a CU, and the same among more of them: 128 x 64 by rotate_planes.hip then, 96 x 148
    by rotate_bf16_device.h before."""
    g = torch.Generator(device=DEV)
    g.manual_seed(M)
    R1, R2 = (torch.linalg.qr(torch.randn(n, n, device=DEV, generator=g))[0].contiguous() for n in (n1, n2))
    X = _tokens(g, 600, n1 * n2, "bf16").view(600, n1, n2)
    q, s = _rotate(X[:M], R1, R2, 8)
    qm, sm = _rotate(X, R1, R2, 8)
    assert torch.equal(s, sm[:M]) and torch.equal(q, qm[:M])


@pytest.mark.parametrize("M,n1,n2", [(3, 16, 32), (20, 64, 64), (300, 64, 80), (5, 128, 86)])
def test_an_infinite_fp32_value_is_not_lost(M, n1, n2):
    """The step of a token with an infinite value is infinite, and so is its result; no other token knows of it."""
    from paper_2605_00422_amd import binding as B
    g = torch.Generator(device=DEV)
    g.manual_seed(M)
    K = n1 * n2
    R1, R2 = (torch.linalg.qr(torch.randn(n, n, device=DEV, generator=g))[0].contiguous() for n in (n1, n2))
    layer = B.pack_weights(torch.randn(32, K, device=DEV, generator=g), R1, R2, None, None, n1, n2)
    X = torch.randn(M, K, device=DEV, generator=g)
    want = B.decode_forward(layer, X, B.Activations(layer, M), torch.empty(M, 32, device=DEV)).clone()
    X[1, 7] = float("inf")
    act = B.Activations(layer, M)
    Y = B.decode_forward(layer, X, act, torch.empty(M, 32, device=DEV))
    torch.cuda.synchronize()
    assert torch.isinf(act.scale[1]) and not torch.isfinite(Y[1]).any()
    rest = torch.arange(M, device=DEV) != 1
    assert torch.equal(Y[rest], want[rest])
