"""Epilogue of the streaming GEMMs (csrc/gemm_epilogue.h) where its pieces end: ranks around its steps of 16 and chunks of
64, ranks and channels that are no multiple of four, rows of tiles that are half empty or missing, plain, gated and with
nibble codes, against fp64."""
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


# tokens, K, N, rank
SHAPES = [(17, 512, 4096, 1), (32, 1024, 2050, 64), (33, 1024, 1999, 17), (64, 512, 33, 128), (65, 2048, 4100, 65),
          (96, 4096, 4096, 15), (97, 1024, 8200, 96), (200, 1024, 12288, 33), (256, 512, 6150, 4), (600, 2048, 11008, 48),
          (130, 1024, 4102, 0), (1024, 512, 5120, 100)]


@pytest.mark.parametrize("M,K,N,r", SHAPES)
def test_epilogue(M, K, N, r):
    from paper_2605_00422_amd import binding as B
    g = torch.Generator(device=DEV)
    g.manual_seed(M + N)
    W = torch.randn(N, K, device=DEV, generator=g)
    U = torch.randn(K, r, device=DEV, generator=g) if r else None
    V = torch.randn(N, r, device=DEV, generator=g).half().float() if r else None
    n1 = {512: 16, 1024: 32, 2048: 32, 4096: 64}[K]
    eye = lambda n: torch.eye(n, device=DEV)
    layer = B.pack_weights(W, eye(n1), eye(K // n1), U, V, n1, K // n1)
    sgn, alpha = B.unpack_signs(layer)
    act = B.Activations(layer, M)
    T64 = None
    if r:
        # rows of very different sizes, one of them zero
        act.T.normal_(generator=g)
        act.T.mul_(torch.exp2(torch.randint(-20, 20, (M, 1), device=DEV, generator=g).float()))
        act.T[M // 2] = 0
        T64 = act.T.double()
    act.scale.uniform_(0.01, 1.0, generator=g)
    for form in ("plain", "gated", "nibbles"):
        if form == "gated" and N % 2:
            continue
        top = 7 if form == "nibbles" else 31
        act.q.random_(-top, top + 1, generator=g)
        act.qsum.copy_(act.q.to(torch.int32).sum(1))
        acc = act.q.double() @ sgn.double().T
        main = act.scale.double()[:, None] * alpha.double()[None, :] * acc
        low = T64 @ V.double().T if r else torch.zeros_like(main)
        size = main.abs() + (T64.abs() @ V.double().abs().T if r else 0.0)
        # fp32: three roundings of the main term, T to 2^-22 in two terms, two additions per 16 ranks (and 16 products in each)
        steps = (r + 15) // 16
        bound = (24 + 2 * steps) * 2.0 ** -24 * size
        want = main + low
        if form == "plain":
            Y = torch.full((M, N), float("nan"), device=DEV)
            a = torch.full((M, N), -7, dtype=torch.int32, device=DEV)
            B.linear_forward(layer, act, Y, a)
            torch.cuda.synchronize()
            assert torch.equal(a.double(), acc)
            assert bool(((Y.double() - want).abs() <= bound).all())
        elif form == "nibbles":
            Y = torch.full((M, N), float("nan"), device=DEV)
            B.linear_forward_a4(layer, B.pack_codes_a4(act.q), act, Y)
            torch.cuda.synchronize()
            assert bool(((Y.double() - want).abs() <= bound).all())
        else:
            H = torch.full((M, N // 2), float("nan"), dtype=torch.bfloat16, device=DEV)
            B.linear_forward_swiglu(layer, act, H, None)
            torch.cuda.synchronize()
            gt, up = want[:, 0::2], want[:, 1::2]
            h = gt * torch.sigmoid(gt) * up
            # |d silu| <= 1.1 |d gate|; two bf16 units of the product, and 2^-20 for the exponential and the division
            b = 1.1 * bound[:, 0::2] * (up.abs() + bound[:, 1::2]) + (gt.abs() + 1e-30) * bound[:, 1::2] + (2.0 ** -8 + 2.0 ** -20) * h.abs() + 1e-30
            assert bool(((H.double() - h).abs() <= b).all())
