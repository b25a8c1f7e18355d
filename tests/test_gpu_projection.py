"""T = X U where the projection has a launch of its own in front of the rotation and leaves partial tiles that workgroups
behind the rotation's own add up (and beside that range, where it rides in the rotation launch or hands its sums over),
for every rotation kernel that carries such workgroups: against fp64."""
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


# (tokens, n1, n2, rank, type)
CASES = [
    (192, 64, 80, 96, "bf16"),      # one token a workgroup; two column groups, the second of 32
    (300, 64, 80, 33, "bf16"),      # tokens in a loop; a rank that is no multiple of four
    (300, 128, 86, 20, "bf16"),
    (129, 192, 128, 64, "bf16"),    # factors streamed; one token in the last tile
    (256, 64, 64, 64, "bf16"),      # the kernel that walks over the tokens, from its first size on
    (257, 128, 64, 1, "bf16"),
    (700, 160, 160, 8, "bf16"),
    (1792, 224, 128, 17, "bf16"),   # the largest that leaves its tiles
    (1793, 128, 64, 17, "bf16"),    # the first that hands them over
    (384, 64, 64, 128, "f32"),      # fp32 tokens
    (1000, 128, 64, 31, "f32"),
    (255, 64, 32, 8, "bf16"),       # rides
    (257, 64, 80, 8, "bf16"),       # rides in the shadow of the second round
    (768, 137, 32, 20, "bf16"),     # factors that the fp32 kernel rotates: the largest that leaves its tiles
    (769, 137, 32, 20, "bf16"),     # and the first that hands them over
    (185, 172, 64, 8, "bf16"),      # a slow rotation, in whose shadow it rides
    (158, 163, 32, 64, "bf16"),     # likewise, by the fp32 kernel
    (192, 80, 64, 37, "f32"),       # fp32 tokens ride by the number of workgroups
    (384, 64, 64, 37, "f32"),
]


@pytest.mark.parametrize("M,n1,n2,r,x", CASES)
def test_projection(M, n1, n2, r, x):
    from paper_2605_00422_amd import binding as B
    K, N = n1 * n2, 64
    g = torch.Generator(device=DEV)
    g.manual_seed(M + K + r)
    W = torch.randn(N, K, device=DEV, generator=g)
    U = torch.randn(K, r, device=DEV, generator=g).half().float()
    V = torch.randn(N, r, device=DEV, generator=g).half().float()
    R = [torch.linalg.qr(torch.randn(n, n, device=DEV, generator=g))[0].contiguous() for n in (n1, n2)]
    layer = B.pack_weights(W, R[0], R[1], U, V, n1, n2)
    act, alone = B.Activations(layer, M), B.Activations(layer, 1)
    for seed in (1, 2):                                     # twice on one scratch
        X = torch.randn(M, K, device=DEV, generator=g)
        X[:, ::97] *= 50.0
        X = X.to(torch.bfloat16) if x == "bf16" else X
        act.T.fill_(float("nan"))
        B.rotate_quant(layer, X, act)
        torch.cuda.synchronize()
        want = X.double() @ U.double()
        # fp32 sums: no path adds more than K / 32 + 72 terms in a row (steps of an MFMA in one wavefront; wavefronts;
        # slices), the 32 products of a step among themselves; products are exact
        bound = (K / 32 + 72 + 32) * 2.0 ** -23 * (X.double().abs() @ U.double().abs())
        assert bool(((act.T.double() - want).abs() <= bound).all())
        # the rest of the call is not touched by it: one token by itself has the same scale
        i = M - 1
        B.rotate_quant(layer, X[i:i + 1].contiguous(), alone)
        torch.cuda.synchronize()
        assert abs(alone.scale[0].item() / act.scale[i].item() - 1) < 1e-5
