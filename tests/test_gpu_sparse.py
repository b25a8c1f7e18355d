"""The GEMM on the sparse INT8 instructions (csrc/gemm_sparse.hip) against the dense one, which the oracle checks
(test_gpu_parity.py), and against exact integer products: it computes the same sums and the same epilogue, so its outputs
are the dense kernel's bit for bit."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

# (tokens, K, N, rank): edges of tiles, supersteps and ranks of each tile that the dispatch chooses from
SHAPES = [
    (848, 384, 21104, 16),      # 64 x 256: three quarters of a superstep, a quarter of the last tile
    (2859, 512, 4285, 0),       # 64 x 256: odd channels, no ranks
    (69, 9728, 25770, 37),      # 64 x 256: five tokens in the last tile, a rank that is no multiple of four
    (80, 16384, 26729, 96),     # 64 x 256: sixteen tokens in the last tile, odd channels, two chunks of ranks
    (345, 5248, 22035, 16),     # 64 x 640: a quarter of a superstep at the end, odd channels
    (455, 5632, 19040, 37),     # 64 x 640, channels end inside a tile
    (2048, 25600, 5120, 64),    # 64 x 640, fifty supersteps
    (855, 2944, 16948, 0),      # 128 x 512: 87 tokens in the last tile, no ranks
    (601, 5120, 20923, 37),     # 128 x 512, odd channels
    (598, 8064, 20415, 96),     # 128 x 512: two chunks of ranks, three quarters of a superstep at the end
]


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_00422_amd import binding as B
    B.load()


def _layer(M, K, N, r, centered=False, asym=False):
    from paper_2605_00422_amd import binding as B
    g = torch.Generator(device=DEV)
    g.manual_seed(M + K + N + r)
    n1, n2 = B.kron_factor(K)
    W = torch.randn(N, K, device=DEV, generator=g)
    U = V = None
    if r:
        U = torch.randn(K, r, device=DEV, generator=g).half().float()
        V = (torch.randn(N, r, device=DEV, generator=g) * 0.1).half().float()
    q = [torch.linalg.qr(torch.randn(n, n, device=DEV, generator=g))[0].contiguous() for n in (n1, n2)]
    return B.pack_weights(W, q[0], q[1], U, V, n1, n2, centered=centered, asym=asym), g


def _acts(layer, M, K, g, lo, hi):
    from paper_2605_00422_amd import binding as B
    act = B.Activations(layer, M)
    act.q.copy_(torch.randint(lo, hi + 1, (M, K), device=DEV, generator=g))
    act.q[:, ::7] = hi                                      # equal neighbours at the ends of the range: largest sums
    act.q[-1, ::3] = lo
    act.scale.copy_((torch.rand(act.scale.shape, device=DEV, generator=g) + 0.5) * 0.01)
    if act.T is not None:
        act.T.copy_(torch.randn(act.T.shape, device=DEV, generator=g))
    B.code_sums(act.q, act.qsum)
    return act


def _run(layer, act, N, act_bits, gated):
    from paper_2605_00422_amd import binding as B
    act.act_bits = act_bits
    Y = torch.full((act.M, N), float("nan"), device=DEV)
    acc = torch.full((act.M, N), -7, dtype=torch.int32, device=DEV)
    B.linear_forward(layer, act, Y, acc)
    Y2 = torch.full_like(Y, float("nan"))
    B.linear_forward(layer, act, Y2)
    H = None
    if gated:
        H = torch.full((act.M, N // 2), float("nan"), dtype=torch.bfloat16, device=DEV)
        B.linear_forward_swiglu(layer, act, H)
    torch.cuda.synchronize()
    assert torch.equal(Y, Y2)
    return Y, acc, H


def _same(a, b):
    for x, y in zip(a, b):
        assert (x is None) == (y is None)
        if x is not None:
            assert bool(torch.isfinite(x.float()).all())
            assert torch.equal(x, y)


@pytest.mark.parametrize("M,K,N,r", SHAPES)
def test_same_bits_as_the_dense_kernel(M, K, N, r):
    from paper_2605_00422_amd import binding as B
    layer, g = _layer(M, K, N, r)
    act = _acts(layer, M, K, g, -64, 63)
    room, ws = act.room, act.ws.clone()
    room.fill_(0x5a)                                        # where the codes are laid out anew
    dense = _run(layer, act, N, 8, N % 2 == 0)
    assert bool((room == 0x5a).all())                       # (the dense kernel leaves it alone)
    sparse = _run(layer, act, N, 7, N % 2 == 0)
    assert not bool((room == 0x5a).all()), "the shape is not served by the sparse kernel"
    _same(sparse, dense)
    sgn, _ = B.unpack_signs(layer)
    want = act.q.float() @ sgn.float().t()                  # exact: |acc| <= 64 K < 2^24
    assert torch.equal(sparse[1].float(), want)
    assert torch.equal(act.ws, ws)                          # the scratch, which another Activations may use meanwhile
    # less than the room: the dense kernel
    act.room_bytes -= 256
    room.fill_(0x5a)
    _same(_run(layer, act, N, 7, N % 2 == 0), dense)
    assert bool((room == 0x5a).all())


@pytest.mark.parametrize("M,K,N,r", [SHAPES[0], SHAPES[4], SHAPES[7]])
@pytest.mark.parametrize("where", ["last", "first", "all"])
def test_codes_wider_than_announced_are_found(M, K, N, r, where):
    """act_bits says which kernel to start; a code outside [-64, 63] sends its tile to the dense instructions."""
    from paper_2605_00422_amd import binding as B
    layer, g = _layer(M, K, N, r)
    act = _acts(layer, M, K, g, -64, 63)
    if where == "last":
        act.q[M - 1, K - 1] = 64
    elif where == "first":
        act.q[0, 0] = -65
        act.q[70, 5] = 127
    else:
        act.q.copy_(torch.randint(-127, 128, (M, K), device=DEV, generator=g))
    B.code_sums(act.q, act.qsum)
    _same(_run(layer, act, N, 6, N % 2 == 0), _run(layer, act, N, 8, N % 2 == 0))


@pytest.mark.parametrize("bits,centered,asym,x", [(6, False, False, torch.bfloat16), (7, False, True, torch.bfloat16),
                                                  (4, True, True, torch.float32), (8, True, False, torch.bfloat16)])
def test_whole_layer(bits, centered, asym, x):
    """decode_forward with the room for the codes and without it."""
    from paper_2605_00422_amd import binding as B
    M, K, N, r = 1111, 4096, 22001, 20
    layer, g = _layer(M, K, N, r, centered, asym)
    X = torch.randn(M, K, device=DEV, generator=g).to(x)
    outs = []
    for room in (True, False):
        act = B.Activations(layer, M)
        if not room:
            act.room_bytes -= 256
        Y = torch.full((M, N), float("nan"), device=DEV)
        acc = torch.full((M, N), -7, dtype=torch.int32, device=DEV)
        B.decode_forward(layer, X, act, Y, acc, act_bits=bits)
        torch.cuda.synchronize()
        outs.append((Y, acc, act.q, act.T, act.scale))
    _same(*outs)


@pytest.mark.parametrize("M,K,N,r", [SHAPES[0], SHAPES[8]])
def test_room_at_the_end_of_a_scratch(M, K, N, r):
    """The calls of the C ABI that take one scratch for everything: in one of bwla_psp_workspace_size they lay the codes
    out in its last bytes, in a smaller one nowhere, and the results are the same."""
    from ctypes import byref
    from paper_2605_00422_amd import binding as B
    lib, p, st = B.load(), B._ptr, B._stream()
    layer, g = _layer(M, K, N, r)
    X = torch.randn(M, K, device=DEV, generator=g).to(torch.bfloat16)
    act = B.Activations(layer, M)
    want = B.decode_forward(layer, X, act, torch.empty(M, N, device=DEV)).clone()
    H = torch.empty(M, N // 2, dtype=torch.bfloat16, device=DEV) if N % 2 == 0 else None
    wantH = B.linear_forward_swiglu(layer, act, H).clone() if H is not None else None
    nbytes = B.psp_workspace_size(layer, M)
    codes = (p(act.q), p(act.scale), p(act.qsum), p(act.T))
    for less in (0, 256):
        ws = torch.zeros(nbytes, dtype=torch.uint8, device=DEV)
        room = ws[-act.room_bytes:]
        n = nbytes - less

        def used():
            torch.cuda.synchronize()
            u = bool(room[:-256].any())
            room.zero_()
            return u

        Y = torch.full((M, N), float("nan"), device=DEV)
        assert lib.bwla_decode_forward(byref(layer.desc), p(X), B.BWLA_X_BF16, M, *codes, p(ws), n, p(Y), None, st) == B.BWLA_OK
        assert used() == (less == 0) and torch.equal(Y, want)
        Y.fill_(float("nan"))
        assert lib.bwla_linear_forward_bits(byref(layer.desc), *codes, M, 6, p(ws), n, p(Y), None, st) == B.BWLA_OK
        assert used() == (less == 0) and torch.equal(Y, want)
        if H is not None:
            H.fill_(float("nan"))
            assert lib.bwla_linear_forward_swiglu_bits(byref(layer.desc), *codes, M, 6, p(ws), n, p(H), None, 0, st) == B.BWLA_OK
            assert used() == (less == 0) and torch.equal(H, wantH)


def test_one_scratch_for_calls_of_several_sizes():
    """The room for the codes lies at the end of a scratch, behind the arrival counters: calls that lay codes out there, on
    fewer tokens and of a layer without a projection among them, leave the counters of the others at zero.  Once in a
    scratch for the most tokens, once in the smallest that has a room at all."""
    from ctypes import byref
    from paper_2605_00422_amd import binding as B
    lib, p, st = B.load(), B._ptr, B._stream()
    K, N = 4096, 22016
    layers = {r: _layer(4096, K, N, r)[0] for r in (32, 0)}
    g = torch.Generator(device=DEV)
    g.manual_seed(7)
    X = torch.randn(4096, K, device=DEV, generator=g).to(torch.bfloat16)
    acts = {r: B.Activations(layers[r], 4096) for r in layers}
    Y = torch.empty(4096, N, device=DEV)
    want = {}

    def call(r, M, ws, sparse):
        """rank, tokens; whether codes are laid out (the kernel is the sparse one)"""
        layer, act = layers[r], acts[r]
        if (r, M) not in want:
            want[r, M] = B.decode_forward(layer, X[:M], act, Y[:M]).clone()
        tail = ws[-4096 * 16:]                              # the last codes and the flags behind them
        tail.fill_(0x5a)
        if act.T is not None:
            act.T.fill_(float("nan"))
        Y.fill_(float("nan"))
        assert lib.bwla_decode_forward(byref(layer.desc), p(X), B.BWLA_X_BF16, M, p(act.q), p(act.scale), p(act.qsum), p(act.T),
                                       p(ws), ws.numel(), p(Y), None, st) == B.BWLA_OK
        torch.cuda.synchronize()
        assert torch.equal(Y[:M], want[r, M]), (r, M)
        assert not bool(ws[7168:7168 + 16384].any()), (r, M)
        assert bool((tail != 0x5a).any()) == sparse, (r, M)

    # 4096 tokens hand their projection's sums over inside its launch, which counts arrivals
    ws = torch.zeros(B.psp_workspace_size(layers[32], 4096), dtype=torch.uint8, device=DEV)
    for r, M, sparse in ((32, 848, True), (32, 4096, True), (0, 848, True), (32, 4096, True), (32, 200, False), (32, 848, True),
                         (32, 4096, True)):
        call(r, M, ws, sparse)
    # without a projection nothing but the counters lies in front of the room
    ws = torch.zeros(B.psp_workspace_size(layers[0], 848), dtype=torch.uint8, device=DEV)
    assert ws.numel() == 7168 + 16384 + B.code_room_size(layers[0], 848)
    assert B.psp_workspace_size(layers[32], 64) <= ws.numel()
    for r, M, sparse in ((0, 848, True), (32, 64, False), (0, 848, True), (32, 17, False), (0, 848, True)):
        call(r, M, ws, sparse)


def test_replayed_from_a_graph():
    from paper_2605_00422_amd import binding as B
    M, K, N, r = 1024, 8192, 20480, 32
    layer, g = _layer(M, K, N, r)
    act = B.Activations(layer, M)
    Xs = [torch.randn(M, K, device=DEV, generator=g).to(torch.bfloat16) for _ in range(3)]
    X, Y = Xs[0].clone(), torch.empty(M, N, device=DEV)
    want = [B.decode_forward(layer, x, act, Y).clone() for x in Xs]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        B.decode_forward(layer, X, act, Y)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        B.decode_forward(layer, X, act, Y)
    for x, w in zip(Xs + Xs, want + want):
        X.copy_(x)
        Y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y, w)
