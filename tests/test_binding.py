"""What the Python binding hands to the library (no GPU: a stand-in records the calls)."""
import pytest

torch = pytest.importorskip("torch")

from paper_2605_00422_amd import binding as B  # noqa: E402

ROTATE, ROOM = 4096, 8192           # bytes of scratch and of room that the stand-in asks for


class _Recorder:
    def __init__(self):
        self.calls = []

    def __getattr__(self, name):
        def call(*args):
            if name == "bwla_psp_workspace_size":
                args[2]._obj.value = ROTATE + ROOM
            elif name == "bwla_code_room_size":
                args[2]._obj.value = ROOM
            else:
                self.calls.append((name, args))
            return B.BWLA_OK
        return call


@pytest.fixture
def lib(monkeypatch):
    lib = _Recorder()
    monkeypatch.setattr(B, "load", lambda: lib)
    monkeypatch.setattr(B, "_stream", lambda: 0)
    return lib


def _layer():
    desc = B.BwlaLayer()
    desc.N, desc.K, desc.n1, desc.n2, desc.r = 64, 512, 16, 32, 8
    return B.PackedLayer(desc, torch.empty(16, dtype=torch.uint8))


def _inside(args, t):
    return [a for a in args if isinstance(a, int) and t.data_ptr() <= a < t.data_ptr() + t.numel()]


def test_forward_calls_on_codes_are_not_given_the_scratch(lib):
    """Activations that share a scratch share nothing that linear_forward and linear_forward_swiglu may write."""
    layer = _layer()
    one, two = B.Activations(layer, 100), B.Activations(layer, 100)
    two.ws, two.ws_bytes = one.ws, one.ws_bytes
    X, Y = torch.empty(100, 512, dtype=torch.bfloat16), torch.empty(100, 64)
    for act in (one, two):
        B.rotate_quant(layer, X, act, 6)
        del lib.calls[:]
        B.linear_forward(layer, act, Y)
        B.linear_forward_swiglu(layer, act, Y)
        for _, args in lib.calls:
            assert not _inside(args, act.ws)
            assert _inside(args, act.room) and not _inside(args, (two if act is one else one).room)
        # the whole layer in one call: its scratch ends where it says, the room is handed over beside it
        del lib.calls[:]
        B.decode_forward(layer, X, act, Y)
        args = lib.calls[0][1]
        assert _inside(args, act.ws) and _inside(args, act.room)
        assert act.ws.numel() >= act.ws_bytes and act.room.numel() >= act.room_bytes == ROOM
        assert act.ws_bytes == ROTATE


def test_objects_from_before_there_was_a_room(lib):
    layer = _layer()
    act = B.Activations.__new__(B.Activations)
    act.__dict__.update(M=100, q=torch.empty(100, 512, dtype=torch.int8), scale=torch.empty(100),
                        qsum=torch.empty(100, dtype=torch.int32), T=torch.empty(100, 8), ws=torch.zeros(16, dtype=torch.uint8),
                        ws_bytes=0)
    X, Y = torch.empty(100, 512, dtype=torch.bfloat16), torch.empty(100, 64)
    B.linear_forward(layer, act, Y)
    B.linear_forward_swiglu(layer, act, Y)
    B.decode_forward(layer, X, act, Y)
    B.linear_forward(layer, act, Y)
    assert [n for n, _ in lib.calls] == ["bwla_linear_forward", "bwla_linear_forward_swiglu", "bwla_decode_forward",
                                         "bwla_linear_forward_room"]


@pytest.mark.parametrize("bits", [6.0, torch.tensor(6), True + 5])
@pytest.mark.parametrize("call", ["rotate_quant", "decode_forward"])
def test_width_of_the_codes_in_any_type_that_these_calls_take(lib, call, bits):
    """The GEMM behind them gets it as a plain integer, as ctypes asks."""
    layer = _layer()
    act = B.Activations(layer, 100)
    X, Y = torch.empty(100, 512, dtype=torch.bfloat16), torch.empty(100, 64)
    if call == "rotate_quant":
        B.rotate_quant(layer, X, act, bits)
    else:
        B.decode_forward(layer, X, act, Y, act_bits=bits)
    del lib.calls[:]
    B.linear_forward(layer, act, Y)
    B.linear_forward_swiglu(layer, act, Y)
    for name, args in lib.calls:
        assert name.endswith("_room") and type(args[6]) is int and args[6] == 6
