"""bwla_psp_workspace_size on the host: a scratch for M tokens also serves fewer, and asking for it costs little."""
import ctypes
import time
from ctypes import byref, c_int64, c_size_t

import pytest

from paper_2605_00422_amd import binding as B


@pytest.fixture(scope="module")
def lib():
    import os
    if not os.path.exists(B.LIB_PATH):
        from paper_2605_00422_amd.build import build_library
        build_library()
    return B.load()


def _up(x, to=256):
    return (x + to - 1) // to * to


def _layer(lib, N, n1, n2, r, mode=0):
    """A descriptor as bwla_pack_weights_mode fills it in; nothing is launched on it."""
    d = B.BwlaLayer()
    extra = (2 if mode & 2 else 0) + (mode & 1)
    d.N, d.K, d.n1, d.n2, d.r, d.mode = N, n1 * n2, n1, n2, r + extra, mode
    planes = lambda n: 3 * _up(n, 16) * _up(n, 32) * 2                       # noqa: E731
    off = 0
    for name, size in (("bits", _up(N, 16) // 16 * (_up(d.K, 512) // 512) * 1024), ("alpha", 2 * N),
                       ("V", 2 * N * _up(d.r, 16)), ("U", 2 * d.K * _up(r, 16)), ("R1", 4 * n1 * n1), ("R2", 4 * n2 * n2),
                       ("R1p", planes(n1)), ("R2p", planes(n2))):
        setattr(d, "off_" + name, off)
        off = _up(off + size)
    total = c_size_t()
    assert lib.bwla_packed_size_mode(N, d.K, n1, n2, r, mode, byref(total)) == B.BWLA_OK
    d.off_Rd = off if total.value > off else 0
    d.blob_bytes, d.d_blob = total.value, 0x100000
    return d


def _sizes(lib, d, tokens):
    ws, room, out = c_size_t(), c_size_t(), []
    for M in tokens:
        assert lib.bwla_psp_workspace_size(byref(d), c_int64(M), byref(ws)) == B.BWLA_OK
        assert lib.bwla_code_room_size(byref(d), c_int64(M), byref(room)) == B.BWLA_OK
        out.append((ws.value, room.value))
    return out


# (n1, n2, rank, mode): one and two column groups of the projection (rank above 64); rotations that may be split, that
# the walking kernel serves, and neither; short rows
LAYERS = [(64, 64, 32, 0), (64, 64, 96, 3), (128, 64, 64, 0), (128, 64, 128, 0), (80, 64, 37, 0), (128, 86, 32, 3),
          (160, 160, 8, 0), (160, 160, 112, 0), (224, 128, 64, 0), (224, 128, 96, 1), (137, 32, 20, 0), (16, 32, 8, 0),
          (16, 12, 70, 0), (172, 104, 64, 0), (224, 128, 0, 0)]


@pytest.mark.parametrize("n1,n2,r,mode", LAYERS)
def test_a_scratch_for_more_tokens_serves_fewer(lib, n1, n2, r, mode):
    """What a call on M tokens of either type wants is part of the size for M tokens, so that sizes that never fall cover
    every smaller number of tokens: all up to 2200, and those around the last that are split."""
    d = _layer(lib, 16, n1, n2, r, mode)                                     # (16 channels: no room for codes)
    tokens = list(range(1, 2201)) + list(range(2240, 5000, 63)) + [x + y for x in (131072, 262144) for y in (-64, -1, 0, 1, 64)]
    sizes = _sizes(lib, d, tokens)
    assert all(room == 0 for _, room in sizes)
    for (a, b), M in zip(zip(sizes, sizes[1:]), tokens[1:]):
        assert a[0] <= b[0], M


def test_the_room_for_codes_lies_behind_all_of_that(lib):
    """... and behind the arrival counters, which calls on any layer and token count rely on."""
    for n1, n2, r, mode in LAYERS:
        plain, wide = _layer(lib, 16, n1, n2, r, mode), _layer(lib, 64, n1, n2, r, mode)
        tokens = [1, 64, 65, 257, 1000, 4096]
        for M, (need, _), (ws, room) in zip(tokens, _sizes(lib, plain, tokens), _sizes(lib, wide, tokens)):
            assert (room > 0) == (M > 64 and wide.K % 128 == 0)
            if room:
                assert ws - room >= max(need, 7168 + 16384) and ws - room < max(need, 7168 + 16384) + 256
            else:
                assert ws == need


@pytest.mark.parametrize("n1,n2,r", [(64, 64, 32), (160, 160, 64), (224, 128, 64)])
def test_the_size_is_quick_to_ask_for(lib, n1, n2, r):
    """Activations asks for it whenever they are made.  All numbers of tokens gone through took 500 to 900 us here, the ones
    that can need the most 30 to 60: half of the former is the limit, and the fastest of fifty calls is compared."""
    d, out, best = _layer(lib, 64, n1, n2, r), c_size_t(), 1.0
    for _ in range(50):
        t = time.perf_counter()
        lib.bwla_psp_workspace_size(byref(d), 4096, byref(out))
        best = min(best, time.perf_counter() - t)
    assert best < 250e-6
