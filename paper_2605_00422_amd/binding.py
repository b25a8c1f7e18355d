"""ctypes binding of libbwla: same names as the C ABI in include/bwla.h, argument marshalling
only.  Device memory and streams come from PyTorch; every step of the path runs in the HIP
kernels of the library.  There is no fallback: if the library is missing, loading raises."""
from __future__ import annotations

import ctypes
import os
from ctypes import POINTER, Structure, byref, c_char_p, c_int, c_int32, c_int64, c_size_t, c_uint64, c_void_p

HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(HERE, "libbwla.so")

BWLA_OK = 0
BWLA_ERR_NULL, BWLA_ERR_SHAPE, BWLA_ERR_ALIGN, BWLA_ERR_BUFSIZE, BWLA_ERR_UNSUPPORTED, BWLA_ERR_HIP = 1, 2, 3, 4, 5, 6
BWLA_X_F32, BWLA_X_BF16 = 0, 1
BWLA_MODE_ROW_SHIFT, BWLA_MODE_ASYM_ACT = 1, 2

EXPORTS = ["bwla_status_string", "bwla_version", "bwla_kron_factor", "bwla_packed_size", "bwla_pack_weights",
           "bwla_unpack_signs", "bwla_psp_workspace_size", "bwla_rotate_quant", "bwla_code_sums",
           "bwla_linear_forward", "bwla_decode_forward", "bwla_packed_size_centered", "bwla_pack_weights_centered", "bwla_rotate_quant_bits",
           "bwla_packed_size_mode", "bwla_pack_weights_mode", "bwla_swiglu_workspace_size",
           "bwla_linear_forward_swiglu", "bwla_decode_forward_static", "bwla_probe_hbm_read",
           "bwla_probe_mfma_int8", "bwla_decode_forward_launches", "bwla_decode_forward_bits", "bwla_pack_codes_a4",
           "bwla_linear_forward_a4", "bwla_probe_empty_launch", "bwla_probe_load_latency", "bwla_probe_clock",
           "bwla_linear_forward_bits", "bwla_linear_forward_swiglu_bits", "bwla_code_room_size", "bwla_decode_forward_room",
           "bwla_linear_forward_room", "bwla_linear_forward_swiglu_room", "bwla_linear_forward_kernel"]


class BwlaLayer(Structure):
    _fields_ = [("N", c_int64), ("K", c_int64), ("n1", c_int32), ("n2", c_int32), ("r", c_int32),
                ("mode", c_int32), ("off_bits", c_uint64), ("off_alpha", c_uint64), ("off_V", c_uint64),
                ("off_U", c_uint64), ("off_R1", c_uint64), ("off_R2", c_uint64), ("off_R1p", c_uint64), ("off_R2p", c_uint64),
                ("off_Rd", c_uint64), ("blob_bytes", c_uint64),
                ("d_blob", c_void_p)]


class BwlaError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = status
        super().__init__(f"{where}: {status_string(status)} (status {status})")


_lib = None


def load() -> ctypes.CDLL:
    """Load libbwla.so from the package directory (build it first with build.py)."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(LIB_PATH):
        raise FileNotFoundError(f"{LIB_PATH} is missing: run `python -m paper_2605_00422_amd.build` "
                                "(or __graft_entry__.build()) first")
    lib = ctypes.CDLL(LIB_PATH)
    lib.bwla_status_string.restype = c_char_p
    lib.bwla_status_string.argtypes = [c_int]
    lib.bwla_version.restype = c_int
    lib.bwla_kron_factor.argtypes = [c_int64, POINTER(c_int32), POINTER(c_int32)]
    lib.bwla_packed_size.argtypes = [c_int64, c_int64, c_int32, c_int32, c_int32, POINTER(c_size_t)]
    lib.bwla_pack_weights.argtypes = [c_void_p] * 5 + [c_int64, c_int64, c_int32, c_int32, c_int32, c_void_p,
                                                       c_size_t, c_void_p, POINTER(BwlaLayer)]
    lib.bwla_packed_size_centered.argtypes = lib.bwla_packed_size.argtypes
    lib.bwla_pack_weights_centered.argtypes = lib.bwla_pack_weights.argtypes
    lib.bwla_packed_size_mode.argtypes = [c_int64, c_int64, c_int32, c_int32, c_int32, c_int32, POINTER(c_size_t)]
    lib.bwla_pack_weights_mode.argtypes = [c_void_p] * 5 + [c_int64, c_int64, c_int32, c_int32, c_int32, c_int32,
                                                            c_void_p, c_size_t, c_void_p, POINTER(BwlaLayer)]
    lib.bwla_unpack_signs.argtypes = [POINTER(BwlaLayer), c_void_p, c_void_p, c_void_p]
    lib.bwla_psp_workspace_size.argtypes = [POINTER(BwlaLayer), c_int64, POINTER(c_size_t)]
    lib.bwla_rotate_quant.argtypes = [POINTER(BwlaLayer), c_void_p, c_int, c_int64, c_void_p, c_void_p, c_void_p,
                                      c_void_p, c_void_p, c_size_t, c_void_p]
    lib.bwla_rotate_quant_bits.argtypes = [POINTER(BwlaLayer), c_void_p, c_int, c_int, c_int64, c_void_p, c_void_p,
                                           c_void_p, c_void_p, c_void_p, c_size_t, c_void_p]
    lib.bwla_code_sums.argtypes = [c_void_p, c_int64, c_int64, c_void_p, c_void_p]
    lib.bwla_linear_forward.argtypes = [POINTER(BwlaLayer), c_void_p, c_void_p, c_void_p, c_void_p, c_int64,
                                        c_void_p, c_void_p, c_void_p]
    lib.bwla_decode_forward.argtypes = [POINTER(BwlaLayer), c_void_p, c_int, c_int64, c_void_p, c_void_p, c_void_p,
                                        c_void_p, c_void_p, c_size_t, c_void_p, c_void_p, c_void_p]
    lib.bwla_decode_forward_static.argtypes = [POINTER(BwlaLayer), c_void_p, c_int, c_int64, c_void_p, c_void_p,
                                               c_void_p, c_void_p, c_void_p, c_void_p, c_void_p]
    lib.bwla_decode_forward_bits.argtypes = [POINTER(BwlaLayer), c_void_p, c_int, c_int, c_int64, c_void_p, c_void_p, c_void_p,
                                             c_void_p, c_void_p, c_size_t, c_void_p, c_void_p, c_void_p]
    lib.bwla_pack_codes_a4.argtypes = [c_void_p, c_int64, c_int64, c_void_p, c_void_p]
    lib.bwla_linear_forward_a4.argtypes = [POINTER(BwlaLayer), c_void_p, c_void_p, c_void_p, c_void_p, c_int64,
                                           c_void_p, c_void_p, c_void_p]
    lib.bwla_decode_forward_launches.argtypes = [POINTER(BwlaLayer), c_int, c_int64, POINTER(c_int)]
    lib.bwla_probe_hbm_read.argtypes = [c_void_p, c_size_t, c_void_p, c_size_t, c_void_p]
    lib.bwla_probe_mfma_int8.argtypes = [c_int, c_void_p, c_size_t, POINTER(ctypes.c_int64), c_void_p]
    lib.bwla_probe_empty_launch.argtypes = [c_void_p]
    lib.bwla_probe_clock.argtypes = [c_void_p, c_void_p]
    lib.bwla_probe_load_latency.argtypes = [c_void_p, c_size_t, c_size_t, c_int, c_void_p, c_void_p]
    lib.bwla_swiglu_workspace_size.argtypes = [POINTER(BwlaLayer), c_int64, POINTER(c_size_t)]
    lib.bwla_linear_forward_swiglu.argtypes = [POINTER(BwlaLayer), c_void_p, c_void_p, c_void_p, c_void_p, c_int64,
                                               c_void_p, c_void_p, c_size_t, c_void_p]
    lib.bwla_linear_forward_bits.argtypes = [POINTER(BwlaLayer), c_void_p, c_void_p, c_void_p, c_void_p, c_int64, c_int,
                                             c_void_p, c_size_t, c_void_p, c_void_p, c_void_p]
    lib.bwla_linear_forward_swiglu_bits.argtypes = [POINTER(BwlaLayer), c_void_p, c_void_p, c_void_p, c_void_p, c_int64,
                                                    c_int, c_void_p, c_size_t, c_void_p, c_void_p, c_size_t, c_void_p]
    lib.bwla_linear_forward_room.argtypes = lib.bwla_linear_forward_bits.argtypes
    lib.bwla_linear_forward_swiglu_room.argtypes = lib.bwla_linear_forward_swiglu_bits.argtypes
    lib.bwla_code_room_size.argtypes = [POINTER(BwlaLayer), c_int64, POINTER(c_size_t)]
    lib.bwla_decode_forward_room.argtypes = [POINTER(BwlaLayer), c_void_p, c_int, c_int, c_int64, c_void_p, c_void_p, c_void_p,
                                             c_void_p, c_void_p, c_size_t, c_void_p, c_size_t, c_void_p, c_void_p, c_void_p]
    lib.bwla_linear_forward_kernel.argtypes = [c_int64, c_int64, c_int64, c_int32, c_int, c_int, POINTER(c_char_p)]
    for name in EXPORTS:
        if name not in ("bwla_status_string", "bwla_version"):
            getattr(lib, name).restype = c_int
    _lib = lib
    return lib


def _check(status: int, where: str) -> None:
    if status != BWLA_OK:
        raise BwlaError(status, where)


# A decoding step is a few microseconds on the GPU, so what a call costs here counts: pointers go to
# ctypes as plain integers (the argtypes convert them), the descriptor's reference is made once per
# layer, and the stream is read through torch's raw accessor -- torch.cuda.current_stream() builds a
# Stream object, 2.9 us a call against 0.1.  One-token call of a 4096-wide layer: 9.8 -> 6.4 us of host
# time (the GPU takes 6.2).
def _ptr(t):
    return None if t is None else t.data_ptr()


def _stream():
    global _torch
    if _torch is None:
        import torch
        torch.cuda.init()
        _torch = torch
    c = _torch._C
    return c._cuda_getCurrentRawStream(c._cuda_getDevice())


_torch = None


_xdtypes = {}


def _xdtype(X) -> int:
    if not _xdtypes:
        import torch
        _xdtypes.update({torch.bfloat16: BWLA_X_BF16, torch.float32: BWLA_X_F32})
    xd = _xdtypes.get(X.dtype)
    if xd is None:
        raise TypeError("X must be float32 or bfloat16")
    return xd


# ------------------------------------------------------------------ host-only calls
def status_string(status: int) -> str:
    return load().bwla_status_string(int(status)).decode()


def version() -> int:
    return load().bwla_version()


def kron_factor(K: int) -> tuple[int, int]:
    n1, n2 = c_int32(), c_int32()
    _check(load().bwla_kron_factor(K, byref(n1), byref(n2)), "bwla_kron_factor")
    return n1.value, n2.value


def packed_size(N: int, K: int, n1: int, n2: int, r: int, centered: bool = False, asym: bool = False) -> int:
    out = c_size_t()
    if asym:
        mode = BWLA_MODE_ASYM_ACT | (BWLA_MODE_ROW_SHIFT if centered else 0)
        _check(load().bwla_packed_size_mode(N, K, n1, n2, r, mode, byref(out)), "bwla_packed_size_mode")
        return out.value
    name = "bwla_packed_size_centered" if centered else "bwla_packed_size"
    _check(getattr(load(), name)(N, K, n1, n2, r, byref(out)), name)
    return out.value


# ------------------------------------------------------------------ device calls (torch tensors in, torch tensors out)
class PackedLayer:
    """Owns the device blob (a torch uint8 tensor) and the plain descriptor."""

    def __init__(self, desc: BwlaLayer, blob):
        self.desc = desc
        self.blob = blob

    @property
    def desc(self) -> BwlaLayer:
        return self._desc

    @desc.setter
    def desc(self, desc: BwlaLayer):
        self._desc, self._ref = desc, byref(desc)

    @property
    def shape(self):
        d = self.desc
        return d.N, d.K, d.n1, d.n2, d.r


def pack_weights(W_rot, R1, R2, U, V, n1: int, n2: int, centered: bool = False, asym: bool = False) -> PackedLayer:
    """W_rot (N,K), R1, R2, U (K,r), V (N,r): fp32 CUDA tensors (U, V may be None for r = 0).
    centered: binarize with the row shift (bwla_pack_weights_centered); asym: the layer's
    activations get per-token asymmetric codes (bwla_pack_weights_mode)."""
    import torch
    N, K = W_rot.shape
    r = 0 if U is None else U.shape[1]
    nbytes = packed_size(N, K, n1, n2, r, centered, asym)
    blob = torch.zeros(nbytes, dtype=torch.uint8, device=W_rot.device)
    desc = BwlaLayer()
    if asym:
        mode = BWLA_MODE_ASYM_ACT | (BWLA_MODE_ROW_SHIFT if centered else 0)
        _check(load().bwla_pack_weights_mode(_ptr(W_rot), _ptr(R1), _ptr(R2), _ptr(U), _ptr(V), N, K, n1, n2, r, mode,
                                             _ptr(blob), nbytes, _stream(), byref(desc)), "bwla_pack_weights_mode")
        return PackedLayer(desc, blob)
    name = "bwla_pack_weights_centered" if centered else "bwla_pack_weights"
    _check(getattr(load(), name)(_ptr(W_rot), _ptr(R1), _ptr(R2), _ptr(U), _ptr(V), N, K, n1, n2, r,
                                 _ptr(blob), nbytes, _stream(), byref(desc)), name)
    return PackedLayer(desc, blob)


def unpack_signs(layer: PackedLayer):
    import torch
    N, K = layer.desc.N, layer.desc.K
    sgn = torch.empty((N, K), dtype=torch.int8, device=layer.blob.device)
    alpha = torch.empty((N,), dtype=torch.float32, device=layer.blob.device)
    _check(load().bwla_unpack_signs(layer._ref, _ptr(sgn), _ptr(alpha), _stream()), "bwla_unpack_signs")
    return sgn, alpha


def psp_workspace_size(layer: PackedLayer, M: int) -> int:
    out = c_size_t()
    _check(load().bwla_psp_workspace_size(layer._ref, M, byref(out)), "bwla_psp_workspace_size")
    return out.value


def code_room_size(layer: PackedLayer, M: int) -> int:
    out = c_size_t()
    _check(load().bwla_code_room_size(layer._ref, M, byref(out)), "bwla_code_room_size")
    return out.value


class Activations:
    """Caller-owned outputs of bwla_rotate_quant for M tokens (allocated once, reused).

    ws is the scratch of rotate_quant and decode_forward; several Activations may share one, and calls that use it must not
    overlap.  room (None where nothing uses it) is where decode_forward, linear_forward and linear_forward_swiglu lay out
    this object's codes for the GEMM on the sparse instructions.  It belongs to this object alone, as q does: calls on
    different Activations may overlap whatever scratch they share, and so may linear_forward calls of several layers on one
    (they write the same bytes there)."""

    room = None
    room_bytes = 0
    # width of the codes that rotate_quant wrote last: which GEMM is worth starting (the library looks at the codes,
    # so q may be overwritten with others); 8 = any
    act_bits = 8

    def __init__(self, layer: PackedLayer, M: int):
        import torch
        dev = layer.blob.device
        d = layer.desc
        self.M = M
        self.q = torch.empty((M, d.K), dtype=torch.int8, device=dev)
        self.scale = torch.empty((M,), dtype=torch.float32, device=dev)
        self.qsum = torch.empty((M,), dtype=torch.int32, device=dev)
        self.T = torch.empty((M, d.r), dtype=torch.float32, device=dev) if d.r > 0 else None
        self.room_bytes = code_room_size(layer, M)
        self.room = torch.empty(self.room_bytes, dtype=torch.uint8, device=dev) if self.room_bytes else None
        ws = psp_workspace_size(layer, M) - self.room_bytes                 # (a scratch may have the room at its end: not this one)
        self.ws_bytes = ws
        self.ws = torch.zeros(max(ws, 16), dtype=torch.uint8, device=dev)   # zero-filled once, as the ABI asks


def rotate_quant(layer: PackedLayer, X, act: Activations, act_bits: int = 6) -> Activations:
    """X: (M,K) CUDA tensor, float32 or bfloat16.  act_bits other than 6: bwla_rotate_quant_bits."""
    xd = _xdtype(X)
    if act_bits == 6:
        _check(load().bwla_rotate_quant(layer._ref, _ptr(X), xd, X.shape[0], _ptr(act.q), _ptr(act.scale),
                                        _ptr(act.qsum), _ptr(act.T), _ptr(act.ws), act.ws_bytes, _stream()),
               "bwla_rotate_quant")
        act.act_bits = 6
    else:
        _check(load().bwla_rotate_quant_bits(layer._ref, _ptr(X), xd, act_bits, X.shape[0], _ptr(act.q),
                                             _ptr(act.scale), _ptr(act.qsum), _ptr(act.T), _ptr(act.ws),
                                             act.ws_bytes, _stream()), "bwla_rotate_quant_bits")
        act.act_bits = int(act_bits)
    return act


def decode_forward(layer: PackedLayer, X, act: Activations, Y, acc=None, act_bits: int = 6):
    """bwla_rotate_quant + bwla_linear_forward in one call (one kernel launch where possible)."""
    xd = _xdtype(X)
    M = X.shape[0]
    if M > 64 and act.room is not None:                                     # (up to 64 tokens nothing is laid out)
        _check(load().bwla_decode_forward_room(layer._ref, _ptr(X), xd, int(act_bits), M, _ptr(act.q),
                                               _ptr(act.scale), _ptr(act.qsum), _ptr(act.T), _ptr(act.ws), act.ws_bytes,
                                               _ptr(act.room), act.room_bytes, _ptr(Y), _ptr(acc), _stream()),
               "bwla_decode_forward_room")
    elif act_bits == 6:
        # (a call of one token takes the host as long as the GPU: no conversion here)
        _check(load().bwla_decode_forward(layer._ref, _ptr(X), xd, M, _ptr(act.q), _ptr(act.scale),
                                          _ptr(act.qsum), _ptr(act.T), _ptr(act.ws), act.ws_bytes, _ptr(Y), _ptr(acc),
                                          _stream()), "bwla_decode_forward")
        act.act_bits = 6
        return Y
    else:
        _check(load().bwla_decode_forward_bits(layer._ref, _ptr(X), xd, int(act_bits), M, _ptr(act.q),
                                               _ptr(act.scale), _ptr(act.qsum), _ptr(act.T), _ptr(act.ws), act.ws_bytes,
                                               _ptr(Y), _ptr(acc), _stream()), "bwla_decode_forward_bits")
    act.act_bits = int(act_bits)
    return Y


def decode_forward_launches(layer: PackedLayer, M: int, bf16: bool = True) -> int:
    n = c_int()
    _check(load().bwla_decode_forward_launches(layer._ref, BWLA_X_BF16 if bf16 else BWLA_X_F32, M, byref(n)),
           "bwla_decode_forward_launches")
    return n.value


def decode_forward_static(layer: PackedLayer, X, act: Activations, Y, acc=None):
    """bwla_decode_forward with the library's own fixed scratch (act.ws is not used)."""
    xd = _xdtype(X)
    _check(load().bwla_decode_forward_static(layer._ref, _ptr(X), xd, X.shape[0], _ptr(act.q), _ptr(act.scale),
                                             _ptr(act.qsum), _ptr(act.T), _ptr(Y), _ptr(acc), _stream()),
           "bwla_decode_forward_static")
    return Y


def probe_hbm_read(src, sink) -> None:
    """One streaming read of the whole tensor `src` (measurement aid)."""
    _check(load().bwla_probe_hbm_read(_ptr(src), src.numel() * src.element_size(), _ptr(sink),
                                      sink.numel() * sink.element_size(), _stream()), "bwla_probe_hbm_read")


def probe_mfma_int8(iters: int, sink) -> int:
    """One launch of back-to-back INT8 MFMAs (measurement aid); returns its operation count."""
    ops = ctypes.c_int64()
    _check(load().bwla_probe_mfma_int8(int(iters), _ptr(sink), sink.numel() * sink.element_size(), byref(ops),
                                       _stream()), "bwla_probe_mfma_int8")
    return ops.value


def probe_empty_launch() -> None:
    _check(load().bwla_probe_empty_launch(_stream()), "bwla_probe_empty_launch")


def probe_clock(out) -> None:
    """out: int64 CUDA tensor of one element; gets the GPU's 100 MHz counter when the launch runs."""
    _check(load().bwla_probe_clock(_ptr(out), _stream()), "bwla_probe_clock")


def probe_load_latency(buf, stride_bytes: int, iters: int, out) -> None:
    """out: int64 CUDA tensor of two elements (ticks of 10 ns, last index)."""
    _check(load().bwla_probe_load_latency(_ptr(buf), buf.numel() * buf.element_size(), stride_bytes, iters, _ptr(out),
                                          _stream()), "bwla_probe_load_latency")


def pack_codes_a4(q, q4=None):
    """int8 codes in [-8, 7] (M x K) -> nibble-packed codes (M x K / 2 bytes)."""
    import torch
    if q4 is None:
        q4 = torch.empty((q.shape[0], q.shape[1] // 2), dtype=torch.uint8, device=q.device)
    _check(load().bwla_pack_codes_a4(_ptr(q), q.shape[0], q.shape[1], _ptr(q4), _stream()), "bwla_pack_codes_a4")
    return q4


def linear_forward_a4(layer: PackedLayer, q4, act: Activations, Y, acc=None):
    """bwla_linear_forward on nibble-packed 4-bit codes (scale, code sums and T from `act`)."""
    _check(load().bwla_linear_forward_a4(layer._ref, _ptr(q4), _ptr(act.scale), _ptr(act.qsum), _ptr(act.T),
                                         act.M, _ptr(Y), _ptr(acc), _stream()), "bwla_linear_forward_a4")
    return Y


def linear_forward_kernel(M: int, N: int, K: int, r: int, act_bits: int = 8, nibbles: bool = False) -> str:
    """Name of the kernel that linear_forward (of codes of act_bits), or linear_forward_a4, runs; r: columns of V."""
    out = c_char_p()
    _check(load().bwla_linear_forward_kernel(M, N, K, r, act_bits, int(nibbles), byref(out)), "bwla_linear_forward_kernel")
    return out.value.decode()


def code_sums(q, qsum) -> None:
    _check(load().bwla_code_sums(_ptr(q), q.shape[0], q.shape[1], _ptr(qsum), _stream()), "bwla_code_sums")


def swiglu_workspace_size(layer: PackedLayer, M: int) -> int:
    out = c_size_t()
    _check(load().bwla_swiglu_workspace_size(layer._ref, M, byref(out)), "bwla_swiglu_workspace_size")
    return out.value


def linear_forward_swiglu(layer: PackedLayer, act: Activations, H, ws=None):
    """H (bf16, M x N/2) = silu(gate) * up of a layer whose rows interleave gate and up channels.  Of `act` only room is
    written; ws is the gating workspace (swiglu_workspace_size)."""
    nbytes = 0 if ws is None else ws.numel() * ws.element_size()
    if act.act_bits <= 7:
        _check(load().bwla_linear_forward_swiglu_room(layer._ref, _ptr(act.q), _ptr(act.scale), _ptr(act.qsum),
                                                      _ptr(act.T), act.M, act.act_bits, _ptr(act.room), act.room_bytes,
                                                      _ptr(H), _ptr(ws), nbytes, _stream()),
               "bwla_linear_forward_swiglu_room")
        return H
    _check(load().bwla_linear_forward_swiglu(layer._ref, _ptr(act.q), _ptr(act.scale), _ptr(act.qsum),
                                             _ptr(act.T), act.M, _ptr(H), _ptr(ws), nbytes, _stream()),
           "bwla_linear_forward_swiglu")
    return H


def linear_forward(layer: PackedLayer, act: Activations, Y, acc=None):
    """Y from the codes in `act`, of which only room is written."""
    if act.act_bits <= 7:
        _check(load().bwla_linear_forward_room(layer._ref, _ptr(act.q), _ptr(act.scale), _ptr(act.qsum), _ptr(act.T),
                                               act.M, act.act_bits, _ptr(act.room), act.room_bytes, _ptr(Y), _ptr(acc),
                                               _stream()), "bwla_linear_forward_room")
        return Y
    _check(load().bwla_linear_forward(layer._ref, _ptr(act.q), _ptr(act.scale), _ptr(act.qsum), _ptr(act.T),
                                      act.M, _ptr(Y), _ptr(acc), _stream()), "bwla_linear_forward")
    return Y
