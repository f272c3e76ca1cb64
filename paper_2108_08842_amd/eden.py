"""ctypes binding of the EDEN C ABI (include/eden.h).  Argument marshalling only.

Tensors are torch CUDA(HIP) tensors; the binding passes their `data_ptr()` and the current torch
stream to the library.  Nothing here computes: every step of the path runs in the HIP kernels.
"""
from __future__ import annotations

import ctypes
import os
from array import array
from operator import index
from typing import Optional, Sequence

_PKG = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(_PKG, "libeden_hip.so")
_lib = None

OK = 0
ERR_INVALID_ARG = -1
ERR_CAPACITY = -2
ERR_HIP = -3
ERR_NO_DEVICE = -4
ERR_STATIC_LIMIT = -5
STATIC_MAX_D = 1 << 20
STATIC_MAX_N = 8
DEV_ZERO_VECTOR = 1
DEV_NONFINITE = 2
DEV_HEADER_MISMATCH = 4
DEV_NOTHING_ARRIVED = 8
HEADER_BYTES = 64
PACKET_COORDS = 1024

EXPORTS = [
    "eden_create", "eden_destroy", "eden_message_bytes", "eden_encode", "eden_decode_accumulate",
    "eden_finalize_mean", "eden_last_device_status", "eden_make_loss_bitmap", "eden_make_sign_bits",
    "eden_make_subsample_bits", "eden_get_tables", "eden_strerror", "eden_profile_enable", "eden_profile_collect",
    "eden_kernel_name", "eden_sq_error", "eden_index_entropy", "eden_encode_static",
    "eden_last_decode_flags", "eden_message_length", "eden_decode_mean",
]
_SEED_MASK = 2 ** 64 - 1
B_HALF_PRE = 0x10080     # b = 1/2 with the sparsification before the rotation (EDEN_B_HALF_PRE)


def B_GRID(delta: float) -> int:
    """Uniform-grid quantizer of Sec. 4.3 with step `delta` (0 < delta < 2): EDEN_B_GRID(round(delta * 32768))."""
    q = int(round(delta * 32768))
    assert 1 <= q <= 65535
    return 0x30000 | q


def B_SPARSE(m: int) -> int:
    """b = m/64, 1 <= m <= 63: m of every 64 coordinates are kept before the rotation (EDEN_B_SPARSE(m))."""
    assert 1 <= m <= 63
    return 0x20000 | m


def B_COIN(b: float) -> int:
    """General non-integer budget 1 < b < 4 (Sec. 4.1): every coordinate gets the extra bit with probability b - floor(b),
    by an independent coin from the shared seed (EDEN_B_COIN(round(256 b)))."""
    q = int(round(256 * b))
    assert 256 < q < 1024 and q % 256 != 0
    return 0x40000 | q


KERNEL_KINDS = ["enc_first", "mid", "enc_last", "dec_prepare", "dec_first", "dec_last", "finalize_mean",
                "enc_small", "dec_small", "enc_norm", "enc_finish"]


class EdenError(RuntimeError):
    def __init__(self, code: int, what: str):
        super().__init__(f"{what}: {strerror(code)} ({code})")
        self.code = code


def lib():
    """Loads the built library; raises if it has not been built (there is no fallback path)."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(_LIB_PATH):
        raise FileNotFoundError(
            f"{_LIB_PATH} is missing: build it with `python -m paper_2108_08842_amd.build` "
            "(or __graft_entry__.build()); the EDEN path has no CPU fallback")
    L = ctypes.CDLL(_LIB_PATH)
    vp, u64, u32, sz, ci = ctypes.c_void_p, ctypes.c_uint64, ctypes.c_uint32, ctypes.c_size_t, ctypes.c_int
    P = ctypes.POINTER
    L.eden_create.argtypes = [P(vp), u64, u32, ci]
    L.eden_create.restype = ci
    L.eden_destroy.argtypes = [vp]
    L.eden_destroy.restype = ci
    L.eden_message_bytes.argtypes = [u64, u32]
    L.eden_message_bytes.restype = sz
    # (the arrays of a batch travel as addresses: see _elements)
    L.eden_encode.argtypes = [vp, vp, vp, vp, u32, u64, u64, vp, vp, vp]
    L.eden_encode.restype = ci
    L.eden_encode_static.argtypes = [vp, vp, vp, u32, u64, u64, vp, vp, vp]
    L.eden_encode_static.restype = ci
    L.eden_decode_accumulate.argtypes = [vp, vp, vp, vp, u32, u64, u64, vp, vp, vp]
    L.eden_decode_accumulate.restype = ci
    L.eden_decode_mean.argtypes = [vp, vp, vp, vp, u32, u64, u64, vp, vp, vp]
    L.eden_decode_mean.restype = ci
    L.eden_finalize_mean.argtypes = [vp, vp, u64, u32, vp, vp]
    L.eden_finalize_mean.restype = ci
    L.eden_last_decode_flags.argtypes = [vp, vp, P(u32), u32]
    L.eden_last_decode_flags.restype = ci
    L.eden_message_length.argtypes = [vp]
    L.eden_message_length.restype = sz
    L.eden_last_device_status.argtypes = [vp, vp, P(u32)]
    L.eden_last_device_status.restype = ci
    L.eden_make_loss_bitmap.argtypes = [vp, u64, u32, u64, u32, vp, vp]
    L.eden_make_loss_bitmap.restype = ci
    L.eden_make_sign_bits.argtypes = [vp, u64, u32, u64, vp, vp]
    L.eden_make_sign_bits.restype = ci
    L.eden_make_subsample_bits.argtypes = [vp, u64, u32, u64, vp, vp]
    L.eden_make_subsample_bits.restype = ci
    L.eden_get_tables.argtypes = [u32, P(ctypes.c_double), P(ctypes.c_double)]
    L.eden_get_tables.restype = ci
    L.eden_strerror.argtypes = [ci]
    L.eden_strerror.restype = ctypes.c_char_p
    L.eden_profile_enable.argtypes = [vp, u32, u32]
    L.eden_profile_enable.restype = ci
    L.eden_profile_collect.argtypes = [vp, P(u32), P(u32), P(ctypes.c_float), u32, P(u32)]
    L.eden_profile_collect.restype = ci
    L.eden_kernel_name.argtypes = [u32]
    L.eden_kernel_name.restype = ctypes.c_char_p
    L.eden_sq_error.argtypes = [vp, vp, vp, u64, vp, vp]
    L.eden_sq_error.restype = ci
    L.eden_index_entropy.argtypes = [vp, vp, u64, u32, vp, vp]
    L.eden_index_entropy.restype = ci
    _lib = L
    return L


def strerror(code: int) -> str:
    return lib().eden_strerror(code).decode()


def message_bytes(d: int, b_q8: int) -> int:
    return int(lib().eden_message_bytes(d, b_q8))


def message_length(header: bytes) -> int:
    """Bytes of a message that have to travel, from a host copy of (at least) its 64-byte header."""
    assert len(header) >= HEADER_BYTES
    buf = ctypes.create_string_buffer(bytes(header[:HEADER_BYTES]), HEADER_BYTES)
    return int(lib().eden_message_length(ctypes.cast(buf, ctypes.c_void_p)))


def get_tables(bits: int):
    n = 1 << bits
    t = (ctypes.c_double * (n - 1))()
    q = (ctypes.c_double * n)()
    rc = lib().eden_get_tables(bits, t, q)
    if rc != OK:
        raise EdenError(rc, "eden_get_tables")
    return list(t), list(q)


def _stream_ptr(stream=None):
    """Address of a stream, by default the current one of the current device (without a Stream object around it where torch
    offers that)."""
    import torch
    if stream is not None:
        return stream.cuda_stream
    try:
        return torch._C._cuda_getCurrentRawStream(torch.cuda.current_device())
    except AttributeError:
        return torch.cuda.current_stream().cuda_stream


# Arrays of a batch as (object that owns the memory, address): the C side takes them by address and copies what it needs before
# the call returns.  The array module builds them several times faster than ctypes does, which matters for calls whose kernels
# take a few microseconds.
def _elements(values):
    """A sequence as a list of its elements (the array module would take bytes as raw memory, and an iterator that fails half
    way could not be read again: without a length it is refused)."""
    len(values)
    return list(values)


def _u64s(values):
    if type(values) is not list:
        values = _elements(values)
    try:
        a = array("Q", values)
    except (TypeError, OverflowError):                           # anything int() takes
        a = array("Q", [int(v) & _SEED_MASK for v in values])
    return a, a.buffer_info()[0]


def _u32s(values):
    if type(values) is not list:
        values = _elements(values)
    try:
        a = array("I", values)
    except (TypeError, OverflowError):
        a = array("I", [int(v) & 0xFFFFFFFF for v in values])
    return a, a.buffer_info()[0]


def _ptrs(values):
    if type(values) is not list:
        values = _elements(values)
    try:
        a = array("Q", values)
    except (TypeError, OverflowError):                           # None is a null pointer; no conversions
        a = array("Q", [0 if v is None else index(v) & _SEED_MASK for v in values])
    return a, a.buffer_info()[0]


def _ptrs_or_null(ptrs):
    return (None, None) if ptrs is None else _ptrs(ptrs)        # null: no bitmap at all, or none for that sender


def _device_ptrs(tensors):
    return [t.data_ptr() for t in tensors]


def encode_static_raw(x_ptrs, client_ids, b_q8, d, seed, msg_ptrs, msg_caps, stream=None) -> int:
    """eden_encode_static on the current device: the library's status code, nothing raised."""
    x, ids, b, m, caps = _ptrs(x_ptrs), _u32s(client_ids), _u32s(b_q8), _ptrs(msg_ptrs), _u64s(msg_caps)
    return lib().eden_encode_static(x[1], ids[1], b[1], len(x_ptrs), d, seed & _SEED_MASK, m[1], caps[1], _stream_ptr(stream))


def encode_static(xs, client_ids, b_q8, seed: int, msgs, stream=None):
    """The sender side without a context and without any allocation: `msgs` are caller-allocated uint8 tensors."""
    d = xs[0].numel()
    rc = encode_static_raw(_device_ptrs(xs), client_ids, b_q8, d, seed, _device_ptrs(msgs), [m.numel() for m in msgs], stream)
    if rc != OK:
        raise EdenError(rc, "eden_encode_static")
    return msgs


class Context:
    """Owns one eden_ctx (workspace + tables) on a HIP device."""

    def __init__(self, d_max: int, n_max: int, device: int = 0):
        h = ctypes.c_void_p()
        rc = lib().eden_create(ctypes.byref(h), d_max, n_max, device)
        if rc != OK:
            raise EdenError(rc, "eden_create")
        self._h = h
        self.d_max, self.n_max, self.device = d_max, n_max, device

    def close(self):
        if self._h:
            lib().eden_destroy(self._h)
            self._h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    # ---- raw calls: return the library's status code, raise nothing
    def encode_raw(self, x_ptrs, client_ids, b_q8, d, seed, msg_ptrs, msg_caps, stream=None) -> int:
        x, ids, b, m, caps = _ptrs(x_ptrs), _u32s(client_ids), _u32s(b_q8), _ptrs(msg_ptrs), _u64s(msg_caps)
        return lib().eden_encode(self._h, x[1], ids[1], b[1], len(x_ptrs), d, seed & _SEED_MASK, m[1], caps[1], _stream_ptr(stream))

    def decode_accumulate_raw(self, msg_ptrs, client_ids, b_q8, d, seed, bitmap_ptrs, acc_ptr, stream=None) -> int:
        m, ids, b, bm = _ptrs(msg_ptrs), _u32s(client_ids), _u32s(b_q8), _ptrs_or_null(bitmap_ptrs)
        return lib().eden_decode_accumulate(self._h, m[1], ids[1], b[1], len(msg_ptrs), d, seed & _SEED_MASK, bm[1], acc_ptr,
                                            _stream_ptr(stream))

    def decode_mean_raw(self, msg_ptrs, client_ids, b_q8, d, seed, bitmap_ptrs, mean_ptr, stream=None) -> int:
        m, ids, b, bm = _ptrs(msg_ptrs), _u32s(client_ids), _u32s(b_q8), _ptrs_or_null(bitmap_ptrs)
        return lib().eden_decode_mean(self._h, m[1], ids[1], b[1], len(msg_ptrs), d, seed & _SEED_MASK, bm[1], mean_ptr,
                                      _stream_ptr(stream))

    def finalize_mean_raw(self, acc_ptr, d, n, mean_ptr, stream=None) -> int:
        return lib().eden_finalize_mean(self._h, ctypes.c_void_p(acc_ptr), d, n, ctypes.c_void_p(mean_ptr),
                                        _stream_ptr(stream))

    # ---- tensor-level convenience (allocation + marshalling only)
    def alloc_messages(self, d: int, b_q8: Sequence[int]):
        import torch
        return [torch.empty(message_bytes(d, b), dtype=torch.uint8, device=f"cuda:{self.device}") for b in b_q8]

    def encode(self, xs, client_ids, b_q8, seed: int, msgs=None, stream=None):
        d = xs[0].numel()
        import torch
        for x in xs:
            assert x.is_cuda and x.dtype is torch.float32 and x.is_contiguous() and x.numel() == d
        if msgs is None:
            msgs = self.alloc_messages(d, b_q8)
        rc = self.encode_raw(_device_ptrs(xs), client_ids, b_q8, d, seed, _device_ptrs(msgs), [m.numel() for m in msgs], stream)
        if rc != OK:
            raise EdenError(rc, "eden_encode")
        return msgs

    def decode_accumulate(self, msgs, client_ids, b_q8, d: int, seed: int, acc, bitmaps=None, stream=None):
        assert acc.is_cuda and acc.element_size() == 4 and acc.numel() == d and acc.is_contiguous()
        bm = None if bitmaps is None else [None if b is None else b.data_ptr() for b in bitmaps]
        rc = self.decode_accumulate_raw(_device_ptrs(msgs), client_ids, b_q8, d, seed, bm,
                                        acc.data_ptr(), stream)
        if rc != OK:
            raise EdenError(rc, "eden_decode_accumulate")
        return acc

    def decode_mean(self, msgs, client_ids, b_q8, d: int, seed: int, mean, bitmaps=None, stream=None):
        """The receiver's whole round: mean = (1/n) sum of the n decoded vectors, written (not added) to `mean`."""
        assert mean.is_cuda and mean.element_size() == 4 and mean.numel() == d and mean.is_contiguous()
        bm = None if bitmaps is None else [None if b is None else b.data_ptr() for b in bitmaps]
        rc = self.decode_mean_raw(_device_ptrs(msgs), client_ids, b_q8, d, seed, bm, mean.data_ptr(), stream)
        if rc != OK:
            raise EdenError(rc, "eden_decode_mean")
        return mean

    def finalize_mean(self, acc, n: int, out=None, stream=None):
        out = acc if out is None else out
        rc = self.finalize_mean_raw(acc.data_ptr(), acc.numel(), n, out.data_ptr(), stream)
        if rc != OK:
            raise EdenError(rc, "eden_finalize_mean")
        return out

    def last_device_status(self, stream=None) -> int:
        v = ctypes.c_uint32(0)
        rc = lib().eden_last_device_status(self._h, _stream_ptr(stream), ctypes.byref(v))
        if rc != OK:
            raise EdenError(rc, "eden_last_device_status")
        return int(v.value)

    def last_decode_flags(self, n: int, stream=None):
        """Status bits of the first n messages of the most recent decode_accumulate / decode_mean call, in call order."""
        out = (ctypes.c_uint32 * n)()
        rc = lib().eden_last_decode_flags(self._h, _stream_ptr(stream), out, n)
        if rc != OK:
            raise EdenError(rc, "eden_last_decode_flags")
        return [int(v) for v in out]

    def profile_enable(self, kinds, max_records: int = 4096):
        """Time every launch of the named kernel kinds with HIP events (empty list = off)."""
        mask = 0
        for k in kinds:
            mask |= 1 << KERNEL_KINDS.index(k)
        rc = lib().eden_profile_enable(self._h, mask, max_records)
        if rc != OK:
            raise EdenError(rc, "eden_profile_enable")

    def profile_collect(self, cap: int = 4096):
        """-> list of (kernel kind name, senders in the launch, milliseconds), in launch order."""
        kinds = (ctypes.c_uint32 * cap)()
        senders = (ctypes.c_uint32 * cap)()
        ms = (ctypes.c_float * cap)()
        cnt = ctypes.c_uint32(0)
        rc = lib().eden_profile_collect(self._h, kinds, senders, ms, cap, ctypes.byref(cnt))
        if rc != OK:
            raise EdenError(rc, "eden_profile_collect")
        return [(KERNEL_KINDS[kinds[i]], int(senders[i]), float(ms[i])) for i in range(cnt.value)]

    def make_loss_bitmap(self, seed: int, client: int, D: int, drop_q32: int, stream=None):
        import torch
        npk = max(1, D // PACKET_COORDS)
        out = torch.empty((npk + 31) // 32, dtype=torch.int32, device=f"cuda:{self.device}")
        rc = lib().eden_make_loss_bitmap(self._h, ctypes.c_uint64(seed), client, D, drop_q32,
                                         ctypes.c_void_p(out.data_ptr()), _stream_ptr(stream))
        if rc != OK:
            raise EdenError(rc, "eden_make_loss_bitmap")
        return out

    def index_entropy(self, msg, d: int, b_q8: int, stream=None):
        """-> device tensor of 1 double: empirical entropy (bits per coordinate) of a uniform-grid message."""
        import torch
        out = torch.empty(1, dtype=torch.float64, device=msg.device)
        rc = lib().eden_index_entropy(self._h, ctypes.c_void_p(msg.data_ptr()), d, b_q8, ctypes.c_void_p(out.data_ptr()),
                                      _stream_ptr(stream))
        if rc != OK:
            raise EdenError(rc, "eden_index_entropy")
        return out

    def sq_error(self, a, b, out=None, stream=None):
        """-> device tensor of 2 doubles: sum (a - b)^2, sum a^2 (asynchronous)."""
        import torch
        assert a.is_cuda and b.is_cuda and a.dtype == torch.float32 and b.dtype == torch.float32
        assert a.is_contiguous() and b.is_contiguous() and a.numel() == b.numel()
        if out is None:
            out = torch.empty(2, dtype=torch.float64, device=a.device)
        rc = lib().eden_sq_error(self._h, ctypes.c_void_p(a.data_ptr()), ctypes.c_void_p(b.data_ptr()), a.numel(),
                                 ctypes.c_void_p(out.data_ptr()), _stream_ptr(stream))
        if rc != OK:
            raise EdenError(rc, "eden_sq_error")
        return out

    def make_sign_bits(self, seed: int, client: int, D: int, stream=None):
        import torch
        out = torch.empty(max(1, D // 64), dtype=torch.int64, device=f"cuda:{self.device}")
        rc = lib().eden_make_sign_bits(self._h, ctypes.c_uint64(seed), client, D, ctypes.c_void_p(out.data_ptr()),
                                       _stream_ptr(stream))
        if rc != OK:
            raise EdenError(rc, "eden_make_sign_bits")
        return out

    def make_subsample_bits(self, seed: int, client: int, D: int, stream=None):
        import torch
        out = torch.empty(max(1, D // 128), dtype=torch.int64, device=f"cuda:{self.device}")
        rc = lib().eden_make_subsample_bits(self._h, ctypes.c_uint64(seed), client, D,
                                            ctypes.c_void_p(out.data_ptr()), _stream_ptr(stream))
        if rc != OK:
            raise EdenError(rc, "eden_make_subsample_bits")
        return out
