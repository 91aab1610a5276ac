"""ctypes binding of libpbkv.so: same names as the C boundary, argument marshalling only.

Every operation runs in the HIP kernels of the library.  There is no CPU or PyTorch
fallback: if the library has not been built, or a call fails, an exception is raised.
Tensors may be torch tensors (anything with ``data_ptr()``) or raw integer addresses;
``prefix_lens`` / ``new_lens`` / ``page_ids`` are host int32 arrays.
"""
import ctypes
import os

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(HERE, "libpbkv.so")

PBKV_BF16, PBKV_F32 = 0, 1
STATUS = {0: "PBKV_OK", -1: "PBKV_ERR_NULL", -2: "PBKV_ERR_SHAPE", -3: "PBKV_ERR_DTYPE",
          -4: "PBKV_ERR_RANGE", -5: "PBKV_ERR_ALIAS", -6: "PBKV_ERR_DEVICE", -7: "PBKV_ERR_LIMIT"}


class PbkvError(RuntimeError):
    def __init__(self, code, message):
        super().__init__("%s (%d): %s" % (STATUS.get(code, "?"), code, message))
        self.code = code


class Shape(ctypes.Structure):
    _fields_ = [("batch", ctypes.c_int32), ("num_q_heads", ctypes.c_int32),
                ("num_kv_heads", ctypes.c_int32), ("head_dim", ctypes.c_int32),
                ("page_size", ctypes.c_int32), ("num_pages", ctypes.c_int32),
                ("max_pages_per_req", ctypes.c_int32), ("dtype", ctypes.c_int32)]


_lib = None


def fast(lib, name, kinds, shape_type):
    """The C function as a callable that takes a binding function's arguments as they are (csrc/calls.cpp), or returns None
    where one of them needs converting."""
    try:
        from . import _calls
    except ImportError as e:
        raise ImportError("the extension _calls is not built for this interpreter: run `python -m paper_2605_06472_amd.build` "
                          "(there is no fallback path)") from e
    _calls.numpy(np.ndarray)
    return _calls.bind(ctypes.cast(getattr(lib, name), ctypes.c_void_p).value, kinds, shape_type)


def load():
    """Load libpbkv.so (built by paper_2605_06472_amd.build); raises if it is missing."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise ImportError("libpbkv.so is not built: run `python -m paper_2605_06472_amd.build` "
                              "(there is no fallback path)")
        lib = ctypes.CDLL(LIB_PATH)
        vp, i32p = ctypes.c_void_p, ctypes.c_void_p
        sp = ctypes.POINTER(Shape)
        lib.pbkv_prefix_prefill.restype = ctypes.c_int
        lib.pbkv_prefix_prefill.argtypes = [sp, vp, vp, vp, vp, i32p, i32p, i32p, vp, vp]
        lib.pbkv_append_kv.restype = ctypes.c_int
        lib.pbkv_append_kv.argtypes = [sp, vp, vp, vp, i32p, i32p, i32p, vp]
        lib.pbkv_swap_in_pages.restype = ctypes.c_int
        lib.pbkv_swap_in_pages.argtypes = [sp, vp, i32p, ctypes.c_int32, vp, vp]
        lib.pbkv_paged_decode.restype = ctypes.c_int
        lib.pbkv_paged_decode.argtypes = [sp, vp, vp, i32p, i32p, vp, vp]
        lib.pbkv_paged_decode_static.restype = ctypes.c_int
        lib.pbkv_paged_decode_static.argtypes = [sp, vp, vp, i32p, i32p, vp, vp]
        lib.pbkv_swap_out_pages.restype = ctypes.c_int
        lib.pbkv_swap_out_pages.argtypes = [sp, vp, i32p, ctypes.c_int32, vp, vp]
        lib.pbkv_gather_probe.restype = ctypes.c_int
        lib.pbkv_gather_probe.argtypes = [sp, vp, vp, vp, i32p, i32p, i32p, vp, ctypes.c_int64,
                                          ctypes.POINTER(ctypes.c_int64), ctypes.POINTER(ctypes.c_int32), vp]
        lib.pbkv_set_attn_waves.restype = ctypes.c_int
        lib.pbkv_set_attn_waves.argtypes = [ctypes.c_int]
        lib.pbkv_page_bytes.restype = ctypes.c_int64
        lib.pbkv_page_bytes.argtypes = [sp]
        lib.pbkv_last_error.restype = ctypes.c_char_p
        lib.pbkv_version.restype = ctypes.c_char_p
        for name, kinds in (("prefix_prefill", "spppppiipt"), ("append_kv", "sppppiit"), ("paged_decode", "spppipt"),
                            ("paged_decode_static", "spppipt"), ("swap_in_pages", "spiNpt"), ("swap_out_pages", "spiNpt")):
            setattr(lib, "fast_" + name, fast(lib, "pbkv_" + name, kinds, Shape))
        _lib = lib
    return _lib


# A call's host cost matters where a decode step makes thousands of small ones, so arguments in their ordinary forms (tensors or
# addresses, int32 arrays) go straight to native code (lib.fast_*): append_kv without the boundary's own work 3.8 -> 1.0 us on one
# host; a small prefill with append 11.4 -> 8.9 us per pass.  Everything else goes through ctypes: the conversions
# below.
def _ptr(t):
    if t is None or isinstance(t, int):
        return t
    return t.data_ptr()


_I32 = np.dtype(np.int32)


def _host_i32(a):
    """The int32 array behind `a` (to be kept until the call returns) and its address for ctypes."""
    if type(a) is np.ndarray and a.dtype == _I32 and a.ndim == 1:
        try:
            return a, ctypes.byref(ctypes.c_int32.from_buffer(a))
        except (TypeError, ValueError):       # read-only, strided or empty: the general way below
            pass
    if hasattr(a, "data_ptr") and not isinstance(a, np.ndarray):      # torch CPU tensor
        a = a.numpy()
    a = np.ascontiguousarray(a, dtype=np.int32)
    return a, a.ctypes.data


_torch = None


def _stream(stream):
    global _torch
    if stream is None:
        first = _torch is None
        if first:
            import torch
            _torch = torch
        # the same stream as torch.cuda.current_stream(), without building an object for it
        current = _torch._C._cuda_getCurrentRawStream(_torch.cuda.current_device())
        if first:                                # torch is up: from now on native code asks it, without the check for a
            from . import _calls                 # forked child that current_device() makes, so not in such a child
            os.register_at_fork(after_in_child=lambda: _calls.torch(None, None))
            _calls.torch(_torch._C._cuda_getDevice, _torch._C._cuda_getCurrentRawStream)
        return current
    if isinstance(stream, int):
        return stream
    return stream.cuda_stream


def _check(rc):
    if rc != 0:
        raise PbkvError(rc, load().pbkv_last_error().decode())


def make_shape(batch, num_q_heads, num_kv_heads, head_dim, page_size, num_pages,
               max_pages_per_req, dtype):
    code = {"bf16": PBKV_BF16, "f32": PBKV_F32}.get(dtype, dtype)
    return Shape(batch, num_q_heads, num_kv_heads, head_dim, page_size, num_pages,
                 max_pages_per_req, code)


def page_bytes(shape):
    return int(load().pbkv_page_bytes(ctypes.byref(shape)))


def version():
    return load().pbkv_version().decode()


def set_attn_waves(waves):
    """4, 8 or 64: work-group shape of every later bf16 attention launch; 0: the library chooses."""
    _check(load().pbkv_set_attn_waves(int(waves)))


def prefix_prefill(shape, q, k_new, v_new, kv_pool, block_table, prefix_lens, new_lens, out,
                   stream=None):
    rc = load().fast_prefix_prefill(shape, q, k_new, v_new, kv_pool, block_table, prefix_lens, new_lens, out, stream)
    if rc is not None:
        return _check(rc)
    pl, plp = _host_i32(prefix_lens)
    nl, nlp = _host_i32(new_lens)
    _check(load().pbkv_prefix_prefill(ctypes.byref(shape), _ptr(q), _ptr(k_new), _ptr(v_new),
                                      _ptr(kv_pool), _ptr(block_table), plp, nlp, _ptr(out),
                                      _stream(stream)))


def append_kv(shape, k_new, v_new, kv_pool, block_table, prefix_lens, new_lens, stream=None):
    rc = load().fast_append_kv(shape, k_new, v_new, kv_pool, block_table, prefix_lens, new_lens, stream)
    if rc is not None:
        return _check(rc)
    pl, plp = _host_i32(prefix_lens)
    nl, nlp = _host_i32(new_lens)
    _check(load().pbkv_append_kv(ctypes.byref(shape), _ptr(k_new), _ptr(v_new), _ptr(kv_pool),
                                 _ptr(block_table), plp, nlp, _stream(stream)))


def swap_in_pages(shape, host_pages, page_ids, kv_pool, stream=None):
    rc = load().fast_swap_in_pages(shape, host_pages, page_ids, kv_pool, stream)
    if rc is not None:
        return _check(rc)
    ids, idp = _host_i32(page_ids)
    _check(load().pbkv_swap_in_pages(ctypes.byref(shape), _ptr(host_pages), idp,
                                     int(ids.shape[0]), _ptr(kv_pool), _stream(stream)))


def paged_decode(shape, q, kv_pool, block_table, context_lens, out, stream=None):
    rc = load().fast_paged_decode(shape, q, kv_pool, block_table, context_lens, out, stream)
    if rc is not None:
        return _check(rc)
    cl, clp = _host_i32(context_lens)
    _check(load().pbkv_paged_decode(ctypes.byref(shape), _ptr(q), _ptr(kv_pool), _ptr(block_table), clp,
                                    _ptr(out), _stream(stream)))


def paged_decode_static(shape, q, kv_pool, block_table, context_lens, out, stream=None):
    rc = load().fast_paged_decode_static(shape, q, kv_pool, block_table, context_lens, out, stream)
    if rc is not None:
        return _check(rc)
    cl, clp = _host_i32(context_lens)
    _check(load().pbkv_paged_decode_static(ctypes.byref(shape), _ptr(q), _ptr(kv_pool), _ptr(block_table), clp,
                                           _ptr(out), _stream(stream)))


def swap_out_pages(shape, kv_pool, page_ids, host_pages, stream=None):
    rc = load().fast_swap_out_pages(shape, kv_pool, page_ids, host_pages, stream)
    if rc is not None:
        return _check(rc)
    ids, idp = _host_i32(page_ids)
    _check(load().pbkv_swap_out_pages(ctypes.byref(shape), _ptr(kv_pool), idp, int(ids.shape[0]),
                                      _ptr(host_pages), _stream(stream)))


def gather_probe(shape, k_new, v_new, kv_pool, block_table, prefix_lens, new_lens, unit_xor=None,
                 stream=None):
    """Returns (n_units, unit_tokens).  ``unit_xor`` is a device 32-bit integer tensor that
    receives one word per unit; None only asks for the two numbers."""
    pl, plp = _host_i32(prefix_lens)
    nl, nlp = _host_i32(new_lens)
    n_units, unit_tokens = ctypes.c_int64(0), ctypes.c_int32(0)
    cap = 0 if unit_xor is None else int(unit_xor.numel())
    _check(load().pbkv_gather_probe(ctypes.byref(shape), _ptr(k_new), _ptr(v_new), _ptr(kv_pool),
                                    _ptr(block_table), plp, nlp, _ptr(unit_xor), cap,
                                    ctypes.byref(n_units), ctypes.byref(unit_tokens),
                                    None if unit_xor is None else _stream(stream)))
    return n_units.value, unit_tokens.value
