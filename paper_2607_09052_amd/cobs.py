"""Thin Python binding of libcobs.so (the COBS decode-step C ABI, include/cobs.h).

Argument marshalling only: every stage runs in the library's HIP kernels.
Tensors are torch tensors on the GPU; torch supplies device memory and the
stream (the current stream of the tensors' device, unless one is passed).
A missing library raises at import of this module's functions' first use -
there is no other implementation to fall back to.
"""

import ctypes
import dataclasses
import math
import os

import torch

LIB_PATH = os.path.join(os.path.dirname(os.path.abspath(__file__)), "libcobs.so")

F32, BF16, E2M1 = 0, 1, 2
DTYPES = {"f32": F32, "bf16": BF16, "e2m1": E2M1}
OP_BUILD, OP_SELECT, OP_DECODE, OP_STEP, OP_SELECT_EXACT = 0, 1, 2, 3, 4
OPT_SKEW, OPT_VALUE_MEAN = 1, 2
BLOCK = 64


class CobsError(RuntimeError):
    pass


class _Config(ctypes.Structure):
    _fields_ = [("batch", ctypes.c_int32), ("num_q_heads", ctypes.c_int32),
                ("num_kv_heads", ctypes.c_int32), ("head_dim", ctypes.c_int32),
                ("max_seq_len", ctypes.c_int32), ("block_size", ctypes.c_int32),
                ("rank", ctypes.c_int32), ("budget", ctypes.c_int32), ("window", ctypes.c_int32),
                ("kv_dtype", ctypes.c_int), ("mean_dtype", ctypes.c_int),
                ("factor_dtype", ctypes.c_int), ("softmax_scale", ctypes.c_float),
                ("options", ctypes.c_int32), ("subspace_dim", ctypes.c_int32),
                ("query_basis", ctypes.c_void_p)]


class _KV(ctypes.Structure):
    _fields_ = [("k", ctypes.c_void_p), ("v", ctypes.c_void_p), ("stride_b", ctypes.c_int64),
                ("stride_h", ctypes.c_int64), ("stride_t", ctypes.c_int64),
                ("block_table", ctypes.c_void_p), ("num_pages", ctypes.c_int64)]


_P = ctypes.c_void_p
_SIGS = {
    "cobs_record_bytes": (ctypes.c_size_t, [_P]),
    "cobs_workspace_bytes": (ctypes.c_size_t, [_P, ctypes.c_int]),
    "cobs_build_block_stats": (ctypes.c_int, [_P, _P, _P, ctypes.c_int32, ctypes.c_int32, _P, _P,
                                              ctypes.c_size_t, _P]),
    "cobs_select": (ctypes.c_int, [_P, _P, _P, _P, _P, _P, _P, ctypes.c_size_t, _P]),
    "cobs_select_exact": (ctypes.c_int, [_P, _P, _P, _P, _P, _P, _P, ctypes.c_size_t, _P]),
    "cobs_select_quest": (ctypes.c_int, [_P, _P, _P, _P, _P, _P, _P, ctypes.c_size_t, _P]),
    "cobs_sparse_decode": (ctypes.c_int, [_P, _P, _P, _P, _P, _P, _P, _P, ctypes.c_size_t, _P]),
    "cobs_sparse_decode_branches": (ctypes.c_int, [_P, _P, _P, _P, _P, _P, _P, _P, _P, _P, ctypes.c_size_t, _P]),
    "cobs_decode_step": (ctypes.c_int, [_P, _P, _P, _P, _P, _P, _P, _P, _P, ctypes.c_size_t, _P]),
    "cobs_decode_step_noalloc": (ctypes.c_int, [_P, _P, _P, _P, _P, _P, _P, _P, _P]),
    "cobs_compression_branch": (ctypes.c_int, [_P, _P, _P, _P, _P, _P, _P]),
    "cobs_pack_e2m1": (ctypes.c_int, [_P, ctypes.c_int64, ctypes.c_int32, _P, _P, _P]),
    "cobs_status_string": (ctypes.c_char_p, [ctypes.c_int]),
}
EXPORTS = tuple(_SIGS)

_lib = None


def lib():
    """The loaded library (raises if it has not been built)."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise CobsError(f"{LIB_PATH} is missing: build it with `python -m paper_2607_09052_amd.build`")
        h = ctypes.CDLL(LIB_PATH)
        for name, (res, args) in _SIGS.items():
            fn = getattr(h, name)
            fn.restype = res
            fn.argtypes = args
        _lib = h
    return _lib


class _CForm:
    """The place of a Config's C form (Config.marshalled): outside its __dict__, so
    that vars(), comparisons, copies and pickles see the fields alone."""
    __slots__ = ("_c_form",)


@dataclasses.dataclass
class Config(_CForm):
    """Problem description (cobs_config_t)."""
    batch: int
    num_q_heads: int
    num_kv_heads: int
    head_dim: int
    max_seq_len: int
    rank: int
    budget: int
    window: int
    kv_dtype: str = "bf16"
    mean_dtype: str = "f32"
    factor_dtype: str = "f32"
    softmax_scale: float = 0.0
    block_size: int = BLOCK
    skew: bool = False           # records carry the diagonal third-cumulant coefficients
    value_mean: bool = False     # records carry the block's mean value (compression branch)
    subspace_dim: int = 0        # subspace factors of this many elements (Sec. 5.4); 0: full space
    # U_Q of every KV head for subspace factors: fp32 [Hkv, d, subspace_dim] on the GPU
    query_basis: object = dataclasses.field(default=None, compare=False, repr=False)

    def __setattr__(self, name, value):
        object.__setattr__(self, name, value)
        object.__setattr__(self, "_c_form", None)      # after the field: see marshalled

    def __getstate__(self):
        return self.__dict__

    def marshalled(self):
        """The C form of the fields: (struct, record bytes, K/V torch dtype or None).
        It is kept with a copy of the fields that it was made from, until a field is
        assigned, and used while they are equal: a field may also be set past
        __setattr__ (vars(), a new __dict__).  Only plain numbers and texts are
        kept: with anything that can change in place (a query basis, an array) the
        form is made anew for each call."""
        kept = getattr(self, "_c_form", None)
        if kept is not None and self.__dict__ == kept[0]:
            return kept[1]
        fields = dict(self.__dict__)
        plain = (type(self) is Config and fields.keys() == _FIELDS and fields["query_basis"] is None and
                 all(type(x) in _PLAIN for x in fields.values()))
        src = Config(**fields) if plain else self      # the values read, if another thread sets one meanwhile
        c = src.c_struct()
        form = (c, int(lib().cobs_record_bytes(ctypes.byref(c))), _TORCH_DTYPE.get(src.kv_dtype))
        if plain:
            object.__setattr__(self, "_c_form", (fields, form))
        return form

    @property
    def options(self):
        return (OPT_SKEW if self.skew else 0) | (OPT_VALUE_MEAN if self.value_mean else 0)

    def c_struct(self):
        basis = None
        if self.query_basis is not None:
            want = (self.num_kv_heads, self.head_dim, self.subspace_dim)
            _need("query_basis", self.query_basis, torch.float32, math.prod(want))
            if tuple(self.query_basis.shape) != want:
                raise CobsError(f"query_basis must have shape {list(want)}, got {list(self.query_basis.shape)}")
            basis = self.query_basis.data_ptr()
        return _Config(self.batch, self.num_q_heads, self.num_kv_heads, self.head_dim,
                       self.max_seq_len, self.block_size, self.rank, self.budget, self.window,
                       DTYPES[self.kv_dtype], DTYPES[self.mean_dtype], DTYPES[self.factor_dtype],
                       float(self.softmax_scale), self.options, int(self.subspace_dim), basis)

    @property
    def num_blocks(self):
        return self.max_seq_len // self.block_size

    @property
    def scale(self):
        return self.softmax_scale if self.softmax_scale > 0 else 1.0 / math.sqrt(self.head_dim)


_FIELDS = {f.name for f in dataclasses.fields(Config)}
_PLAIN = (int, float, bool, str, type(None))


def _ptr(t):
    return None if t is None else t.data_ptr()


_raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None)


def _stream(stream, dev_tensor):
    if stream is not None:
        return stream if isinstance(stream, int) else stream.cuda_stream
    if _raw_stream is not None:
        return _raw_stream(dev_tensor.get_device())
    return torch.cuda.current_stream(dev_tensor.device).cuda_stream


def _check(status):
    if status != 0:
        msg = lib().cobs_status_string(status).decode()
        raise CobsError(msg)


_TORCH_DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16}


def _need(name, t, dtype, numel):
    """Reject a tensor the kernels would misread: wrong dtype, not contiguous,
    or fewer elements than the call reads or writes.  Returns it."""
    if t is None:
        raise CobsError(f"{name} is required")
    if t.dtype != dtype:
        raise CobsError(f"{name} must be {dtype}, got {t.dtype}")
    if not t.is_contiguous():
        raise CobsError(f"{name} must be contiguous")
    if t.numel() < numel:
        raise CobsError(f"{name} holds {t.numel()} elements, the call needs {numel}")
    return t


def _opt(name, t, dtype, numel):
    return None if t is None else _need(name, t, dtype, numel)


def _same_gpu(**tensors):
    """Every given tensor on one GPU (checked after the shapes and types)."""
    dev = None
    for name, t in tensors.items():
        if t is None:
            continue
        if not t.is_cuda:
            raise CobsError(f"{name} must be on a GPU")
        if dev is None:
            dev = t.device
        elif t.device != dev:
            raise CobsError(f"{name} is on {t.device}, the call runs on {dev}")


# Every entry point looks its arguments over in one pass (_fits, _kv_fits); only
# when something does not fit does it run the checks one by one (_need, _kv,
# _same_gpu), which name the fault, or find that there is none.  A small decode
# step is bound by the calling thread, and the separate checks were most of it.

def _gpu(t):
    """Index of the tensor's GPU; -1 for anything else, which the separate checks name."""
    return t.get_device() if isinstance(t, torch.Tensor) else -1


def _fits(dev, *checks):
    """Every (tensor or None, dtype, elements) contiguous on GPU `dev`, and large enough."""
    for t, dtype, n in checks:
        if t is not None and not (t.dtype is dtype and t.numel() >= n and t.get_device() == dev and t.is_contiguous()):
            return False
    return dev >= 0


def _kv_fits(cfg, dtype, dev, k, v):
    """The C view of a contiguous-mode cache on GPU `dev`, or None if anything does not fit."""
    if k.dtype is not dtype or v.dtype is not dtype:
        return None
    shape, stride = k.shape, k.stride()
    if len(shape) != 4 or v.shape != shape or v.stride() != stride or k.get_device() != dev or v.get_device() != dev:
        return None
    if (shape[3] != cfg.head_dim or stride[3] != 1 or shape[0] < cfg.batch or shape[1] < cfg.num_kv_heads or
            shape[2] < cfg.max_seq_len):
        return None
    return _KV(k.data_ptr(), v.data_ptr(), stride[0], stride[1], stride[2], None, 0)


def _kv(cfg, k, v, block_table=None, num_pages=0):
    """Validated K/V view (contiguous [>=B, >=Hkv, >=T_max, d] with the head
    dimension dense, or pages [num_pages, Hkv, L, d] with a [B, T_max/L] table)."""
    want = _TORCH_DTYPE[cfg.kv_dtype]
    for name, t in (("k", k), ("v", v)):
        if t is None or t.dtype != want:
            raise CobsError(f"{name} must be {want} (kv_dtype {cfg.kv_dtype})")
        if t.dim() != 4 or t.shape[-1] != cfg.head_dim or t.stride(-1) != 1:
            raise CobsError(f"{name} must be 4-D with a dense head dimension of {cfg.head_dim}")
    if block_table is not None:
        for name, t in (("k", k), ("v", v)):
            if tuple(t.shape[1:]) != (cfg.num_kv_heads, cfg.block_size, cfg.head_dim) or not t.is_contiguous():
                raise CobsError(f"paged {name} must be a contiguous [pages, Hkv, L, d] pool")
            if not 1 <= int(num_pages) <= t.shape[0]:
                raise CobsError(f"num_pages must lie in [1, {t.shape[0]}]")
        _need("block_table", block_table, torch.int32, cfg.batch * cfg.num_blocks)
        return _KV(k.data_ptr(), v.data_ptr(), 0, 0, 0, block_table.data_ptr(), int(num_pages))
    if k.stride() != v.stride() or k.shape != v.shape:
        raise CobsError("K and V must share shape and strides")
    if k.shape[0] < cfg.batch or k.shape[1] < cfg.num_kv_heads or k.shape[2] < cfg.max_seq_len:
        raise CobsError(f"K/V of shape {tuple(k.shape)} is smaller than "
                        f"[{cfg.batch}, {cfg.num_kv_heads}, {cfg.max_seq_len}, {cfg.head_dim}]")
    return _KV(k.data_ptr(), v.data_ptr(), k.stride(0), k.stride(1), k.stride(2), None, 0)


def _units(cfg):
    return cfg.batch * cfg.num_kv_heads


def _ws(ws):
    """Workspace tensor (any element type, contiguous) and its size in bytes."""
    if ws is None:
        raise CobsError("ws is required")
    if not ws.is_contiguous():
        raise CobsError("ws must be contiguous")
    return ws.numel() * ws.element_size()


def _summaries(cfg, summaries, rec_bytes):
    return _need("summaries", summaries, torch.uint8, _units(cfg) * cfg.num_blocks * rec_bytes)


def record_bytes(cfg):
    return int(lib().cobs_record_bytes(ctypes.byref(cfg.c_struct())))


def workspace_bytes(cfg, op):
    return int(lib().cobs_workspace_bytes(ctypes.byref(cfg.c_struct()), int(op)))


def new_workspace(cfg, op, device):
    """Zero-filled workspace for `op` (the library requires zeros before first use)."""
    n = workspace_bytes(cfg, op)
    return torch.zeros(max(n, 256), dtype=torch.uint8, device=device)


def new_summaries(cfg, device):
    return torch.zeros((cfg.batch, cfg.num_kv_heads, cfg.num_blocks, record_bytes(cfg)),
                       dtype=torch.uint8, device=device)


def cobs_build_block_stats(cfg, k, v, seq_lens, summaries, first_block=0, num_blocks=None,
                           ws=None, block_table=None, num_pages=0, stream=None):
    if num_blocks is None:
        num_blocks = cfg.num_blocks - first_block
    c, rb, kvt = cfg.marshalled()
    kv = None
    if (seq_lens is not None and summaries is not None and k is not None and v is not None and
            block_table is None and cfg.query_basis is None):
        dev = _gpu(summaries)
        if _fits(dev, (seq_lens, torch.int32, cfg.batch), (summaries, torch.uint8, _units(cfg) * cfg.num_blocks * rb)):
            kv = _kv_fits(cfg, kvt, dev, k, v)
    if kv is None:
        _need("seq_lens", seq_lens, torch.int32, cfg.batch)
        _summaries(cfg, summaries, rb)
        kv = _kv(cfg, k, v, block_table, num_pages)
        _same_gpu(seq_lens=seq_lens, summaries=summaries, k=k, v=v, block_table=block_table,
                  query_basis=cfg.query_basis)
    _check(lib().cobs_build_block_stats(ctypes.byref(c), ctypes.byref(kv),
                                        _ptr(seq_lens), int(first_block), int(num_blocks),
                                        _ptr(summaries), _ptr(ws),
                                        0 if ws is None else ws.numel() * ws.element_size(),
                                        _stream(stream, summaries)))


def _select_io(cfg, q, seq_lens, sel, scores):
    _need("q", q, torch.float32, cfg.batch * cfg.num_q_heads * cfg.head_dim)
    _need("seq_lens", seq_lens, torch.int32, cfg.batch)
    _need("sel", sel, torch.int32, _units(cfg) * cfg.budget)
    _opt("scores", scores, torch.float32, _units(cfg) * cfg.num_blocks)


def cobs_select(cfg, q, summaries, seq_lens, sel, ws, scores=None, stream=None):
    _select_io(cfg, q, seq_lens, sel, scores)
    c, rb, _ = cfg.marshalled()
    _summaries(cfg, summaries, rb)
    nws = _ws(ws)
    _same_gpu(q=q, summaries=summaries, seq_lens=seq_lens, sel=sel, scores=scores, ws=ws,
              query_basis=cfg.query_basis)
    _check(lib().cobs_select(ctypes.byref(c), _ptr(q), _ptr(summaries),
                             _ptr(seq_lens), _ptr(sel), _ptr(scores), _ptr(ws), nws, _stream(stream, q)))


def _dense_key_select(fn, cfg, q, k, v, seq_lens, sel, ws, scores, block_table, num_pages, stream):
    _select_io(cfg, q, seq_lens, sel, scores)
    kv = _kv(cfg, k, v, block_table, num_pages)
    nws = _ws(ws)
    _same_gpu(q=q, k=k, v=v, seq_lens=seq_lens, sel=sel, scores=scores, ws=ws, block_table=block_table)
    _check(fn(ctypes.byref(cfg.c_struct()), _ptr(q), ctypes.byref(kv), _ptr(seq_lens), _ptr(sel), _ptr(scores),
              _ptr(ws), nws, _stream(stream, q)))


def cobs_select_exact(cfg, q, k, v, seq_lens, sel, ws, scores=None, block_table=None, num_pages=0,
                      stream=None):
    _dense_key_select(lib().cobs_select_exact, cfg, q, k, v, seq_lens, sel, ws, scores, block_table, num_pages,
                      stream)


def cobs_select_quest(cfg, q, k, v, seq_lens, sel, ws, scores=None, block_table=None, num_pages=0,
                      stream=None):
    _dense_key_select(lib().cobs_select_quest, cfg, q, k, v, seq_lens, sel, ws, scores, block_table, num_pages,
                      stream)


def _decode_io(cfg, q, seq_lens, sel, outs, lses, sel_required=True):
    _need("q", q, torch.float32, cfg.batch * cfg.num_q_heads * cfg.head_dim)
    _need("seq_lens", seq_lens, torch.int32, cfg.batch)
    if (sel_required and cfg.budget > 0) or sel is not None:
        _need("sel", sel, torch.int32, _units(cfg) * cfg.budget)
    for name, o in outs.items():
        _need(name, o, torch.float32, cfg.batch * cfg.num_q_heads * cfg.head_dim)
    for name, l in lses.items():
        _opt(name, l, torch.float32, cfg.batch * cfg.num_q_heads)


def cobs_sparse_decode(cfg, q, k, v, seq_lens, sel, out, ws, lse=None, block_table=None,
                       num_pages=0, stream=None):
    _decode_io(cfg, q, seq_lens, sel, dict(out=out), dict(lse=lse))
    kv = _kv(cfg, k, v, block_table, num_pages)
    nws = _ws(ws)
    _same_gpu(q=q, k=k, v=v, seq_lens=seq_lens, sel=sel, out=out, lse=lse, ws=ws, block_table=block_table)
    _check(lib().cobs_sparse_decode(ctypes.byref(cfg.c_struct()), _ptr(q), ctypes.byref(kv),
                                    _ptr(seq_lens), _ptr(sel), _ptr(out), _ptr(lse), _ptr(ws), nws,
                                    _stream(stream, q)))


def _attend_fits(cfg, rec_bytes, kv_dtype, q, k, v, seq_lens, sel, outs, lses, ws, block_table, summaries=None):
    """The C view of the cache if every argument of an attention call fits, else None."""
    if (q is None or seq_lens is None or ws is None or k is None or v is None or block_table is not None or
            cfg.query_basis is not None or any(o is None for o in outs)):
        return None
    dev, nq = _gpu(q), cfg.batch * cfg.num_q_heads
    if not _fits(dev, (q, torch.float32, nq * cfg.head_dim), (seq_lens, torch.int32, cfg.batch),
                 (sel, torch.int32, _units(cfg) * cfg.budget), (ws, ws.dtype, 0),
                 (summaries, torch.uint8, _units(cfg) * cfg.num_blocks * rec_bytes),
                 *((o, torch.float32, nq * cfg.head_dim) for o in outs), *((l, torch.float32, nq) for l in lses)):
        return None
    return _kv_fits(cfg, kv_dtype, dev, k, v)


def cobs_sparse_decode_branches(cfg, q, k, v, seq_lens, sel, out_sel, out_win, ws, lse_sel=None, lse_win=None,
                                block_table=None, num_pages=0, stream=None):
    c, rb, kvt = cfg.marshalled()
    kv = None
    if sel is not None:
        kv = _attend_fits(cfg, rb, kvt, q, k, v, seq_lens, sel, (out_sel, out_win), (lse_sel, lse_win), ws,
                          block_table)
    if kv is None:
        _decode_io(cfg, q, seq_lens, sel, dict(out_sel=out_sel, out_win=out_win),
                   dict(lse_sel=lse_sel, lse_win=lse_win))
        kv = _kv(cfg, k, v, block_table, num_pages)
        _ws(ws)
        _same_gpu(q=q, k=k, v=v, seq_lens=seq_lens, sel=sel, out_sel=out_sel, out_win=out_win, lse_sel=lse_sel,
                  lse_win=lse_win, ws=ws, block_table=block_table)
    _check(lib().cobs_sparse_decode_branches(ctypes.byref(c), _ptr(q), ctypes.byref(kv),
                                             _ptr(seq_lens), _ptr(sel), _ptr(out_sel), _ptr(lse_sel),
                                             _ptr(out_win), _ptr(lse_win), _ptr(ws),
                                             ws.numel() * ws.element_size(), _stream(stream, q)))


def cobs_decode_step(cfg, q, k, v, seq_lens, summaries, out, ws, sel=None, lse=None,
                     block_table=None, num_pages=0, stream=None):
    c, rb, kvt = cfg.marshalled()
    kv = None
    if summaries is not None:
        kv = _attend_fits(cfg, rb, kvt, q, k, v, seq_lens, sel, (out,), (lse,), ws, block_table, summaries)
    if kv is None:
        _decode_io(cfg, q, seq_lens, sel, dict(out=out), dict(lse=lse), sel_required=False)
        _summaries(cfg, summaries, rb)
        kv = _kv(cfg, k, v, block_table, num_pages)
        _ws(ws)
        _same_gpu(q=q, k=k, v=v, seq_lens=seq_lens, summaries=summaries, sel=sel, out=out, lse=lse, ws=ws,
                  block_table=block_table, query_basis=cfg.query_basis)
    _check(lib().cobs_decode_step(ctypes.byref(c), _ptr(q), ctypes.byref(kv),
                                  _ptr(seq_lens), _ptr(summaries), _ptr(sel), _ptr(out), _ptr(lse),
                                  _ptr(ws), ws.numel() * ws.element_size(), _stream(stream, q)))


def cobs_decode_step_noalloc(cfg, q, k, v, seq_lens, summaries, out, sel=None, lse=None,
                             block_table=None, num_pages=0, stream=None):
    """cobs_decode_step on the library's own per-GPU workspace (no ws argument)."""
    _decode_io(cfg, q, seq_lens, sel, dict(out=out), dict(lse=lse), sel_required=False)
    c, rb, _ = cfg.marshalled()
    _summaries(cfg, summaries, rb)
    kv = _kv(cfg, k, v, block_table, num_pages)
    _same_gpu(q=q, k=k, v=v, seq_lens=seq_lens, summaries=summaries, sel=sel, out=out, lse=lse,
              block_table=block_table, query_basis=cfg.query_basis)
    _check(lib().cobs_decode_step_noalloc(ctypes.byref(c), _ptr(q), ctypes.byref(kv),
                                          _ptr(seq_lens), _ptr(summaries), _ptr(sel), _ptr(out), _ptr(lse),
                                          _stream(stream, q)))


def cobs_compression_branch(cfg, q, summaries, seq_lens, out, lse=None, stream=None):
    """The mean-pool compression branch over value-mean records (cfg.value_mean)."""
    c, rb, _ = cfg.marshalled()
    nq = cfg.batch * cfg.num_q_heads
    if (q is None or summaries is None or seq_lens is None or out is None or
            not _fits(_gpu(q), (q, torch.float32, nq * cfg.head_dim), (seq_lens, torch.int32, cfg.batch),
                      (summaries, torch.uint8, _units(cfg) * cfg.num_blocks * rb),
                      (out, torch.float32, nq * cfg.head_dim), (lse, torch.float32, nq))):
        _need("q", q, torch.float32, nq * cfg.head_dim)
        _need("seq_lens", seq_lens, torch.int32, cfg.batch)
        _summaries(cfg, summaries, rb)
        _need("out", out, torch.float32, nq * cfg.head_dim)
        _opt("lse", lse, torch.float32, nq)
        _same_gpu(q=q, summaries=summaries, seq_lens=seq_lens, out=out, lse=lse)
    _check(lib().cobs_compression_branch(ctypes.byref(c), _ptr(q), _ptr(summaries), _ptr(seq_lens),
                                         _ptr(out), _ptr(lse), _stream(stream, q)))


def cobs_pack_e2m1(x, codes, scales, stream=None):
    if x is None or x.dim() != 2:
        raise CobsError("x must be a 2-D [num_vectors, dim] tensor")
    n, dim = x.shape
    _need("x", x, torch.float32, n * dim)
    _need("codes", codes, torch.uint8, n * (dim // 2))
    _need("scales", scales, torch.float32, n)
    _same_gpu(x=x, codes=codes, scales=scales)
    _check(lib().cobs_pack_e2m1(_ptr(x), int(n), int(dim), _ptr(codes), _ptr(scales),
                                _stream(stream, x)))
