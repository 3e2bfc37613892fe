"""Python binding for libcure. Argument marshalling only.

Each function has the name of the C entry point it calls and runs on the
current torch stream of the tensors' device. PyTorch provides the device memory
(outputs and workspaces are allocated as torch tensors) and the stream; every
step of the computation runs in libcure's HIP kernels. The calls of a decoding
loop are marshalled by the extension module _native (csrc/binding.cpp), which
also keeps the zero-filled device workspaces, one per call kind, device and
stream; lib() is the C ABI itself, through ctypes. If the library is not built,
the first call raises -- there is no fallback implementation.
"""

import ctypes
import importlib.util
import os
import threading

import numpy as np
import torch


CURE_OK = 0
CURE_ERR_INVALID_ARG = 1
CURE_ERR_UNSUPPORTED = 2
CURE_ERR_BAD_TREE = 3
CURE_ERR_HIP = 4
CURE_ERR_WORKSPACE = 5
CURE_F32 = 0
CURE_BF16 = 1
CURE_ATTN_FORCE_VALU = 1
CURE_MAX_TREE_NODES = 256

_lock = threading.Lock()
_lib = None
_ext = None

_vp, _i32, _i64, _f32, _sz, _u32 = (ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64,
                                    ctypes.c_float, ctypes.c_size_t, ctypes.c_uint32)

_SIGNATURES = {
    "cure_status_string": (ctypes.c_char_p, [ctypes.c_int]),
    "cure_version": (ctypes.c_int, []),
    "cure_margins_workspace_size": (_sz, [_i32, _i32, _i32]),
    "cure_margins": (ctypes.c_int, [_vp, _i32, _i32, _i32, _i32, _i64,
                                    _vp, _vp, _vp, _vp, _vp, _vp,
                                    _i32, _f32, _i32, _i32, _vp, _vp, _vp, _sz, _vp]),
    "cure_margins_accept": (ctypes.c_int, [_vp, _i32, _i32, _i32, _i32, _i64,
                                           _vp, _vp, _vp, _vp, _vp, _vp,
                                           _i32, _f32, _i32, _i32, _vp, _vp,
                                           _vp, _vp, _vp, _vp, _vp, _vp, _vp, _vp, _vp,
                                           _vp, _sz, _vp]),
    "cure_margins_noalloc_scratch_bytes": (_sz, []),
    "cure_margins_noalloc": (ctypes.c_int, [_vp, _i32, _i32, _i32, _i32, _i64,
                                            _vp, _vp, _vp, _vp, _vp, _vp,
                                            _i32, _f32, _i32, _i32, _vp, _vp, _vp]),
    "cure_tree_attn_workspace_size": (_sz, [_i32, _i32, _i32, _i32, _i32, _vp, _vp, _i32]),
    "cure_tree_attn": (ctypes.c_int, [_vp, _vp, _vp, _vp, _vp, _i32, _i32, _i32, _i32, _i32,
                                      _i32, _f32, _vp, _vp, _vp, _vp, _i32, _vp, _vp, _i32,
                                      _u32, _vp, _vp, _sz, _vp]),
    "cure_accept": (ctypes.c_int, [_vp, _vp, _vp, _vp, _vp, _i32, _i32, _i32,
                                   _vp, _vp, _vp, _vp, _vp, _vp]),
    "cure_repair_tree_workspace_size": (_sz, [_i32, _i32, _i32, _i32, _i32]),
    "cure_repair_tree": (ctypes.c_int, [_vp, _i32, _i32, _i32, _i32, _i64, _vp, _vp, _vp, _vp,
                                        _i32, _i32, _i32, _f32, _i32, _i32, _vp, _i32,
                                        _vp, _vp, _vp, _vp, _vp, _sz, _vp]),
    "cure_read_ceiling_chunks": (_sz, [_sz]),
    "cure_read_ceiling": (ctypes.c_int, [_vp, _sz, _vp, _vp]),
    "cure_commit": (ctypes.c_int, [_vp, _vp, _i32, _i32, _i64, _i32, _i32, _i32,
                                   _vp, _vp, _vp, _vp, _vp, _vp, _vp, _i32, _i32,
                                   _vp, _vp, _vp, _vp, _vp, _vp]),
}


class CureError(RuntimeError):
    pass


def library_path():
    return os.path.join(os.path.dirname(os.path.abspath(__file__)), "_lib", "libcure.so")


def lib():
    """The loaded libcure (ctypes.CDLL). Raises if the library has not been built."""
    global _lib
    with _lock:
        if _lib is None:
            path = library_path()
            if not os.path.exists(path):
                raise CureError("libcure is not built (%s missing); run "
                                "`python -m paper_2608_00531_amd.build`" % path)
            l = ctypes.CDLL(path)
            for name, (res, args) in _SIGNATURES.items():
                fn = getattr(l, name)
                fn.restype = res
                fn.argtypes = args
            _lib = l
        return _lib


def _native():
    """The extension module. Raises if it has not been built."""
    global _ext
    if _ext is None:
        lib()
        with _lock:
            if _ext is None:
                path = os.path.join(os.path.dirname(library_path()), "_native.so")
                if not os.path.exists(path):
                    raise CureError("the binding is not built (%s missing); run "
                                    "`python -m paper_2608_00531_amd.build`" % path)
                spec = importlib.util.spec_from_file_location("_native", path)
                ext = importlib.util.module_from_spec(spec)
                spec.loader.exec_module(ext)
                ext.setup(CureError, lambda a: _host_i32(a)[0])
                _ext = ext
    return _ext


def _check(status, what):
    if status != CURE_OK:
        name = lib().cure_status_string(status).decode()
        raise CureError("%s failed: %s" % (what, name))


def _ptr(t):
    return None if t is None else ctypes.c_void_p(t.data_ptr())


def _stream(device):
    return ctypes.c_void_p(torch.cuda.current_stream(device).cuda_stream)


def _require_cuda(*ts):
    for t in ts:
        if t is not None and not t.is_cuda:
            raise CureError("tensor arguments must live on the GPU")


def cure_margins(logits, chain_len=0, tau=float("inf"), repair_budget=0, branch_depth=1,
                 gate=True):
    """Margin pass over logits [batch, rows, vocab] (or [rows, vocab]).

    Returns a dict of tensors shaped [batch, rows]: top1_val, top1_idx, top2_val,
    top2_idx, lse, margin; with gate=True also ufp_pos [batch, chain_len] and
    ufp_cnt [batch].
    """
    return _native().margins(logits, chain_len, tau, repair_budget, branch_depth, gate, False)


def cure_margins_accept(logits, parent, token, root_tgt, n_nodes, chain_len, tau=float("inf"),
                        repair_budget=0, branch_depth=1, gate=True):
    """Margin pass over a tree's node logits [batch, n_max, vocab] followed by
    the acceptance walk on their argmaxes, in one call. parent/token int32
    [batch, n_max], root_tgt/n_nodes int32 [batch] (GPU tensors). Returns
    cure_margins' dict plus cure_accept's (acc_len, path, best, bonus, resync)."""
    return _native().margins(logits, chain_len, tau, repair_budget, branch_depth, gate, False,
                             parent, token, root_tgt, n_nodes)


def cure_margins_noalloc(logits, chain_len=0, tau=float("inf"), repair_budget=0,
                         branch_depth=1, gate=True):
    """As cure_margins, through the allocation-free entry point: no workspace
    is passed; the library's fixed scratch array serves the call."""
    return _native().margins(logits, chain_len, tau, repair_budget, branch_depth, gate, True)


def _host_i32(a):
    a = np.ascontiguousarray(np.asarray(a, dtype=np.int32))
    return a, a.ctypes.data_as(ctypes.c_void_p)


def cure_tree_attn_workspace_size(batch, hq, hkv, d, n_max, host_ctx_len, host_n_nodes,
                                  kv_split=0):
    c, cp = _host_i32(host_ctx_len)
    n, np_ = _host_i32(host_n_nodes)
    return lib().cure_tree_attn_workspace_size(batch, hq, hkv, d, n_max, cp, np_, kv_split)


def cure_tree_attn(q, k, v, kv_off, ctx_len, n_nodes, parent, host_ctx_len, host_n_nodes,
                   scale, out_dtype=None, kv_split=0, flags=0, with_lse=True):
    """Tree-masked verification attention.

    q [batch, n_max, hq, d]; k, v [rows, hkv, d]; kv_off int64 [batch]; ctx_len,
    n_nodes int32 [batch]; parent int32 [batch, n_max] (all on the GPU);
    host_ctx_len / host_n_nodes: host copies (numpy or lists).
    Returns (o [batch, n_max, hq, d], lse [batch, n_max, hq] or None, tree_status [batch]).
    """
    return _native().tree_attn(q, k, v, kv_off, ctx_len, n_nodes, parent, host_ctx_len, host_n_nodes,
                               scale, out_dtype, kv_split, flags, with_lse)


def cure_accept(parent, token, tgt, root_tgt, n_nodes, chain_len):
    """Acceptance walk. All arguments int32 GPU tensors: parent/token/tgt
    [batch, n_max], root_tgt/n_nodes [batch]. Returns a dict of tensors."""
    return _native().accept(parent, token, tgt, root_tgt, n_nodes, chain_len)


def cure_repair_tree(logits, margin, ufp_pos, ufp_cnt, chain_tok, repair_budget, branch_depth,
                     margin_scale, b_min=1, b_max=5, suffix=None, n_max=None):
    """Repair tree per sequence.

    logits [batch, rows, vocab] (or [rows, vocab]) -- the draft block's rows;
    margin [batch, rows] float32, ufp_pos [batch, chain_len], ufp_cnt [batch] as
    cure_margins returned them; chain_tok int32 [batch, chain_len]; suffix int32
    [batch, chain_len, b_max, branch_depth - 1] or None.
    Returns a dict: parent, token [batch, n_max] (valid below n_nodes), n_nodes
    [batch], branch_cnt [batch, chain_len].
    """
    return _native().repair_tree(logits, margin, ufp_pos, ufp_cnt, chain_tok, repair_budget,
                                 branch_depth, margin_scale, b_min, b_max, suffix, n_max)


def cure_commit(k, v, kv_off, ctx_len, n_nodes, path, acc_len, token, bonus, chain_len,
                layer_stride=None):
    """Commit each sequence's winning path, in place.

    k, v: one layer's cache [rows, hkv, d], or n_layers caches [n_layers, rows,
    hkv, d] (contiguous per layer; layer_stride in elements defaults to the
    distance between layers). kv_off int64 [batch]; ctx_len, n_nodes, acc_len,
    bonus int32 [batch]; path, token int32 [batch, n_max] (all on the GPU; path,
    acc_len and bonus as cure_accept returned them).
    Returns a dict: new_ctx_len [batch], emit [batch, n_max + 1], emit_cnt,
    replay_start and status [batch].
    """
    return _native().commit(k, v, kv_off, ctx_len, n_nodes, path, acc_len, token, bonus, chain_len,
                            layer_stride)


def cure_read_ceiling(buf):
    """Streams a contiguous GPU tensor (size a multiple of 16 bytes) once; returns
    the per-256-KB-chunk XOR of its 32-bit words (int32 tensor)."""
    _require_cuda(buf)
    if not buf.is_contiguous():
        raise CureError("the buffer must be contiguous")
    nbytes = buf.numel() * buf.element_size()
    L = lib()
    out = torch.empty(max(int(L.cure_read_ceiling_chunks(nbytes)), 1), dtype=torch.int32,
                      device=buf.device)
    _check(L.cure_read_ceiling(_ptr(buf), nbytes, _ptr(out), _stream(buf.device)),
           "cure_read_ceiling")
    return out
