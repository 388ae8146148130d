"""ctypes binding of libbpt.so (the C ABI declared in include/bpt.h).

Argument marshalling only: every step of the path runs in the library's HIP
kernels.  torch supplies device memory and the stream, nothing else.  There is
no CPU fallback: a missing library is an error.
"""
from __future__ import annotations

import ctypes
import os
from typing import Optional, Tuple

import numpy as np
import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libbpt.so")

BPT_F32, BPT_BF16 = 0, 1
BPT_OK, BPT_ERR_INVALID_ARG, BPT_ERR_UNSUPPORTED, BPT_ERR_ALLOC, BPT_ERR_LAUNCH, BPT_ERR_OVERFLOW, BPT_ERR_SCRATCH = range(7)
BPT_STATIC_SCRATCH_BYTES = 32 << 20

EXPORTS = [
    "bpt_build_graph", "bpt_build_batch_graph", "bpt_build_batch_graph_on", "bpt_graph_layout", "bpt_graph_info", "bpt_graph_csr", "bpt_graph_transposed", "bpt_graph_to_host",
    "bpt_graph_transposed_to_host", "bpt_graph_destroy", "bpt_attn_fwd_workspace", "bpt_attn_bwd_workspace",
    "bpt_attn_fwd", "bpt_attn_fwd_static", "bpt_attn_bwd", "bpt_attn_bwd_query_side", "bpt_attn_bwd_key_side", "bpt_profile_enable",
    "bpt_profile_report", "bpt_calibrate_gather", "bpt_layer_fwd_workspace", "bpt_layer_fwd", "bpt_layer_bwd_workspace", "bpt_layer_bwd",
    "bpt_stack_fwd_workspace", "bpt_stack_fwd", "bpt_stack_bwd_workspace", "bpt_stack_bwd",
    "bpt_count_edges", "bpt_strerror",
]


class BptShape(ctypes.Structure):
    _fields_ = [("B", ctypes.c_int32), ("H", ctypes.c_int32), ("D", ctypes.c_int32), ("dtype", ctypes.c_int32),
                ("stride_b", ctypes.c_int64), ("stride_h", ctypes.c_int64), ("stride_n", ctypes.c_int64),
                ("scale", ctypes.c_float), ("seq_len", ctypes.c_void_p), ("dropout_p", ctypes.c_float),
                ("dropout_seed", ctypes.c_uint32), ("leave_unkept", ctypes.c_int32), ("grad_dtype", ctypes.c_int32)]


class BptLayerParams(ctypes.Structure):
    _fields_ = [(name, ctypes.c_void_p) for name in ("Wq", "Wk", "Wv", "Wo", "W1", "W2", "b1", "b2", "g1", "beta1", "g2",
                                                     "beta2")] + [("d_ff", ctypes.c_int32), ("eps", ctypes.c_float)]


GRAD_NAMES = ("dWq", "dWk", "dWv", "dWo", "dW1", "db1", "dW2", "db2", "dg1", "dbeta1", "dg2", "dbeta2")


class BptLayerGrads(ctypes.Structure):
    _fields_ = [(name, ctypes.c_void_p) for name in GRAD_NAMES]


class BptError(RuntimeError):
    def __init__(self, status: int, what: str):
        self.status = status
        super().__init__("%s: %s (status %d)" % (what, strerror(status), status))


_lib = None


def load_library() -> ctypes.CDLL:
    """Loads the in-tree libbpt.so; building it is __graft_entry__.build()'s job."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(LIB_PATH):
        raise FileNotFoundError(
            "%s is missing: build it with `python -m paper_1911_04070_amd.build` "
            "(there is no CPU fallback)" % LIB_PATH)
    L = ctypes.CDLL(LIB_PATH)
    i32, i64, vp, sz = ctypes.c_int32, ctypes.c_int64, ctypes.c_void_p, ctypes.c_size_t
    P = ctypes.POINTER
    L.bpt_build_graph.restype = ctypes.c_int
    L.bpt_build_graph.argtypes = [i32, i32, i32, vp, P(vp)]
    L.bpt_build_batch_graph.restype = ctypes.c_int
    L.bpt_build_batch_graph.argtypes = [i32, i32, i32, vp, i32, vp, P(vp)]
    L.bpt_build_batch_graph_on.restype = ctypes.c_int
    L.bpt_build_batch_graph_on.argtypes = [vp, vp, i32, i32, vp, P(vp)]
    L.bpt_graph_layout.restype = ctypes.c_int
    L.bpt_graph_layout.argtypes = [vp, P(i32), P(i32), vp, vp]
    L.bpt_graph_info.restype = ctypes.c_int
    L.bpt_graph_info.argtypes = [vp, P(i32), P(i32), P(i32), P(i32), P(i64), P(i32), P(i32), P(i32)]
    L.bpt_graph_csr.restype = ctypes.c_int
    L.bpt_graph_csr.argtypes = [vp, P(vp), P(vp), P(vp)]
    L.bpt_graph_transposed.restype = ctypes.c_int
    L.bpt_graph_transposed.argtypes = [vp, P(vp), P(vp), P(vp)]
    L.bpt_graph_to_host.restype = ctypes.c_int
    L.bpt_graph_to_host.argtypes = [vp, vp, vp, vp]
    L.bpt_graph_transposed_to_host.restype = ctypes.c_int
    L.bpt_graph_transposed_to_host.argtypes = [vp, vp, vp, vp]
    L.bpt_graph_destroy.restype = None
    L.bpt_graph_destroy.argtypes = [vp]
    L.bpt_attn_fwd_workspace.restype = sz
    L.bpt_attn_fwd_workspace.argtypes = [vp, P(BptShape)]
    L.bpt_attn_bwd_workspace.restype = sz
    L.bpt_attn_bwd_workspace.argtypes = [vp, P(BptShape)]
    L.bpt_attn_fwd.restype = ctypes.c_int
    L.bpt_attn_fwd.argtypes = [vp, P(BptShape), vp, vp, vp, vp, vp, vp, vp, sz, vp]
    L.bpt_attn_fwd_static.restype = ctypes.c_int
    L.bpt_attn_fwd_static.argtypes = [vp, P(BptShape), vp, vp, vp, vp, vp, vp, vp]
    L.bpt_attn_bwd.restype = ctypes.c_int
    L.bpt_attn_bwd.argtypes = [vp, P(BptShape)] + [vp] * 11 + [sz, vp]
    L.bpt_attn_bwd_query_side.restype = ctypes.c_int
    L.bpt_attn_bwd_query_side.argtypes = [vp, P(BptShape)] + [vp] * 9 + [sz, vp]
    L.bpt_attn_bwd_key_side.restype = ctypes.c_int
    L.bpt_attn_bwd_key_side.argtypes = [vp, P(BptShape)] + [vp] * 9 + [sz, vp]
    L.bpt_profile_enable.restype = ctypes.c_int
    L.bpt_profile_enable.argtypes = [ctypes.c_int]
    L.bpt_profile_report.restype = ctypes.c_int64
    L.bpt_profile_report.argtypes = [ctypes.c_char_p, sz]
    L.bpt_calibrate_gather.restype = ctypes.c_int
    L.bpt_calibrate_gather.argtypes = [vp, vp, vp, i64, vp]
    L.bpt_layer_fwd_workspace.restype = sz
    L.bpt_layer_fwd_workspace.argtypes = [vp, i32, i32, i32]
    L.bpt_layer_fwd.restype = ctypes.c_int
    L.bpt_layer_fwd.argtypes = [vp, i32, i32, ctypes.c_float, vp, vp, vp, P(BptLayerParams), vp, vp, sz, vp]
    L.bpt_layer_bwd_workspace.restype = sz
    L.bpt_layer_bwd_workspace.argtypes = [vp, i32, i32, i32]
    L.bpt_layer_bwd.restype = ctypes.c_int
    L.bpt_layer_bwd.argtypes = [vp, i32, i32, ctypes.c_float, vp, vp, vp, P(BptLayerParams), vp, sz, vp, vp, vp,
                                P(BptLayerGrads), vp, sz, vp]
    L.bpt_stack_fwd_workspace.restype = sz
    L.bpt_stack_fwd_workspace.argtypes = [vp, i32, i32, i32, i32]
    L.bpt_stack_fwd.restype = ctypes.c_int
    L.bpt_stack_fwd.argtypes = [vp, i32, i32, i32, ctypes.c_float, vp, P(vp), vp, P(BptLayerParams), vp, vp, vp, sz, vp]
    L.bpt_stack_bwd_workspace.restype = sz
    L.bpt_stack_bwd_workspace.argtypes = [vp, i32, i32, i32]
    L.bpt_stack_bwd.restype = ctypes.c_int
    L.bpt_stack_bwd.argtypes = [vp, i32, i32, i32, ctypes.c_float, vp, P(vp), P(BptLayerParams), vp, sz, vp, vp, vp, P(vp),
                                P(BptLayerGrads), vp, sz, vp]
    L.bpt_count_edges.restype = ctypes.c_int
    L.bpt_count_edges.argtypes = [i32, i32, i32, i32, P(i64)]
    L.bpt_strerror.restype = ctypes.c_char_p
    L.bpt_strerror.argtypes = [ctypes.c_int]
    _lib = L
    return L


def strerror(status: int) -> str:
    return load_library().bpt_strerror(int(status)).decode()


def _check(status: int, what: str) -> None:
    if status != BPT_OK:
        raise BptError(status, what)


def _stream_ptr() -> int:
    return int(torch.cuda.current_stream().cuda_stream)


class Graph:
    """Device-resident binary-partition graph (bpt_build_graph; with `lengths`, bpt_build_batch_graph)."""

    def __init__(self, n: int, k: int, causal: bool, lengths=None, tree: "Optional[Graph]" = None, with_edges: bool = True):
        L = load_library()
        handle = ctypes.c_void_p()
        self.is_batch = lengths is not None
        self._tree = tree      # a shared tree has to outlive this graph
        if tree is not None:
            lens = np.ascontiguousarray(lengths, dtype=np.int32)
            if lens.ndim != 1:
                raise ValueError("lengths must be one-dimensional")
            _check(L.bpt_build_batch_graph_on(tree.handle, lens.ctypes.data, int(lens.size), int(bool(with_edges)), _stream_ptr(),
                                              ctypes.byref(handle)), "bpt_build_batch_graph_on(batch=%d)" % lens.size)
        elif lengths is None:
            _check(L.bpt_build_graph(int(n), int(k), int(bool(causal)), _stream_ptr(), ctypes.byref(handle)),
                   "bpt_build_graph(n=%d, k=%d, causal=%d)" % (n, k, causal))
        else:
            lens = np.ascontiguousarray(lengths, dtype=np.int32)
            if lens.ndim != 1:
                raise ValueError("lengths must be one-dimensional")
            _check(L.bpt_build_batch_graph(int(n), int(k), int(bool(causal)), lens.ctypes.data, int(lens.size), _stream_ptr(),
                                           ctypes.byref(handle)),
                   "bpt_build_batch_graph(n=%d, k=%d, causal=%d, batch=%d)" % (n, k, causal, lens.size))
        self._h = handle
        i32, i64 = ctypes.c_int32, ctypes.c_int64
        vals = [i32(), i32(), i32(), i32(), i64(), i32(), i32(), i32()]
        _check(L.bpt_graph_info(self._h, *[ctypes.byref(v) for v in vals]), "bpt_graph_info")
        (self.n, self.k, causal_i, self.num_nodes, self.num_edges, self.num_levels, self.rel_width,
         self.ctx_levels) = [int(v.value) for v in vals]
        self.causal = bool(causal_i)
        batch, n_tokens = i32(), i32()
        _check(L.bpt_graph_layout(self._h, ctypes.byref(batch), ctypes.byref(n_tokens), None, None), "bpt_graph_layout")
        self.batch, self.n_tokens = int(batch.value), int(n_tokens.value)
        self.first_row = np.empty((self.num_levels, self.batch), dtype=np.int32)
        self.row_count = np.empty((self.num_levels, self.batch), dtype=np.int32)
        _check(L.bpt_graph_layout(self._h, None, None, self.first_row.ctypes.data, self.row_count.ctypes.data),
               "bpt_graph_layout")

    @property
    def handle(self) -> ctypes.c_void_p:
        if self._h is None:
            raise RuntimeError("graph was destroyed")
        return self._h

    def destroy(self) -> None:
        if getattr(self, "_h", None) is not None:
            load_library().bpt_graph_destroy(self._h)
            self._h = None

    def __del__(self):
        try:
            self.destroy()
        except Exception:
            pass

    def csr_to_host(self) -> Tuple[np.ndarray, np.ndarray, np.ndarray]:
        row_ptr = np.empty(self.num_nodes + 1, dtype=np.int32)
        col = np.empty(self.num_edges, dtype=np.int32)
        rel = np.empty(self.num_edges, dtype=np.int32)
        _check(load_library().bpt_graph_to_host(self.handle, row_ptr.ctypes.data, col.ctypes.data, rel.ctypes.data),
               "bpt_graph_to_host")
        return row_ptr, col, rel

    def transposed_to_host(self) -> Tuple[np.ndarray, np.ndarray, np.ndarray]:
        t_ptr = np.empty(self.num_nodes + 1, dtype=np.int32)
        t_src = np.empty(self.num_edges, dtype=np.int32)
        t_eid = np.empty(self.num_edges, dtype=np.int32)
        _check(load_library().bpt_graph_transposed_to_host(self.handle, t_ptr.ctypes.data, t_src.ctypes.data,
                                                           t_eid.ctypes.data), "bpt_graph_transposed_to_host")
        return t_ptr, t_src, t_eid

    def device_pointers(self) -> dict:
        L = load_library()
        a, b, c = ctypes.c_void_p(), ctypes.c_void_p(), ctypes.c_void_p()
        _check(L.bpt_graph_csr(self.handle, ctypes.byref(a), ctypes.byref(b), ctypes.byref(c)), "bpt_graph_csr")
        d, e, f = ctypes.c_void_p(), ctypes.c_void_p(), ctypes.c_void_p()
        _check(L.bpt_graph_transposed(self.handle, ctypes.byref(d), ctypes.byref(e), ctypes.byref(f)),
               "bpt_graph_transposed")
        return {"row_ptr": a.value, "col": b.value, "rel": c.value, "t_ptr": d.value, "t_src": e.value,
                "t_eid": f.value}


def bpt_count_edges(n: int, k: int, causal: bool, length: int) -> int:
    """Edges of the graph over n tokens that a sequence of `length` tokens keeps (host arithmetic)."""
    out = ctypes.c_int64()
    _check(load_library().bpt_count_edges(n, k, int(bool(causal)), int(length), ctypes.byref(out)), "bpt_count_edges")
    return int(out.value)


def bpt_build_graph(n: int, k: int, causal: bool) -> Graph:
    return Graph(n, k, causal)


def bpt_build_batch_graph(n: int, k: int, causal: bool, lengths) -> Graph:
    """One graph for a batch of sequences of the given lengths, rows packed (see include/bpt.h)."""
    return Graph(n, k, causal, lengths)


def bpt_build_batch_graph_on(tree: Graph, lengths, with_edges: bool = False) -> Graph:
    """The same sharing an existing graph of (n, k, causal); without edge lists it is made by host arithmetic and a few
    small copies and serves the calls that run on the matrix-core kernels."""
    return Graph(tree.n, tree.k, tree.causal, lengths, tree=tree, with_edges=with_edges)


def _shape_of(g: Graph, x: torch.Tensor, scale: Optional[float], seq_len: Optional[torch.Tensor] = None,
              dropout: Optional[Tuple[float, int]] = None, leave_unkept: bool = False, bf16_grads: bool = False) -> BptShape:
    if x.dim() != 4 or x.shape[2] != g.num_nodes:
        raise ValueError("expected a [B,H,N=%d,D] tensor, got %s" % (g.num_nodes, tuple(x.shape)))
    if x.stride(3) != 1:
        raise ValueError("the feature dimension must be contiguous")
    if x.dtype == torch.float32:
        dt = BPT_F32
    elif x.dtype == torch.bfloat16:
        dt = BPT_BF16
    else:
        raise ValueError("dtype must be float32 or bfloat16")
    B, H, _, D = x.shape
    lens = None
    if seq_len is not None:
        if seq_len.dtype != torch.int32 or tuple(seq_len.shape) != (B,) or not seq_len.is_contiguous() or \
                seq_len.device != x.device:
            raise ValueError("seq_len must be a contiguous int32 tensor of B entries on the tensors' device")
        lens = seq_len.data_ptr()
    return BptShape(B, H, D, dt, x.stride(0), x.stride(1), x.stride(2), float(scale) if scale else 0.0, lens,
                    float(dropout[0]) if dropout else 0.0, (int(dropout[1]) & 0xFFFFFFFF) if dropout else 0,
                    1 if leave_unkept else 0, BPT_BF16 if bf16_grads else BPT_F32)


def _same_layout(ref: torch.Tensor, *others: torch.Tensor) -> None:
    for t in others:
        if t.shape != ref.shape or t.stride() != ref.stride() or t.device != ref.device:
            raise ValueError("tensors must share shape, strides and device")


SIZE_MAX = 2 ** 64 - 1   # a workspace query's answer for a graph / shape the calls refuse


def _need(nbytes: int, what: str) -> int:
    if nbytes == SIZE_MAX:
        raise BptError(BPT_ERR_UNSUPPORTED, what)
    return nbytes


def _workspace(nbytes: int, device) -> Tuple[Optional[torch.Tensor], int]:
    if nbytes == 0:
        return None, 0
    ws = torch.empty(nbytes, dtype=torch.uint8, device=device)
    return ws, ws.data_ptr()


def bpt_attn_fwd(g: Graph, Q: torch.Tensor, K: torch.Tensor, V: torch.Tensor, rel: torch.Tensor,
                 scale: Optional[float] = None, out: Optional[torch.Tensor] = None,
                 lse: Optional[torch.Tensor] = None, workspace: Optional[torch.Tensor] = None,
                 seq_len: Optional[torch.Tensor] = None, dropout: Optional[Tuple[float, int]] = None, leave_unkept: bool = False):
    """out, lse = graph attention of eq. (8).  Q,K,V: [B,H,N,D] cuda tensors; rel: [levels,W,D];
    seq_len: optional int32 [B] token counts of sequences shorter than n; dropout: (rate, seed) of the dropout on
    the attention weights."""
    L = load_library()
    shp = _shape_of(g, Q, scale, seq_len, dropout, leave_unkept)
    _same_layout(Q, K, V)
    if K.dtype != Q.dtype or V.dtype != Q.dtype or rel.dtype != Q.dtype:
        raise ValueError("Q, K, V and rel must share a dtype")
    if tuple(rel.shape) != (g.num_levels, g.rel_width, shp.D) or not rel.is_contiguous():
        raise ValueError("rel must be contiguous [%d,%d,%d]" % (g.num_levels, g.rel_width, shp.D))
    if out is None:
        out = torch.empty_strided(Q.shape, Q.stride(), dtype=Q.dtype, device=Q.device)
    if lse is None:
        lse = torch.empty(Q.shape[:3], dtype=torch.float32, device=Q.device)
    _same_layout(Q, out)
    need = _need(int(L.bpt_attn_fwd_workspace(g.handle, ctypes.byref(shp))), "bpt_attn_fwd_workspace")
    if workspace is None:
        workspace, ws_ptr = _workspace(need, Q.device)
    else:
        ws_ptr = workspace.data_ptr()
    ws_bytes = workspace.numel() * workspace.element_size() if workspace is not None else 0
    _check(L.bpt_attn_fwd(g.handle, ctypes.byref(shp), Q.data_ptr(), K.data_ptr(), V.data_ptr(), rel.data_ptr(),
                          out.data_ptr(), lse.data_ptr(), ws_ptr, ws_bytes, _stream_ptr()), "bpt_attn_fwd")
    return out, lse


def bpt_attn_fwd_static(g: Graph, Q: torch.Tensor, K: torch.Tensor, V: torch.Tensor, rel: torch.Tensor,
                        out: torch.Tensor, lse: torch.Tensor, scale: Optional[float] = None,
                        seq_len: Optional[torch.Tensor] = None, dropout: Optional[Tuple[float, int]] = None, leave_unkept: bool = False):
    """bpt_attn_fwd into caller-provided out and lse with the library's static scratch: this wrapper and the call
    allocate nothing."""
    L = load_library()
    shp = _shape_of(g, Q, scale, seq_len, dropout, leave_unkept)
    _same_layout(Q, K, V, out)
    if K.dtype != Q.dtype or V.dtype != Q.dtype or rel.dtype != Q.dtype or out.dtype != Q.dtype:
        raise ValueError("Q, K, V, rel and out must share a dtype")
    if tuple(rel.shape) != (g.num_levels, g.rel_width, shp.D) or not rel.is_contiguous():
        raise ValueError("rel must be contiguous [%d,%d,%d]" % (g.num_levels, g.rel_width, shp.D))
    if lse.dtype != torch.float32 or tuple(lse.shape) != tuple(Q.shape[:3]) or not lse.is_contiguous():
        raise ValueError("lse must be contiguous fp32 [B,H,N]")
    _check(L.bpt_attn_fwd_static(g.handle, ctypes.byref(shp), Q.data_ptr(), K.data_ptr(), V.data_ptr(), rel.data_ptr(),
                                 out.data_ptr(), lse.data_ptr(), _stream_ptr()), "bpt_attn_fwd_static")
    return out, lse


def _check_bwd_inputs(g, shp, Q, K, V, rel, lse, dout):
    """What the C side cannot see behind its raw pointers: dtypes, shapes and layouts of the backward's inputs."""
    _same_layout(Q, K, V, dout)
    if K.dtype != Q.dtype or V.dtype != Q.dtype or dout.dtype != Q.dtype or rel.dtype != Q.dtype:
        raise ValueError("Q, K, V, dout and rel must share a dtype")
    if tuple(rel.shape) != (g.num_levels, g.rel_width, shp.D) or not rel.is_contiguous() or rel.device != Q.device:
        raise ValueError("rel must be contiguous [%d,%d,%d] on the tensors' device" % (g.num_levels, g.rel_width, shp.D))
    if lse.dtype != torch.float32 or tuple(lse.shape) != tuple(Q.shape[:3]) or not lse.is_contiguous() or \
            lse.device != Q.device:
        raise ValueError("lse must be contiguous fp32 [B,H,N] on the tensors' device")


def _check_grad(Q, *grads) -> bool:
    """The gradients share Q's layout and are all fp32 or, for bf16 tensors, all bf16; returns whether they are bf16."""
    bf = grads[0].dtype == torch.bfloat16
    for t in grads:
        if t.dtype != (torch.bfloat16 if bf else torch.float32):
            raise ValueError("dQ, dK, dV must all be float32, or all bfloat16")
    if bf and Q.dtype != torch.bfloat16:
        raise ValueError("bfloat16 gradients need bfloat16 tensors")
    _same_layout(Q, *grads)
    return bf


def _check_d_rel(g, shp, Q, d_rel) -> None:
    if d_rel.dtype != torch.float32 or tuple(d_rel.shape) != (g.num_levels, g.rel_width, shp.D) or \
            not d_rel.is_contiguous() or d_rel.device != Q.device:
        raise ValueError("d_rel must be contiguous fp32 [%d,%d,%d] on the tensors' device"
                         % (g.num_levels, g.rel_width, shp.D))


def _check_bwd_workspace(L, g, shp, workspace) -> int:
    need = _need(int(L.bpt_attn_bwd_workspace(g.handle, ctypes.byref(shp))), "bpt_attn_bwd_workspace")
    ws_bytes = workspace.numel() * workspace.element_size()
    if ws_bytes < need:
        raise ValueError("the backward needs a workspace of %d bytes, got %d" % (need, ws_bytes))
    return ws_bytes


def _bwd_prepare(g, Q, K, V, rel, lse, dout, scale, grads, workspace, seq_len=None, dropout=None, leave_unkept=False,
                 bf16_grads=False):
    L = load_library()
    if grads is None:
        gdt = torch.bfloat16 if bf16_grads else torch.float32
        dQ, dK, dV = (torch.empty_strided(Q.shape, Q.stride(), dtype=gdt, device=Q.device) for _ in range(3))
        d_rel = torch.empty((g.num_levels, g.rel_width, Q.shape[3]), dtype=torch.float32, device=Q.device)
    else:
        dQ, dK, dV, d_rel = grads
    shp = _shape_of(g, Q, scale, seq_len, dropout, leave_unkept, _check_grad(Q, dQ, dK, dV))
    _check_bwd_inputs(g, shp, Q, K, V, rel, lse, dout)
    _check_d_rel(g, shp, Q, d_rel)
    if workspace is None:
        need = _need(int(L.bpt_attn_bwd_workspace(g.handle, ctypes.byref(shp))), "bpt_attn_bwd_workspace")
        workspace, _ = _workspace(max(need, 256), Q.device)
    ws_bytes = _check_bwd_workspace(L, g, shp, workspace)
    return L, shp, (dQ, dK, dV, d_rel), workspace, ws_bytes


def bpt_attn_bwd(g: Graph, Q, K, V, rel, lse, dout, scale: Optional[float] = None,
                 grads: Optional[Tuple[torch.Tensor, ...]] = None, workspace: Optional[torch.Tensor] = None,
                 seq_len: Optional[torch.Tensor] = None, dropout: Optional[Tuple[float, int]] = None, leave_unkept: bool = False,
                 bf16_grads: bool = False):
    """dQ, dK, dV, d_rel = gradient of eq. (8) given dout and the forward's lse (and its dropout).  All fp32; with
    bf16_grads (or bf16 tensors passed in `grads`) dQ, dK, dV are rounded to bf16 (bpt_shape_t.grad_dtype)."""
    L, shp, (dQ, dK, dV, d_rel), ws, ws_bytes = _bwd_prepare(g, Q, K, V, rel, lse, dout, scale, grads, workspace,
                                                             seq_len, dropout, leave_unkept, bf16_grads)
    _check(L.bpt_attn_bwd(g.handle, ctypes.byref(shp), Q.data_ptr(), K.data_ptr(), V.data_ptr(), rel.data_ptr(),
                          lse.data_ptr(), dout.data_ptr(), dQ.data_ptr(), dK.data_ptr(), dV.data_ptr(),
                          d_rel.data_ptr(), ws.data_ptr(), ws_bytes, _stream_ptr()), "bpt_attn_bwd")
    return dQ, dK, dV, d_rel


def bpt_attn_bwd_query_side(g: Graph, Q, K, V, rel, lse, dout, dQ, d_rel, workspace,
                            scale: Optional[float] = None, seq_len: Optional[torch.Tensor] = None,
                            dropout: Optional[Tuple[float, int]] = None, leave_unkept: bool = False):
    """First stage of the backward: dQ, d_rel, and delta into the workspace."""
    L = load_library()
    shp = _shape_of(g, Q, scale, seq_len, dropout, leave_unkept, _check_grad(Q, dQ))
    _check_bwd_inputs(g, shp, Q, K, V, rel, lse, dout)
    _check_d_rel(g, shp, Q, d_rel)
    _check_bwd_workspace(L, g, shp, workspace)
    _check(L.bpt_attn_bwd_query_side(g.handle, ctypes.byref(shp), Q.data_ptr(), K.data_ptr(), V.data_ptr(),
                                     rel.data_ptr(), lse.data_ptr(), dout.data_ptr(), dQ.data_ptr(),
                                     d_rel.data_ptr(), workspace.data_ptr(), workspace.numel() * workspace.element_size(),
                                     _stream_ptr()), "bpt_attn_bwd_query_side")
    return dQ, d_rel


def bpt_attn_bwd_key_side(g: Graph, Q, K, V, rel, lse, dout, dK, dV, workspace, scale: Optional[float] = None,
                          seq_len: Optional[torch.Tensor] = None, dropout: Optional[Tuple[float, int]] = None, leave_unkept: bool = False):
    """Second stage of the backward: dK, dV (reads delta from the workspace)."""
    L = load_library()
    shp = _shape_of(g, Q, scale, seq_len, dropout, leave_unkept, _check_grad(Q, dK, dV))
    _check_bwd_inputs(g, shp, Q, K, V, rel, lse, dout)
    _check_bwd_workspace(L, g, shp, workspace)
    _check(L.bpt_attn_bwd_key_side(g.handle, ctypes.byref(shp), Q.data_ptr(), K.data_ptr(), V.data_ptr(),
                                   rel.data_ptr(), lse.data_ptr(), dout.data_ptr(), dK.data_ptr(), dV.data_ptr(),
                                   workspace.data_ptr(),
                                   workspace.numel() * workspace.element_size(), _stream_ptr()),
           "bpt_attn_bwd_key_side")
    return dK, dV


def _layer_params(g: Graph, B: int, device, rel: torch.Tensor, params: dict, heads: int, eps: float,
                  seq_len: Optional[torch.Tensor]):
    """Checks the table, the parameters and the lengths of a layer call on B batch entries; returns (d_ff, the
    parameter struct, the seq_len pointer)."""
    d = heads * 64
    if rel.dtype != torch.bfloat16 or tuple(rel.shape) != (g.num_levels, g.rel_width, 64) or not rel.is_contiguous():
        raise ValueError("rel must be contiguous bf16 [%d,%d,64]" % (g.num_levels, g.rel_width))
    d_ff = params["W1"].shape[1]
    want = {"Wq": (d, d), "Wk": (d, d), "Wv": (d, d), "Wo": (d, d), "W1": (d, d_ff), "W2": (d_ff, d), "b1": (d_ff,),
            "b2": (d,), "g1": (d,), "beta1": (d,), "g2": (d,), "beta2": (d,)}
    for name, shape in want.items():
        t = params[name]
        dt = torch.bfloat16 if name.startswith("W") else torch.float32
        if t.dtype != dt or tuple(t.shape) != shape or not t.is_contiguous() or t.device != device:
            raise ValueError("parameter %s must be a contiguous %s tensor of shape %s on the device of the input"
                             % (name, dt, shape))
    lens = None
    if seq_len is not None:
        if seq_len.dtype != torch.int32 or tuple(seq_len.shape) != (B,) or not seq_len.is_contiguous():
            raise ValueError("seq_len must be a contiguous int32 tensor of B entries")
        lens = seq_len.data_ptr()
    lp = BptLayerParams(*[params[n].data_ptr() for n in ("Wq", "Wk", "Wv", "Wo", "W1", "W2", "b1", "b2", "g1", "beta1",
                                                          "g2", "beta2")], d_ff, float(eps))
    return d_ff, lp, lens


def _layer_args(g: Graph, X: torch.Tensor, rel: torch.Tensor, params: dict, heads: int, eps: float,
                seq_len: Optional[torch.Tensor]):
    """Checks the tensors of a layer call; returns (d_ff, the parameter struct, the seq_len pointer)."""
    d = heads * 64
    if X.dtype != torch.bfloat16 or X.dim() != 3 or X.shape[1] != g.num_nodes or X.shape[2] != d or not X.is_contiguous():
        raise ValueError("X must be a contiguous bf16 [B, %d, %d] tensor" % (g.num_nodes, d))
    return _layer_params(g, X.shape[0], X.device, rel, params, heads, eps, seq_len)


def bpt_layer_fwd(g: Graph, X: torch.Tensor, rel: torch.Tensor, params: dict, heads: int, scale: Optional[float] = None,
                  eps: float = 1e-5, seq_len: Optional[torch.Tensor] = None, out: Optional[torch.Tensor] = None,
                  workspace: Optional[torch.Tensor] = None) -> torch.Tensor:
    """One graph layer, forward (Sec. 3.3): X [B, N, heads*64] bf16 -> Y of the same shape.  params: Wq, Wk, Wv,
    Wo [d, d], W1 [d, d_ff], W2 [d_ff, d] in bf16 and b1, b2, g1, beta1, g2, beta2 in fp32, all contiguous cuda tensors.
    Pass a `workspace` (layer_workspace_bytes) to keep the activations for bpt_layer_bwd."""
    L = load_library()
    d_ff, lp, lens = _layer_args(g, X, rel, params, heads, eps, seq_len)
    if out is None:
        out = torch.empty_like(X)
    need = _need(int(L.bpt_layer_fwd_workspace(g.handle, X.shape[0], heads, d_ff)), "bpt_layer_fwd_workspace")
    if workspace is None:
        workspace = torch.empty(max(need, 256), dtype=torch.uint8, device=X.device)
    _check(L.bpt_layer_fwd(g.handle, X.shape[0], heads, float(scale) if scale else 0.0, lens, rel.data_ptr(), X.data_ptr(),
                           ctypes.byref(lp), out.data_ptr(), workspace.data_ptr(), workspace.numel(), _stream_ptr()),
           "bpt_layer_fwd")
    return out


def layer_workspace_bytes(g: Graph, B: int, heads: int, d_ff: int) -> Tuple[int, int]:
    """Bytes of workspace bpt_layer_fwd and bpt_layer_bwd need."""
    L = load_library()
    return (_need(int(L.bpt_layer_fwd_workspace(g.handle, B, heads, d_ff)), "bpt_layer_fwd_workspace"), _need(int(L.bpt_layer_bwd_workspace(g.handle, B, heads, d_ff)), "bpt_layer_bwd_workspace"))


def bpt_layer_bwd(g: Graph, X: torch.Tensor, rel: torch.Tensor, params: dict, heads: int, fwd_workspace: torch.Tensor,
                  dY: torch.Tensor, scale: Optional[float] = None, eps: float = 1e-5,
                  seq_len: Optional[torch.Tensor] = None, dX: Optional[torch.Tensor] = None,
                  grads: Optional[dict] = None, d_rel: Optional[torch.Tensor] = None,
                  workspace: Optional[torch.Tensor] = None):
    """Backward of bpt_layer_fwd, called with the same arguments and the workspace that call filled.  dY: bf16
    like X.  Returns (dX bf16, d_rel fp32, grads: dict of fp32 tensors named dWq ... dbeta2, shaped like their
    parameters)."""
    L = load_library()
    d_ff, lp, lens = _layer_args(g, X, rel, params, heads, eps, seq_len)
    if dY.dtype != torch.bfloat16 or dY.shape != X.shape or not dY.is_contiguous() or dY.device != X.device:
        raise ValueError("dY must be a contiguous bf16 tensor shaped like X")
    if dX is None:
        dX = torch.empty_like(X)
    if d_rel is None:
        d_rel = torch.empty(rel.shape, dtype=torch.float32, device=X.device)
    if grads is None:
        grads = {"d" + n: torch.empty(params[n].shape, dtype=torch.float32, device=X.device)
                 for n in ("Wq", "Wk", "Wv", "Wo", "W1", "b1", "W2", "b2", "g1", "beta1", "g2", "beta2")}
    for name in GRAD_NAMES:
        t = grads[name]
        if t.dtype != torch.float32 or t.shape != params[name[1:]].shape or not t.is_contiguous() or t.device != X.device:
            raise ValueError("gradient %s must be a contiguous fp32 tensor shaped like its parameter" % name)
    lg = BptLayerGrads(*[grads[n].data_ptr() for n in GRAD_NAMES])
    need = _need(int(L.bpt_layer_bwd_workspace(g.handle, X.shape[0], heads, d_ff)), "bpt_layer_bwd_workspace")
    if workspace is None:
        workspace = torch.empty(max(need, 256), dtype=torch.uint8, device=X.device)
    _check(L.bpt_layer_bwd(g.handle, X.shape[0], heads, float(scale) if scale else 0.0, lens, rel.data_ptr(), X.data_ptr(),
                           ctypes.byref(lp), fwd_workspace.data_ptr(), fwd_workspace.numel(), dY.data_ptr(), dX.data_ptr(),
                           d_rel.data_ptr(), ctypes.byref(lg), workspace.data_ptr(), workspace.numel(), _stream_ptr()),
           "bpt_layer_bwd")
    return dX, d_rel, grads


def _stack_args(g: Graph, E: torch.Tensor, rels, params, heads: int, eps: float, seq_len: Optional[torch.Tensor]):
    """Checks the tensors of a stack call; returns (d_ff, array of parameter structs, array of rel pointers, the
    seq_len pointer)."""
    d = heads * 64
    if E.dtype != torch.bfloat16 or E.dim() != 3 or E.shape[1] != g.n_tokens or E.shape[2] != d or not E.is_contiguous():
        raise ValueError("E must be a contiguous bf16 [B, %d, %d] tensor" % (g.n_tokens, d))
    if g.is_batch and (E.shape[0] != 1 or seq_len is not None):
        raise ValueError("the graph of a packed batch takes E [1, tokens of all sequences, d] and no seq_len")
    if len(params) < 1 or len(rels) != len(params):
        raise ValueError("one parameter dict and one rel table per layer")
    structs, lens, d_ff = [], None, None
    for rel, p in zip(rels, params):
        f, lp, lens = _layer_params(g, E.shape[0], E.device, rel, p, heads, eps, seq_len)
        if d_ff is not None and f != d_ff:
            raise ValueError("every layer must have the same d_ff")
        d_ff = f
        structs.append(lp)
    return (d_ff, (BptLayerParams * len(params))(*structs),
            (ctypes.c_void_p * len(rels))(*[r.data_ptr() for r in rels]), lens)


def stack_workspace_bytes(g: Graph, B: int, heads: int, d_ff: int, num_layers: int) -> Tuple[int, int]:
    """Bytes of workspace bpt_stack_fwd and bpt_stack_bwd need."""
    L = load_library()
    return (_need(int(L.bpt_stack_fwd_workspace(g.handle, B, heads, d_ff, num_layers)), "bpt_stack_fwd_workspace"),
            _need(int(L.bpt_stack_bwd_workspace(g.handle, B, heads, d_ff)), "bpt_stack_bwd_workspace"))


def bpt_stack_fwd(g: Graph, E: torch.Tensor, rels, params, heads: int, scale: Optional[float] = None, eps: float = 1e-5,
                  seq_len: Optional[torch.Tensor] = None, want_root: bool = True, want_tokens: bool = True,
                  workspace: Optional[torch.Tensor] = None):
    """The update of the graph (Sec. 3.3) over len(params) layers: E [B, n, heads*64] bf16 token embeddings ->
    (root [B, d] or None, tokens [B, n, d] or None); on the graph of a packed batch E and tokens are [1, T, d] (the tokens
    of all sequences in row order) and root is [sequences, d].  rels: one [levels, rel_width, 64] bf16 table per layer;
    params: one dict per layer as for bpt_layer_fwd.  Pass a `workspace` (stack_workspace_bytes) to keep the
    activations for bpt_stack_bwd."""
    L = load_library()
    d_ff, lps, relp, lens = _stack_args(g, E, rels, params, heads, eps, seq_len)
    if not (want_root or want_tokens):
        raise ValueError("ask for the root, the tokens or both")
    B, d = E.shape[0], heads * 64
    roots = g.batch if g.is_batch else B      # one root per sequence
    root = torch.empty((roots, d), dtype=E.dtype, device=E.device) if want_root else None
    tokens = torch.empty_like(E) if want_tokens else None
    need = _need(int(L.bpt_stack_fwd_workspace(g.handle, B, heads, d_ff, len(params))), "bpt_stack_fwd_workspace")
    if workspace is None:
        workspace = torch.empty(max(need, 256), dtype=torch.uint8, device=E.device)
    _check(L.bpt_stack_fwd(g.handle, B, heads, len(params), float(scale) if scale else 0.0, lens, relp, E.data_ptr(), lps,
                           root.data_ptr() if want_root else None, tokens.data_ptr() if want_tokens else None,
                           workspace.data_ptr(), workspace.numel(), _stream_ptr()), "bpt_stack_fwd")
    return root, tokens


def bpt_stack_bwd(g: Graph, E: torch.Tensor, rels, params, heads: int, fwd_workspace: torch.Tensor,
                  d_root: Optional[torch.Tensor], d_tokens: Optional[torch.Tensor], scale: Optional[float] = None,
                  eps: float = 1e-5, seq_len: Optional[torch.Tensor] = None, workspace: Optional[torch.Tensor] = None):
    """Backward of bpt_stack_fwd, called with the same arguments and the workspace that call filled.  d_root [B, d]
    and / or d_tokens [B, n, d] in bf16.  Returns (dE bf16 like E, list of d_rel fp32 per layer, list of dicts of
    fp32 parameter gradients per layer)."""
    L = load_library()
    d_ff, lps, relp, lens = _stack_args(g, E, rels, params, heads, eps, seq_len)
    B, d = E.shape[0], heads * 64
    for name, t, shape in (("d_root", d_root, (g.batch if g.is_batch else B, d)), ("d_tokens", d_tokens, tuple(E.shape))):
        if t is not None and (t.dtype != torch.bfloat16 or tuple(t.shape) != shape or not t.is_contiguous()
                              or t.device != E.device):
            raise ValueError("%s must be a contiguous bf16 tensor of shape %s on the device of E" % (name, shape))
    if d_root is None and d_tokens is None:
        raise ValueError("pass d_root, d_tokens or both")
    dE = torch.empty_like(E)
    d_rels = [torch.empty(r.shape, dtype=torch.float32, device=E.device) for r in rels]
    grads = [{"d" + n: torch.empty(p[n].shape, dtype=torch.float32, device=E.device) for n in
              ("Wq", "Wk", "Wv", "Wo", "W1", "b1", "W2", "b2", "g1", "beta1", "g2", "beta2")} for p in params]
    lgs = (BptLayerGrads * len(params))(*[BptLayerGrads(*[gr[n].data_ptr() for n in GRAD_NAMES]) for gr in grads])
    drp = (ctypes.c_void_p * len(rels))(*[t.data_ptr() for t in d_rels])
    need = _need(int(L.bpt_stack_bwd_workspace(g.handle, B, heads, d_ff)), "bpt_stack_bwd_workspace")
    if workspace is None:
        workspace = torch.empty(max(need, 256), dtype=torch.uint8, device=E.device)
    _check(L.bpt_stack_bwd(g.handle, B, heads, len(params), float(scale) if scale else 0.0, lens, relp, lps,
                           fwd_workspace.data_ptr(), fwd_workspace.numel(),
                           d_root.data_ptr() if d_root is not None else None,
                           d_tokens.data_ptr() if d_tokens is not None else None, dE.data_ptr(), drp, lgs,
                           workspace.data_ptr(), workspace.numel(), _stream_ptr()), "bpt_stack_bwd")
    return dE, d_rels, grads


class GraphAttentionFunction(torch.autograd.Function):
    """Graph self-attention (eq. (8)) as a torch.autograd.Function: the forward and the backward are
    the library's bpt_attn_fwd / bpt_attn_bwd, nothing is computed in Python.  dQ, dK, dV leave the
    backward's kernels in the dtype of their inputs (for bf16 rounded once from the fp32 sums, which saves a pass of
    casts over them: 32 sentences on trees over 512 tokens, forward + backward 278 -> 201 us); d_rel is cast."""

    @staticmethod
    def forward(ctx, g, Q, K, V, rel, scale, seq_len, dropout):
        out, lse = bpt_attn_fwd(g, Q, K, V, rel, scale=scale, seq_len=seq_len, dropout=dropout)
        ctx.save_for_backward(Q, K, V, rel, lse)
        ctx.g, ctx.scale, ctx.seq_len, ctx.dropout = g, scale, seq_len, dropout
        return out

    @staticmethod
    def backward(ctx, dout):
        Q, K, V, rel, lse = ctx.saved_tensors
        if dout.stride() != Q.stride():
            dout = torch.empty_strided(Q.shape, Q.stride(), dtype=Q.dtype, device=Q.device).copy_(dout)
        dQ, dK, dV, d_rel = bpt_attn_bwd(ctx.g, Q, K, V, rel, lse, dout.to(Q.dtype), scale=ctx.scale, seq_len=ctx.seq_len,
                                         dropout=ctx.dropout, bf16_grads=Q.dtype == torch.bfloat16)
        return None, dQ, dK, dV, d_rel.to(rel.dtype), None, None, None


def graph_attention(g: Graph, Q, K, V, rel, scale: Optional[float] = None, seq_len: Optional[torch.Tensor] = None,
                    dropout: Optional[Tuple[float, int]] = None):
    """out = graph self-attention of eq. (8), differentiable with respect to Q, K, V and rel; dropout = (rate, seed)
    of the dropout on the attention weights (give every call of a training step its own seed)."""
    return GraphAttentionFunction.apply(g, Q, K, V, rel, scale, seq_len, dropout)


def bpt_profile_enable(on: bool) -> None:
    _check(load_library().bpt_profile_enable(int(bool(on))), "bpt_profile_enable")


def bpt_profile_report() -> dict:
    """{kernel name: (launches, total milliseconds)} of the launches recorded since profiling was enabled."""
    L = load_library()
    need = int(L.bpt_profile_report(None, 0))
    if need < 0:
        raise BptError(BPT_ERR_LAUNCH, "bpt_profile_report")
    buf = ctypes.create_string_buffer(max(need, 1))
    L.bpt_profile_report(buf, need)
    out = {}
    for line in buf.value.decode().splitlines():
        name, calls, ms = line.rsplit(" ", 2)
        out[name] = (int(calls), float(ms))
    return out


def workspace_bytes(g: Graph, like: torch.Tensor, scale: Optional[float] = None) -> Tuple[int, int]:
    L = load_library()
    shp = _shape_of(g, like, scale)
    return (_need(int(L.bpt_attn_fwd_workspace(g.handle, ctypes.byref(shp))), "bpt_attn_fwd_workspace"),
            _need(int(L.bpt_attn_bwd_workspace(g.handle, ctypes.byref(shp))), "bpt_attn_bwd_workspace"))


def bpt_calibrate_gather(src: torch.Tensor, perm: torch.Tensor, dst: torch.Tensor) -> None:
    """dst row i = src row perm[i] for rows of 128 bytes: a gather of known traffic for scaling hardware counters."""
    rows = perm.numel()
    if perm.dtype != torch.int32 or not perm.is_contiguous() or not src.is_contiguous() or not dst.is_contiguous():
        raise ValueError("perm must be contiguous int32, src and dst contiguous")
    if src.numel() * src.element_size() != rows * 128 or dst.numel() * dst.element_size() != rows * 128:
        raise ValueError("src and dst must hold one row of 128 bytes per entry of perm")
    _check(load_library().bpt_calibrate_gather(src.data_ptr(), perm.data_ptr(), dst.data_ptr(), rows, _stream_ptr()),
           "bpt_calibrate_gather")
