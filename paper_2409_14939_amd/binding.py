"""Binding of libfastgl_agg.so - same names as the C ABI, argument marshalling
only.  PyTorch supplies device memory and the stream handle; every step of the
computation runs in the library's kernels.  The calls that enqueue work are
marshalled natively (csrc/host.cpp: argument checks, allocation of what the
caller did not pass, the current stream), because a small mini-batch is bound by
exactly that; size queries and host-side calls go through ctypes.  There is no
fallback: if a library is missing or an entry point fails, this module raises.
"""
from __future__ import annotations

import ctypes
import os
from typing import Optional

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libfastgl_agg.so")

FASTGL_OK = 0
FASTGL_ERR_INVALID_ARG, FASTGL_ERR_UNSUPPORTED, FASTGL_ERR_WORKSPACE, FASTGL_ERR_HIP = 1, 2, 3, 4
MODES = {"sum": 0, "mean": 1, "gcn": 2}
DTYPES = {"f32": 0, "bf16": 1}
PLAN_FWD, PLAN_BWD, PLAN_ALL, PLAN_SRC_DEG, PLAN_PERM, PLAN_SHORT_DST_ROWS = 1, 2, 3, 4, 8, 16

EXPORTS = [
    "fastgl_block_aggregate_fwd", "fastgl_block_aggregate_bwd", "fastgl_block_aggregate_fwd_static",
    "fastgl_block_plan_bytes",
    "fastgl_block_plan_create", "fastgl_block_plan_create_many", "fastgl_block_plan_export", "fastgl_block_plan_destroy",
    "fastgl_block_workspace_bytes", "fastgl_long_row_threshold", "fastgl_long_row_chunk", "fastgl_work_per_group",
    "fastgl_aggregate_column_tiles", "fastgl_gather_rows", "fastgl_block_validate", "fastgl_last_error",
    "fastgl_update_fwd", "fastgl_update_bwd", "fastgl_update_bwd_workspace_bytes", "fastgl_update_slab_rows",
    "fastgl_update_fwd_bf16", "fastgl_update_bwd_bf16", "fastgl_layer_fwd", "fastgl_layer_fwd_fuses",
    "fastgl_idmap", "fastgl_idmap_table_slots", "fastgl_idmap_workspace_bytes",
    "fastgl_match", "fastgl_match_workspace_bytes", "fastgl_assemble_rows", "fastgl_overlap_counts",
    "fastgl_overlap_workspace_bytes", "fastgl_greedy_reorder",
    "fastgl_edge_workspace_bytes", "fastgl_edge_weight_grad", "fastgl_edge_softmax_fwd", "fastgl_edge_softmax_bwd",
    "fastgl_edge_softmax_long_row", "fastgl_edge_score_fwd", "fastgl_edge_score_bwd",
]
MAX_REORDER_BATCHES = 64
IDMAP_MODES = {"ordered": 0, "fused": 1}


class FastglError(RuntimeError):
    def __init__(self, status: int, msg: str):
        super().__init__(f"fastgl status {status}: {msg}")
        self.status = status


class BlockDesc(ctypes.Structure):
    _fields_ = [("indptr", ctypes.c_void_p), ("indices", ctypes.c_void_p), ("num_dst", ctypes.c_int64),
                ("num_src", ctypes.c_int64), ("num_edges", ctypes.c_int64), ("parts", ctypes.c_int),
                ("plan_mem", ctypes.c_void_p), ("plan_bytes", ctypes.c_size_t)]


class PlanView(ctypes.Structure):
    _fields_ = [(n, ctypes.c_void_p) for n in (
        "din", "dout", "indptr_T", "indices_T", "perm", "dst_inv", "dst_rsqrt", "src_rsqrt",
        "long_dst", "chunk_ptr_dst", "long_src", "chunk_ptr_src", "counters", "split_dst", "split_src")]


_lib = None
_host = None


def lib() -> ctypes.CDLL:
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise ImportError(f"{LIB_PATH} is not built; run `python -c 'import __graft_entry__ as g; g.build()'`")
        L = ctypes.CDLL(LIB_PATH)
        p, i64, i32, sz = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int, ctypes.c_size_t
        agg = [p, p, p, i64, i64, i64, i64, i32, i32, p, p, p, p, sz, p]
        L.fastgl_block_aggregate_fwd.argtypes = agg
        L.fastgl_block_aggregate_bwd.argtypes = agg
        L.fastgl_block_aggregate_fwd_static.argtypes = [p, p, p, i64, i64, i64, i64, i32, i32, p, p, p]
        L.fastgl_block_plan_bytes.argtypes = [i64, i64, i64]
        L.fastgl_block_plan_bytes.restype = sz
        L.fastgl_block_plan_create.argtypes = [p, p, i64, i64, i64, i32, p, sz, p, ctypes.POINTER(p)]
        L.fastgl_block_plan_create_many.argtypes = [i32, ctypes.POINTER(BlockDesc), p, ctypes.POINTER(p)]
        L.fastgl_block_plan_export.argtypes = [p, ctypes.POINTER(PlanView)]
        L.fastgl_block_plan_destroy.argtypes = [p]
        L.fastgl_block_plan_destroy.restype = None
        L.fastgl_block_workspace_bytes.argtypes = [i64, i64, i64, i64, i32]
        L.fastgl_block_workspace_bytes.restype = sz
        L.fastgl_long_row_threshold.restype = ctypes.c_int32
        L.fastgl_long_row_chunk.restype = ctypes.c_int32
        L.fastgl_work_per_group.restype = ctypes.c_int32
        L.fastgl_aggregate_column_tiles.argtypes = [i64, i64, i64, i64, i32]
        L.fastgl_aggregate_column_tiles.restype = ctypes.c_int32
        L.fastgl_gather_rows.argtypes = [p, i64, p, i64, i64, i32, p, p]
        L.fastgl_block_validate.argtypes = [p, p, i64, i64, i64, p, ctypes.POINTER(i64), p]
        L.fastgl_last_error.restype = ctypes.c_char_p
        L.fastgl_update_fwd.argtypes = [p, p, p, i64, i64, i64, i32, p, p]
        L.fastgl_update_fwd_bf16.argtypes = L.fastgl_update_fwd.argtypes
        L.fastgl_update_bwd_workspace_bytes.argtypes = [i64, i64, i64]
        L.fastgl_update_bwd_workspace_bytes.restype = sz
        L.fastgl_update_bwd.argtypes = [p, p, p, p, i64, i64, i64, i32, p, p, p, p, sz, p]
        L.fastgl_match_workspace_bytes.argtypes = [i64, i64]
        L.fastgl_match_workspace_bytes.restype = sz
        L.fastgl_match.argtypes = [p, i64, p, i64, p, p, p, p, p, sz, p]
        L.fastgl_assemble_rows.argtypes = [p, i64, p, i64, p, i64, i64, i32, p, p]
        L.fastgl_overlap_workspace_bytes.argtypes = [i64]
        L.fastgl_overlap_workspace_bytes.restype = sz
        L.fastgl_overlap_counts.argtypes = [p, ctypes.POINTER(i64), i32, p, p, p, sz, p]
        L.fastgl_greedy_reorder.argtypes = [ctypes.POINTER(i64), ctypes.POINTER(i64), i64,
                                            ctypes.POINTER(ctypes.c_int32)]
        L.fastgl_edge_workspace_bytes.argtypes = [i64, i64]
        L.fastgl_edge_workspace_bytes.restype = sz
        L.fastgl_edge_weight_grad.argtypes = [p, p, i64, i64, i64, i64, i32, i32, p, p, p, p, p, sz, p]
        L.fastgl_edge_softmax_fwd.argtypes = [p, i64, i64, p, p, p, sz, p]
        L.fastgl_edge_softmax_bwd.argtypes = [p, i64, i64, p, p, p, p, sz, p]
        L.fastgl_edge_softmax_long_row.restype = ctypes.c_int32
        L.fastgl_edge_score_fwd.argtypes = [p, p, i64, i64, i64, p, p, ctypes.c_float, p, p]
        L.fastgl_edge_score_bwd.argtypes = [p, p, i64, i64, i64, p, p, ctypes.c_float, p, p, p, p, p]
        L.fastgl_idmap_table_slots.argtypes = [i64]
        L.fastgl_idmap_table_slots.restype = i64
        L.fastgl_idmap_workspace_bytes.argtypes = [i64, i64]
        L.fastgl_idmap_workspace_bytes.restype = sz
        L.fastgl_idmap.argtypes = [p, i64, p, i64, i32, p, p, p, p, sz, p]
        L.fastgl_update_bwd_bf16.argtypes = L.fastgl_update_bwd.argtypes
        L.fastgl_layer_fwd.argtypes = [p, p, p, i64, i64, i64, i64, i32, i32, p, p, p, i64, i32, p, p, p, p, sz, p]
        L.fastgl_layer_fwd_fuses.argtypes = [i64, i64, i32]
        L.fastgl_update_slab_rows.argtypes = [i64, i64, i64]
        L.fastgl_update_slab_rows.restype = ctypes.c_int32
        _lib = L
    return _lib


def fastgl_last_error() -> str:
    return lib().fastgl_last_error().decode()


def _check(status: int) -> None:
    if status != FASTGL_OK:
        raise FastglError(status, fastgl_last_error())


def _native():
    """The native marshalling module, loaded on first use (it needs the built library next to it)."""
    global _host
    if _host is None:
        lib()
        try:
            from . import _host as module
        except ImportError as e:
            raise ImportError(f"the native half of the binding is not built ({e}); run "
                              "`python -c 'import __graft_entry__ as g; g.build()'`") from e
        module.set_error_class(FastglError)
        _host = module
    return _host


def _ptr(t: Optional[torch.Tensor]):
    return None if t is None else ctypes.c_void_p(t.data_ptr())


def _stream():
    return ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)


def _dev(t: torch.Tensor, dtype, name: str) -> torch.Tensor:
    if not t.is_cuda or t.dtype != dtype or not t.is_contiguous():
        raise TypeError(f"{name} must be a contiguous device tensor of {dtype}")
    return t


def fastgl_long_row_threshold() -> int:
    return int(lib().fastgl_long_row_threshold())


def fastgl_long_row_chunk() -> int:
    return int(lib().fastgl_long_row_chunk())


def fastgl_work_per_group() -> int:
    return int(lib().fastgl_work_per_group())


def fastgl_block_plan_bytes(num_dst: int, num_src: int, num_edges: int) -> int:
    return int(lib().fastgl_block_plan_bytes(num_dst, num_src, num_edges))


def fastgl_block_workspace_bytes(num_dst: int, num_src: int, num_edges: int, feat: int, dtype: str) -> int:
    return int(lib().fastgl_block_workspace_bytes(num_dst, num_src, num_edges, feat, DTYPES[dtype]))


class Plan:
    """Owner of one fastgl_plan handle and of the device buffer behind it."""

    def __init__(self, handle, mem, indptr, indices, num_src):
        self.handle, self.mem = handle, mem                   # the handle: c_void_p (or an address), None once destroyed
        self.indptr, self.indices, self.num_src = indptr, indices, num_src

    def export(self) -> PlanView:
        v = PlanView()
        _check(lib().fastgl_block_plan_export(self.handle, ctypes.byref(v)))
        return v

    def destroy(self) -> None:
        if self.handle is not None and _lib is not None:      # _lib is gone while the interpreter shuts down
            _lib.fastgl_block_plan_destroy(self.handle)
        self.handle = None

    def __del__(self):
        self.destroy()


def fastgl_block_plan_create(indptr: torch.Tensor, indices: torch.Tensor, num_src: int,
                             parts: int = PLAN_ALL, plan_mem: Optional[torch.Tensor] = None) -> Plan:
    return fastgl_block_plan_create_many(((indptr, indices, num_src),), parts,
                                         None if plan_mem is None else (plan_mem,))[0]


def fastgl_block_plan_create_many(blocks, parts: int = PLAN_ALL, plan_mems=None):
    """blocks: list of (indptr, indices, num_src); returns one Plan per block, built together."""
    made = _native().plan_create_many(blocks, parts, plan_mems)
    return [Plan(ctypes.c_void_p(h), mem, *b) for (h, mem), b in zip(made, blocks)]


def fastgl_block_aggregate_fwd(indptr, indices, edge_w, num_src: int, mode: str, X: torch.Tensor,
                               out: Optional[torch.Tensor] = None, plan: Optional[Plan] = None,
                               workspace: Optional[torch.Tensor] = None) -> torch.Tensor:
    return _native().aggregate(False, indptr, indices, edge_w, num_src, MODES[mode], X, out, plan, workspace)


STATIC_SCRATCH_BYTES = 64 << 20


def fastgl_block_aggregate_fwd_static(indptr, indices, edge_w, num_src: int, mode: str, X: torch.Tensor,
                                      out: torch.Tensor) -> torch.Tensor:
    """The forward aggregation on the library's static scratch array: no plan, no workspace, and this
    wrapper allocates nothing either (the caller passes `out`)."""
    return _native().aggregate_static(indptr, indices, edge_w, num_src, MODES[mode], X, out)


def fastgl_block_aggregate_bwd(indptr, indices, edge_w, num_src: int, mode: str, grad_out: torch.Tensor,
                               grad_X: Optional[torch.Tensor] = None, plan: Optional[Plan] = None,
                               workspace: Optional[torch.Tensor] = None) -> torch.Tensor:
    return _native().aggregate(True, indptr, indices, edge_w, num_src, MODES[mode], grad_out, grad_X, plan, workspace)


def fastgl_gather_rows(table: torch.Tensor, ids: torch.Tensor, out: Optional[torch.Tensor] = None) -> torch.Tensor:
    return _native().gather_rows(table, ids, out)


def fastgl_block_validate(indptr: torch.Tensor, indices: torch.Tensor, num_src: int) -> int:
    _dev(indptr, torch.int32, "indptr")
    _dev(indices, torch.int32, "indices")
    scratch = torch.empty(2, dtype=torch.int64, device=indptr.device)
    n = ctypes.c_int64(-1)
    _check(lib().fastgl_block_validate(_ptr(indptr), _ptr(indices), indptr.numel() - 1, num_src,
                                       indices.numel(), _ptr(scratch), ctypes.byref(n), _stream()))
    return int(n.value)


def fastgl_update_slab_rows(M: int, K: int, N: int) -> int:
    return int(lib().fastgl_update_slab_rows(M, K, N))


def fastgl_update_bwd_workspace_bytes(M: int, K: int, N: int) -> int:
    return int(lib().fastgl_update_bwd_workspace_bytes(M, K, N))


def fastgl_update_fwd(H: torch.Tensor, W: torch.Tensor, bias: Optional[torch.Tensor], relu: bool,
                      Y: Optional[torch.Tensor] = None) -> torch.Tensor:
    """H, W (and Y) float32, or all bfloat16 (the bias stays float32)."""
    return _native().update_fwd(H, W, bias, relu, Y)


def fastgl_layer_fwd_fuses(K: int, N: int, dtype: str) -> bool:
    return bool(lib().fastgl_layer_fwd_fuses(K, N, DTYPES[dtype]))


def fastgl_layer_fwd(indptr, indices, edge_w, num_src: int, mode: str, X: torch.Tensor, W: torch.Tensor,
                     bias: Optional[torch.Tensor], relu: bool, H: Optional[torch.Tensor] = None,
                     Y: Optional[torch.Tensor] = None, want_H: bool = True, plan: Optional[Plan] = None,
                     workspace: Optional[torch.Tensor] = None):
    """Aggregation + update of one layer in one call; returns (H, Y).  want_H=False (and H None) leaves the
    aggregated rows unwritten, which only shapes that fuse allow."""
    return _native().layer_fwd(indptr, indices, edge_w, num_src, MODES[mode], X, W, bias, relu, H, Y, want_H, plan,
                               workspace)


def fastgl_update_bwd(H: torch.Tensor, W: torch.Tensor, Y: Optional[torch.Tensor], dY: torch.Tensor, relu: bool,
                      want=("dH", "dW", "db"), dH=None, dW=None, db=None,
                      workspace: Optional[torch.Tensor] = None):
    """Returns (dH, dW, db); parts not named in `want` (and not passed in) are None.  H, W, Y, dY, dH
    float32, or all bfloat16; dW and db are float32 either way."""
    return _native().update_bwd(H, W, Y, dY, relu, dH is None and "dH" in want, dW is None and "dW" in want,
                                db is None and "db" in want, dH, dW, db, workspace)


def fastgl_idmap_table_slots(n_ids: int) -> int:
    return int(lib().fastgl_idmap_table_slots(n_ids))


def fastgl_idmap_workspace_bytes(n_dst: int, n_nbr: int) -> int:
    return int(lib().fastgl_idmap_workspace_bytes(n_dst, n_nbr))


def fastgl_idmap(dst_gid: torch.Tensor, nbr_gid: torch.Tensor, mode: str = "ordered",
                 local_nbr: Optional[torch.Tensor] = None, unique_gid: Optional[torch.Tensor] = None,
                 result: Optional[torch.Tensor] = None, workspace: Optional[torch.Tensor] = None):
    """Returns (local_nbr int32[n_nbr], unique_gid int64[n_dst+n_nbr], result int32[2]) - all on the
    device, nothing is synchronised: result[0] = number of distinct IDs, result[1] = violations."""
    return _native().idmap(dst_gid, nbr_gid, IDMAP_MODES[mode], local_nbr, unique_gid, result, workspace)


def fastgl_match_workspace_bytes(n_prev: int, n_new: int) -> int:
    return int(lib().fastgl_match_workspace_bytes(n_prev, n_new))


def fastgl_match(prev_gid: torch.Tensor, new_gid: torch.Tensor, src_row=None, load_pos=None, load_gid=None,
                 result=None, workspace=None):
    """Returns (src_row int32[n_new], load_pos int32[n_new], load_gid int64[n_new], result int32[2]) on
    the device, nothing synchronised: result[0] = rows to load, result[1] = violations."""
    return _native().match(prev_gid, new_gid, src_row, load_pos, load_gid, result, workspace)


def fastgl_assemble_rows(X_prev: torch.Tensor, X_load: torch.Tensor, src_row: torch.Tensor, n_load: int,
                         out: Optional[torch.Tensor] = None) -> torch.Tensor:
    """X_load may have more rows than n_load (a buffer sized for the worst case); the first n_load count."""
    return _native().assemble_rows(X_prev, X_load, src_row, n_load, out)


def fastgl_overlap_workspace_bytes(total_ids: int) -> int:
    return int(lib().fastgl_overlap_workspace_bytes(total_ids))


def fastgl_overlap_counts(gid: torch.Tensor, offsets, workspace: Optional[torch.Tensor] = None):
    """gid: the node lists of n mini-batches one after the other (device int64); offsets: n+1 host
    ints.  Returns (counts int64[n,n], violations int32[1]) on the device."""
    return _native().overlap_counts(gid, offsets, workspace)


def fastgl_greedy_reorder(overlap, sizes):
    """Host-side Algorithm 1: overlap = n x n nested sequence / array of ints, sizes = n ints."""
    n = len(sizes)
    flat = [int(x) for row in overlap for x in row]
    if len(flat) != n * n:
        raise ValueError("overlap must be n x n")
    ov = (ctypes.c_int64 * max(n * n, 1))(*flat)
    sz_ = (ctypes.c_int64 * max(n, 1))(*[int(x) for x in sizes])
    order = (ctypes.c_int32 * max(n, 1))()
    _check(lib().fastgl_greedy_reorder(ov, sz_, n, order))
    return [int(order[i]) for i in range(n)]


def fastgl_edge_workspace_bytes(num_dst: int, num_edges: int) -> int:
    return int(lib().fastgl_edge_workspace_bytes(num_dst, num_edges))


def fastgl_edge_softmax_long_row() -> int:
    return int(lib().fastgl_edge_softmax_long_row())


def fastgl_edge_weight_grad(indptr, indices, num_src: int, mode: str, X: torch.Tensor, grad_out: torch.Tensor,
                            plan: Optional[Plan] = None, grad_w: Optional[torch.Tensor] = None,
                            workspace: Optional[torch.Tensor] = None) -> torch.Tensor:
    return _native().edge_weight_grad(indptr, indices, num_src, MODES[mode], X, grad_out, plan, grad_w, workspace)


def fastgl_edge_softmax_fwd(indptr, score: torch.Tensor, alpha: Optional[torch.Tensor] = None,
                            workspace: Optional[torch.Tensor] = None) -> torch.Tensor:
    return _native().edge_softmax_fwd(indptr, score, alpha, workspace)


def fastgl_edge_softmax_bwd(indptr, alpha: torch.Tensor, grad_alpha: torch.Tensor,
                            grad_score: Optional[torch.Tensor] = None,
                            workspace: Optional[torch.Tensor] = None) -> torch.Tensor:
    return _native().edge_softmax_bwd(indptr, alpha, grad_alpha, grad_score, workspace)


def fastgl_edge_score_fwd(indptr, indices, el: torch.Tensor, er: torch.Tensor, slope: float,
                          score: Optional[torch.Tensor] = None) -> torch.Tensor:
    return _native().edge_score_fwd(indptr, indices, el, er, slope, score)


def fastgl_edge_score_bwd(indptr, indices, el: torch.Tensor, er: torch.Tensor, slope: float, grad_score: torch.Tensor,
                          plan: Optional[Plan] = None, want=("el", "er"), grad_el: Optional[torch.Tensor] = None,
                          grad_er: Optional[torch.Tensor] = None):
    """(grad_el, grad_er); `want` selects which are computed when no array is passed in (the other is
    None).  grad_er needs a plan built with PLAN_BWD | PLAN_PERM."""
    return _native().edge_score_bwd(indptr, indices, el, er, slope, grad_score, plan, grad_el is None and "el" in want,
                                    grad_er is None and "er" in want, grad_el, grad_er)
