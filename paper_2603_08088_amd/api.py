"""Thin Python binding of libeagletv.so: shapes, outputs and descriptors; csrc/binding.cpp makes the calls.

Each function has the name of the C entry point it calls (``include/eagletv.h``)
and takes torch tensors that already live on the GPU; outputs are allocated
with ``torch.empty`` unless passed in.  No step of the verification path runs
in Python or in torch ops.  The library must have been built
(``python -m paper_2603_08088_amd.build``); loading fails loudly otherwise -
there is no CPU fallback.
"""
from __future__ import annotations

import ctypes as C
import os
from typing import Dict, Optional

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libeagletv.so")
_lib = None
_calls = None

F32, BF16 = 0, 1
TREE_RANGE, TREE_CYCLE, TREE_CLOSURE = 1, 2, 4
COMMIT_CAPACITY, COMMIT_BAD_NODE, COMMIT_BAD_LEN, COMMIT_BAD_BLOCK = 1, 2, 4, 8
BRANCH_NO_BLOCKS, BRANCH_BAD_FREE = 16, 32
ATTN_FLAG_GENERIC = 1
ATTN_FLAG_SMALL_WG = 2
ATTN_FLAG_WHOLE_TILE = 4
ATTN_FLAG_KEY_HALVES = 8
ATTN_FLAG_LARGE_WG = 16
ATTN_FLAG_UNIFORM_SPLITS = 32
ATTN_FLAG_KEY_BLOCKS = 64
ATTN_FLAG_WIDE = 128
ATTN_KERNELS = ("generic", "f32", "tile", "wide", "key_blocks")   # by ETV_ATTN_KERNEL_*
MAX_TREE, ATTN_MAX_TREE = 256, 256
ATTN_STATIC_WORKSPACE_BYTES = 64 << 20

EXPORTS = ("etv_status_string", "etv_version", "etv_last_hip_error", "etv_build_tree_mask",
           "etv_tensorize_tree",
           "etv_tree_verify_attention_workspace_bytes", "etv_tree_verify_attention_plan", "etv_tree_verify_attention_kernel",
           "etv_tree_verify_attention", "etv_tree_verify_attention_static", "etv_safe_gather_paths",
           "etv_evaluate_posterior_workspace_bytes", "etv_evaluate_posterior", "etv_commit_accepted_kv",
           "etv_verify_epilogue", "etv_lm_head_argmax_workspace_bytes", "etv_lm_head_argmax",
           "etv_lm_head_packed_bytes", "etv_pack_lm_head", "etv_replicate_branches", "etv_commit_path_indices")


class AttnDesc(C.Structure):
    _fields_ = [(n, C.c_int32) for n in ("B", "T_max", "Hq", "Hkv", "d", "dtype", "block_size", "max_blocks",
                                         "num_blocks", "P_cap", "P_max")] + \
               [("scale", C.c_float), ("kv_split", C.c_int32), ("flags", C.c_int32)]


class AttnPlan(C.Structure):
    _fields_ = [(n, C.c_int32) for n in ("mfma", "wavefronts", "key_halves", "ring_stages", "row_groups", "kv_split",
                                         "n_splits", "balanced_splits")] + [("workgroups", C.c_int64)]


class CommitDesc(C.Structure):
    _fields_ = [(n, C.c_int32) for n in ("B", "T_max", "Hkv", "d", "elem_bytes", "n_layers", "W", "block_size",
                                         "max_blocks", "num_blocks", "P_cap", "reserved")] + \
               [("cache_layer_stride", C.c_int64)]


class CacheDesc(C.Structure):
    _fields_ = [(n, C.c_int32) for n in ("B", "Hkv", "d", "elem_bytes", "n_layers", "block_size", "max_blocks",
                                         "num_blocks", "P_cap", "reserved")] + [("cache_layer_stride", C.c_int64)]


class EtvError(RuntimeError):
    def __init__(self, fn: str, rc: int):
        l = lib()
        msg = l.etv_status_string(rc).decode()
        super().__init__(f"{fn}: {msg} (rc={rc}, hip={l.etv_last_hip_error()})")
        self.rc = rc


def lib():
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError(f"{LIB_PATH} is missing: build it with `python -m paper_2603_08088_amd.build` "
                               "(there is no fallback path)")
        l = C.CDLL(LIB_PATH)
        vp, i32, sz = C.c_void_p, C.c_int32, C.c_size_t
        l.etv_status_string.restype = C.c_char_p
        l.etv_status_string.argtypes = [i32]
        l.etv_version.restype = C.c_char_p
        l.etv_last_hip_error.restype = i32
        l.etv_build_tree_mask.restype = i32
        l.etv_build_tree_mask.argtypes = [vp, vp, i32, i32, vp, vp, vp, vp, vp]
        l.etv_tensorize_tree.restype = i32
        l.etv_tensorize_tree.argtypes = [vp, vp, vp, i32, i32, i32, i32, vp, vp, vp, vp, vp, vp, vp, vp]
        l.etv_tree_verify_attention_workspace_bytes.restype = sz
        l.etv_tree_verify_attention_workspace_bytes.argtypes = [C.POINTER(AttnDesc)]
        l.etv_tree_verify_attention_plan.restype = i32
        l.etv_tree_verify_attention_plan.argtypes = [C.POINTER(AttnDesc), C.POINTER(AttnPlan)]
        l.etv_tree_verify_attention_kernel.restype = i32
        l.etv_tree_verify_attention_kernel.argtypes = [C.POINTER(AttnDesc)]
        l.etv_tree_verify_attention.restype = i32
        l.etv_tree_verify_attention.argtypes = [C.POINTER(AttnDesc)] + [vp] * 12 + [sz, vp]
        l.etv_tree_verify_attention_static.restype = i32
        l.etv_tree_verify_attention_static.argtypes = [C.POINTER(AttnDesc)] + [vp] * 12
        l.etv_safe_gather_paths.restype = i32
        l.etv_safe_gather_paths.argtypes = [vp, vp, i32, i32, i32, i32, i32, vp, sz, vp, vp, vp, vp]
        l.etv_lm_head_argmax_workspace_bytes.restype = sz
        l.etv_lm_head_argmax_workspace_bytes.argtypes = [i32, i32, i32]
        l.etv_lm_head_argmax.restype = i32
        l.etv_lm_head_argmax.argtypes = [vp, vp, i32, vp, i32, i32, i32, i32, vp, vp, vp, sz, vp]
        l.etv_lm_head_packed_bytes.restype = sz
        l.etv_lm_head_packed_bytes.argtypes = [i32, i32]
        l.etv_pack_lm_head.restype = i32
        l.etv_pack_lm_head.argtypes = [vp, i32, i32, vp, vp]
        l.etv_verify_epilogue.restype = i32
        l.etv_verify_epilogue.argtypes = [C.POINTER(CommitDesc), vp, i32, vp, vp, i32, i32, vp, sz] + [vp] * 21 + [sz, vp]
        l.etv_evaluate_posterior_workspace_bytes.restype = sz
        l.etv_evaluate_posterior_workspace_bytes.argtypes = [i32, i32, i32]
        l.etv_evaluate_posterior.restype = i32
        l.etv_evaluate_posterior.argtypes = [vp] * 4 + [i32] * 6 + [vp] * 7 + [sz, vp]
        l.etv_commit_accepted_kv.restype = i32
        l.etv_commit_accepted_kv.argtypes = [C.POINTER(CommitDesc)] + [vp] * 14
        l.etv_replicate_branches.restype = i32
        l.etv_replicate_branches.argtypes = [C.POINTER(CacheDesc)] + [vp] * 5 + [i32, vp, i32] + [vp] * 5
        l.etv_commit_path_indices.restype = i32
        l.etv_commit_path_indices.argtypes = [C.POINTER(CacheDesc)] + [vp] * 7 + [i32, vp, vp, i32, vp, vp, vp]
        _lib = l
    return _lib


def _native():
    """The library's calls as a Python module: tensors (or None) where the C prototype has pointers, current stream."""
    global _calls
    if _calls is None:
        lib()
        try:
            from . import _binding
        except ImportError as e:
            raise RuntimeError(f"{_HERE}/_binding.so does not load ({e}): build it with `python -m paper_2603_08088_amd.build`")
        _calls = _binding
    return _calls


def _check(fn: str, rc: int):
    if rc != 0:
        raise EtvError(fn, rc)


def _dtype_code(t: torch.Tensor) -> int:
    if t.dtype == torch.float32:
        return F32
    if t.dtype == torch.bfloat16:
        return BF16
    raise EtvError("dtype", -2)


def _i32(shape, dev) -> torch.Tensor:
    return torch.empty(shape, dtype=torch.int32, device=dev)


# ------------------------------------------------------------------------------------------------
def build_tree_mask(parent: torch.Tensor, n_nodes: torch.Tensor, *, want_dense: bool = True,
                    want_depth: bool = True, out: Optional[Dict[str, torch.Tensor]] = None):
    """parent int32 [B,T_max], n_nodes int32 [B] -> bitmask u64-as-int64 [B,T_max,words], dense u8
    [B,1,T_max,T_max], depth int32 [B,T_max], status int32 [B]."""
    B, T = parent.shape
    dev = parent.device
    words = (T + 63) // 64
    o = out or {}
    bitmask = o.get("bitmask", None)
    if bitmask is None:
        bitmask = torch.empty((B, T, words), dtype=torch.int64, device=dev)
    dense = o.get("dense") if out else (torch.empty((B, 1, T, T), dtype=torch.uint8, device=dev) if want_dense else None)
    depth = o.get("depth") if out else (torch.empty((B, T), dtype=torch.int32, device=dev) if want_depth else None)
    status = o.get("status") if out else None
    if status is None:
        status = torch.empty((B,), dtype=torch.int32, device=dev)
    rc = _native().build_tree_mask(parent, n_nodes, B, T, bitmask, dense, depth, status)
    _check("etv_build_tree_mask", rc)
    return dict(bitmask=bitmask, dense=dense, depth=depth, status=status)


def tensorize_tree(parent: torch.Tensor, n_nodes: torch.Tensor, prefix_len: torch.Tensor, L_max: int, W: int, *,
                   want_dense: bool = True, out: Optional[Dict[str, torch.Tensor]] = None):
    """parent int32 [B,T_max], n_nodes, prefix_len int32 [B] -> the outputs of build_tree_mask plus position_ids
    int32 [B,T_max], retrieve int32 [B,L_max,W] (root-to-leaf paths, -1 padded) and n_paths int32 [B]."""
    B, T = parent.shape
    dev, get = parent.device, (out or {}).get
    bitmask, dense, depth, pos = get("bitmask"), get("dense"), get("depth"), get("position_ids")
    retrieve, n_paths, status = get("retrieve"), get("n_paths"), get("status")
    if bitmask is None:
        bitmask = torch.empty((B, T, (T + 63) // 64), dtype=torch.int64, device=dev)
    if not out and want_dense:
        dense = torch.empty((B, 1, T, T), dtype=torch.uint8, device=dev)
    if depth is None:
        depth = _i32((B, T), dev)
    if pos is None:
        pos = _i32((B, T), dev)
    if retrieve is None:
        retrieve = _i32((B, L_max, W), dev)
    if n_paths is None:
        n_paths = _i32((B,), dev)
    if status is None:
        status = _i32((B,), dev)
    rc = _native().tensorize_tree(parent, n_nodes, prefix_len, B, T, L_max, W, bitmask, dense, depth, pos, retrieve, n_paths,
                                   status)
    _check("etv_tensorize_tree", rc)
    return dict(bitmask=bitmask, dense=dense, depth=depth, position_ids=pos, retrieve=retrieve, n_paths=n_paths,
                status=status)


def attn_desc(q: torch.Tensor, kt: torch.Tensor, k_cache: Optional[torch.Tensor], block_table: Optional[torch.Tensor],
              P_max: int, scale: float = 0.0, kv_split: int = 0, flags: int = 0) -> AttnDesc:
    B, T, Hq, d = q.shape
    # kt None: in-place branch cache, the tree rows are in k_cache / v_cache behind the prefix
    Hkv = kt.shape[2] if kt is not None else (k_cache.shape[1] if block_table is not None else k_cache.shape[2])
    dsc = AttnDesc(B=B, T_max=T, Hq=Hq, Hkv=Hkv, d=d, dtype=_dtype_code(q), block_size=0, max_blocks=0,
                   num_blocks=0, P_cap=0, P_max=int(P_max), scale=float(scale), kv_split=int(kv_split),
                   flags=int(flags))
    if block_table is not None:
        dsc.block_size = k_cache.shape[2]
        dsc.max_blocks = block_table.shape[1]
        dsc.num_blocks = k_cache.shape[0]
    elif k_cache is not None:
        dsc.P_cap = k_cache.shape[1]
    return dsc


def _attn_desc_only(dsc):
    """The binding takes any object with the memory of a descriptor: a caller's own is checked here."""
    if not isinstance(dsc, AttnDesc):
        raise C.ArgumentError("expected AttnDesc instead of " + type(dsc).__name__)
    return dsc


def tree_verify_attention_workspace_bytes(dsc: AttnDesc) -> int:
    return int(lib().etv_tree_verify_attention_workspace_bytes(C.byref(dsc)))


def tree_verify_attention_plan(dsc: AttnDesc) -> Dict[str, int]:
    """The launch shape the library picks for this descriptor (host only)."""
    pl = AttnPlan()
    _check("etv_tree_verify_attention_plan", lib().etv_tree_verify_attention_plan(C.byref(dsc), C.byref(pl)))
    return {n: int(getattr(pl, n)) for n, _ in AttnPlan._fields_ if n != "reserved"}


def tree_verify_attention_kernel(dsc: AttnDesc) -> str:
    """Which of ATTN_KERNELS the library picks for this descriptor (host only)."""
    rc = lib().etv_tree_verify_attention_kernel(C.byref(dsc))
    _check("etv_tree_verify_attention_kernel", min(rc, 0))
    return ATTN_KERNELS[rc]


def tree_verify_attention(q, k_cache, v_cache, prefix_len, kt, vt, bitmask, n_nodes, *, P_max: int,
                          block_table=None, scale: float = 0.0, kv_split: int = 0, flags: int = 0,
                          out=None, lse=None, want_lse: bool = True, workspace=None, desc: Optional[AttnDesc] = None):
    """q [B,T,Hq,d]; kt/vt [B,T,Hkv,d]; cache contiguous [B,P_cap,Hkv,d] or paged [nb,Hkv,16,d] + block_table.
    Returns (out [B,T,Hq,d] in q's dtype, lse float32 [B,Hq,T] or None)."""
    dsc = _attn_desc_only(desc or attn_desc(q, kt, k_cache, block_table, P_max, scale, kv_split, flags))
    if q.dim() != 4:
        raise ValueError("q is [B, T, Hq, d]")
    if out is None:
        out = torch.empty_like(q)
    if lse is None and want_lse:
        B, T, Hq, _ = q.shape
        lse = torch.empty((B, Hq, T), dtype=torch.float32, device=q.device)
    if workspace is None:
        workspace = torch.empty((max(256, tree_verify_attention_workspace_bytes(dsc)),), dtype=torch.uint8,
                                device=q.device)
    rc = _native().tree_verify_attention(dsc, q, k_cache, v_cache, block_table, prefix_len, kt, vt, bitmask,
                                         n_nodes, out, lse, workspace, workspace.numel())
    _check("etv_tree_verify_attention", rc)
    return out, lse


def tree_verify_attention_static(q, k_cache, v_cache, prefix_len, kt, vt, bitmask, n_nodes, out, lse=None, *,
                                 P_max: int, block_table=None, scale: float = 0.0, kv_split: int = 0, flags: int = 0,
                                 desc: Optional[AttnDesc] = None):
    """tree_verify_attention with the split partials in the library's own fixed device array: the caller passes
    every input and output (`out`, optionally `lse`) and nothing is allocated, here or in the library."""
    dsc = desc or attn_desc(q, kt, k_cache, block_table, P_max, scale, kv_split, flags)
    rc = _native().tree_verify_attention_static(_attn_desc_only(dsc), q, k_cache, v_cache, block_table, prefix_len, kt, vt,
                                                bitmask, n_nodes, out, lse)
    _check("etv_tree_verify_attention_static", rc)
    return out, lse


def safe_gather_paths(retrieve, n_nodes, T_max: int, dummy: int = 0, src: Optional[torch.Tensor] = None,
                      out: Optional[Dict[str, torch.Tensor]] = None):
    """retrieve int32 [B,L,W]; src [B,T_max,...] any dtype -> safe int32, pvalid u8, gathered [B,L,W,...]."""
    B, L, W = retrieve.shape
    dev = retrieve.device
    o = out or {}
    safe = o.get("safe") if out else torch.empty((B, L, W), dtype=torch.int32, device=dev)
    pvalid = o.get("pvalid") if out else torch.empty((B, L, W), dtype=torch.uint8, device=dev)
    gathered, row_bytes = None, 0
    if src is not None:
        assert src.shape[0] == B and src.shape[1] == T_max
        row_bytes = src.element_size() * (src.numel() // max(1, B * T_max))
        gathered = o.get("gathered") if out else None
        if gathered is None:
            gathered = torch.empty((B, L, W) + tuple(src.shape[2:]), dtype=src.dtype, device=dev)
    rc = _native().safe_gather_paths(retrieve, n_nodes, B, L, W, T_max, dummy, src, row_bytes, safe, pvalid, gathered)
    _check("etv_safe_gather_paths", rc)
    return dict(safe=safe, pvalid=pvalid, gathered=gathered)


def evaluate_posterior_workspace_bytes(B: int, T_max: int, V: int) -> int:
    return int(lib().etv_evaluate_posterior_workspace_bytes(B, T_max, V))


def evaluate_posterior(logits, tokens, retrieve, n_nodes, dummy: int = 0, workspace=None,
                       out: Optional[Dict[str, torch.Tensor]] = None, head_V: int = 0):
    """logits f32 [B,T,V]; tokens int32 [B,T]; retrieve int32 [B,L,W] -> argmax, len, best, accept_len,
    acc_nodes, bonus (all int32).  With logits=None, out["argmax"] is an input (e.g. from lm_head_argmax), or,
    with head_V > 0, `workspace` is the one lm_head_argmax(..., finish=False) returned for that vocabulary size."""
    if logits is None:
        (B, T), V = tokens.shape, int(head_V)
        assert workspace is not None if V else (out is not None and out.get("argmax") is not None)
    else:
        B, T, V = logits.shape
    _, L, W = retrieve.shape
    dev = tokens.device
    o = out or {}
    i32 = dict(dtype=torch.int32, device=dev)
    def get(name, shape):
        t = o.get(name)
        return t if t is not None else torch.empty(shape, **i32)
    g, ln, best = get("argmax", (B, T)), get("len", (B, L)), get("best", (B,))
    A, acc, bonus = get("accept_len", (B,)), get("acc_nodes", (B, W)), get("bonus", (B,))
    if workspace is None and logits is not None:
        workspace = torch.empty((max(256, evaluate_posterior_workspace_bytes(B, T, V)),), dtype=torch.uint8, device=dev)
    rc = _native().evaluate_posterior(logits, tokens, retrieve, n_nodes, B, T, V, L, W, dummy, g, ln, best, A, acc, bonus,
                                      workspace, workspace.numel() if workspace is not None else 0)
    _check("etv_evaluate_posterior", rc)
    return dict(argmax=g, len=ln, best=best, accept_len=A, acc_nodes=acc, bonus=bonus)


def pack_lm_head(weight: torch.Tensor) -> torch.Tensor:
    """weight bf16 [V,D] -> the same weights in the tile order lm_head_argmax streams fastest (flat bf16 tensor)."""
    V, D = weight.shape
    n = int(lib().etv_lm_head_packed_bytes(V, D))
    if n == 0:
        raise EtvError("etv_lm_head_packed_bytes", -2)
    packed = torch.empty((n // 2,), dtype=weight.dtype, device=weight.device)
    _check("etv_pack_lm_head", _native().pack_lm_head(weight, V, D, packed))
    return packed


def lm_head_argmax(hidden, weight, n_nodes, *, V: Optional[int] = None, want_max: bool = True, workspace=None,
                   out: Optional[Dict[str, torch.Tensor]] = None, finish: bool = True):
    """hidden bf16 [B,T,D]; weight bf16 [V,D], or the flat tensor of pack_lm_head together with V
    -> argmax int32 [B,T] (-1 for padding), maxval float32 [B,T].  finish=False stops after the weight pass and
    returns the workspace, to be handed to evaluate_posterior / verify_epilogue with head_V=V."""
    B, T, D = hidden.shape
    packed = weight.dim() == 1
    if not packed:
        V = weight.shape[0]
    assert V is not None
    dev = hidden.device
    o = out or {}
    g = o.get("argmax")
    if g is None:
        g = torch.empty((B, T), dtype=torch.int32, device=dev)
    mx = o.get("maxval") if out else (torch.empty((B, T), dtype=torch.float32, device=dev) if want_max else None)
    if workspace is None:
        workspace = torch.empty((max(256, int(lib().etv_lm_head_argmax_workspace_bytes(B, T, V))),), dtype=torch.uint8,
                                device=dev)
    rc = _native().lm_head_argmax(hidden, weight, int(packed), n_nodes, B, T, D, V, g if finish else None,
                                  mx if finish else None, workspace, workspace.numel())
    _check("etv_lm_head_argmax", rc)
    return dict(argmax=g, maxval=mx) if finish else dict(workspace=workspace)


def _commit_desc(kt, k_cache, block_table, W: int, B: Optional[int] = None, T_max: Optional[int] = None):
    """The memory of a CommitDesc, from the binding where the shapes are in order."""
    dsc = _native().commit_desc(kt, k_cache, block_table, W)
    if dsc is not None:
        return dsc
    if kt is not None:
        Lyr, B, T, Hkv, d = kt.shape
    else:   # in-place branch cache: shapes from the cache, B and T_max from the caller
        Lyr, T = k_cache.shape[0], int(T_max)
        Hkv, d = (k_cache.shape[2], k_cache.shape[4]) if block_table is not None else (k_cache.shape[3], k_cache.shape[4])
    assert k_cache.shape[0] == Lyr
    stride = k_cache.stride(0) if Lyr > 1 else k_cache.numel()
    elem = k_cache.element_size()
    # positional, in the order of CommitDesc: B ... W, block_size, max_blocks, num_blocks, P_cap, reserved, cache_layer_stride
    if block_table is not None:
        return CommitDesc(B, T, Hkv, d, elem, Lyr, W, k_cache.shape[3], block_table.shape[1], k_cache.shape[1], 0, 0, stride)
    return CommitDesc(B, T, Hkv, d, elem, Lyr, W, 0, 0, 0, k_cache.shape[2], 0, stride)


def verify_epilogue(logits, tokens, retrieve, n_nodes, kt, vt, k_cache, v_cache, prefix_len, capacity, *,
                    block_table=None, dummy: int = 0, src: Optional[torch.Tensor] = None, workspace=None,
                    gather_out: Optional[Dict[str, torch.Tensor]] = None,
                    post_out: Optional[Dict[str, torch.Tensor]] = None,
                    commit_out: Optional[Dict[str, torch.Tensor]] = None, head_V: int = 0):
    """safe_gather_paths + evaluate_posterior + commit_accepted_kv in one to three launches; same tensors and results.
    With logits=None, post_out["argmax"] is an input, or, with head_V > 0, `workspace` is the one
    lm_head_argmax(..., finish=False) returned.  Returns (gather dict, posterior dict, commit dict)."""
    if logits is None:
        (B, T), V = tokens.shape, int(head_V)
        assert workspace is not None if V else (post_out is not None and post_out.get("argmax") is not None)
    else:
        B, T, V = logits.shape
    # Written out: one call of a step of some 20 us, and a closure, a shape and a look-up per output took a third of it.
    _, L, W = retrieve.shape
    dev = tokens.device
    go, po, co = (gather_out or {}).get, (post_out or {}).get, (commit_out or {}).get
    safe, pvalid, gathered, row_bytes = go("safe"), go("pvalid"), None, 0
    if safe is None:
        safe = _i32((B, L, W), dev)
    if pvalid is None:
        pvalid = torch.empty((B, L, W), dtype=torch.uint8, device=dev)
    if src is not None:
        rows = src.shape
        if rows[0] == 0 or rows[1] == 0:
            raise IndexError("src has no row")
        row_bytes = src.element_size() * (src.numel() // (rows[0] * rows[1]))
        gathered = go("gathered")
        if gathered is None:
            gathered = torch.empty((B, L, W) + tuple(rows[2:]), dtype=src.dtype, device=dev)
    g, ln, best, A, acc, bonus = po("argmax"), po("len"), po("best"), po("accept_len"), po("acc_nodes"), po("bonus")
    if g is None:
        g = _i32((B, T), dev)
    if ln is None:
        ln = _i32((B, L), dev)
    if best is None:
        best = _i32((B,), dev)
    if A is None:
        A = _i32((B,), dev)
    if acc is None:
        acc = _i32((B, W), dev)
    if bonus is None:
        bonus = _i32((B,), dev)
    plo, slot, status = co("prefix_len_out"), co("slot_map"), co("status")
    if plo is None:
        plo = _i32((B,), dev)
    if slot is None:
        slot = _i32((B, W), dev)
    if status is None:
        status = _i32((B,), dev)
    if workspace is None and logits is not None:
        workspace = torch.empty((max(256, evaluate_posterior_workspace_bytes(B, T, V)),), dtype=torch.uint8, device=dev)
    dsc = _commit_desc(kt, k_cache, block_table, W, B, T)
    rc = _native().verify_epilogue(dsc, logits, V, tokens, retrieve, L, dummy, src, row_bytes, safe, pvalid, gathered, g, ln,
                                   best, A, acc, bonus, kt, vt, k_cache, v_cache, block_table, prefix_len, capacity, n_nodes,
                                   plo, slot, status, workspace, workspace.numel() if workspace is not None else 0)
    _check("etv_verify_epilogue", rc)
    return (dict(safe=safe, pvalid=pvalid, gathered=gathered),
            dict(argmax=g, len=ln, best=best, accept_len=A, acc_nodes=acc, bonus=bonus),
            dict(prefix_len_out=plo, slot_map=slot, status=status))


def commit_accepted_kv(kt, vt, k_cache, v_cache, prefix_len, capacity, n_nodes, acc_nodes, accept_len, *,
                       block_table=None, prefix_len_out=None, out: Optional[Dict[str, torch.Tensor]] = None,
                       T_max: Optional[int] = None):
    """kt/vt [Lyr,B,T,Hkv,d]; caches [Lyr,B,P_cap,Hkv,d] or [Lyr,nb,Hkv,bs,d] updated in place.
    kt = vt = None (with T_max): in-place branch cache, the tree rows are in the caches behind the prefix.
    Returns prefix_len_out, slot_map, status."""
    B, W = acc_nodes.shape
    dev = k_cache.device
    dsc = _commit_desc(kt, k_cache, block_table, W, B, T_max)
    o = out or {}
    if prefix_len_out is None:
        prefix_len_out = o.get("prefix_len_out")
    if prefix_len_out is None:
        prefix_len_out = torch.empty((B,), dtype=torch.int32, device=dev)
    slot = o.get("slot_map") if out else torch.empty((B, W), dtype=torch.int32, device=dev)
    status = o.get("status") if out else torch.empty((B,), dtype=torch.int32, device=dev)
    rc = _native().commit_accepted_kv(dsc, kt, vt, k_cache, v_cache, block_table, prefix_len, capacity, n_nodes,
                                      acc_nodes, accept_len, prefix_len_out, slot, status)
    _check("etv_commit_accepted_kv", rc)
    return dict(prefix_len_out=prefix_len_out, slot_map=slot, status=status)


def _cache_desc(cache: torch.Tensor, B: int, table: Optional[torch.Tensor]) -> CacheDesc:
    Lyr, n1, n2, n3, d = cache.shape
    stride = cache.stride(0) if Lyr > 1 else cache.numel()
    # positional, in the order of CacheDesc: B, Hkv, d, elem_bytes, n_layers, block_size, max_blocks, num_blocks, P_cap, reserved
    if table is not None:   # [Lyr, num_blocks, Hkv, block_size, d]
        return CacheDesc(B, n2, d, cache.element_size(), Lyr, n3, table.shape[-1], n1, 0, 0, stride)
    return CacheDesc(B, n3, d, cache.element_size(), Lyr, 0, 0, 0, n2, 0, stride)


def replicate_branches(k_cache, v_cache, block_table, prefix_len, tail_len, N: int, free_blocks):
    """Paged caches [Lyr, nb, Hkv, bs, d]; block_table [B, max_blocks]; free_blocks int32 [n_free].
    Returns branch_table [B, N, max_blocks], block_base [B], n_taken [1], status [B] (device tensors)."""
    B = block_table.shape[0]
    dsc = _cache_desc(k_cache, B, block_table)
    empty = _native().empty_i32
    bt, base = empty(k_cache, B, N, block_table.shape[1]), empty(k_cache, B)
    taken, status = empty(k_cache, 1), empty(k_cache, B)
    rc = _native().replicate_branches(dsc, k_cache, v_cache, block_table, prefix_len, tail_len, N, free_blocks,
                                      free_blocks.numel(), bt, base, taken, status)
    _check("etv_replicate_branches", rc)
    return dict(branch_table=bt, block_base=base, n_taken=taken, status=status)


def commit_path_indices(src_k, src_v, dst_k, dst_v, path_indices, src_len, new_len, *, src_table=None, dst_table=None,
                        fast: bool = False):
    """Caches [Lyr, B, P_cap, Hkv, d] (two buffers) or [Lyr, nb, Hkv, bs, d] with two block tables (dst_table is
    updated in place with the shared blocks).  Returns kept_len, status."""
    B, L_cap = path_indices.shape
    dsc = _cache_desc(src_k, B, src_table)
    kept, status = _native().empty_i32(src_k, B), _native().empty_i32(src_k, B)
    rc = _native().commit_path_indices(dsc, src_k, src_v, dst_k, dst_v, src_table, dst_table, path_indices, L_cap,
                                       src_len, new_len, int(fast), kept, status)
    _check("etv_commit_path_indices", rc)
    return dict(kept_len=kept, status=status)
