"""Thin binding of libsage_hip.so (include/sage.h): same names, argument marshalling only.

Tensors are torch CUDA(HIP) tensors used as device buffers; nothing here computes anything.  The library is
loaded on first use and a missing library is an error (there is no fallback path of any kind).
"""
from __future__ import annotations

import ctypes
import inspect
import os

import torch  # noqa: F401  (its libraries have to be loaded before the binding's)

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.environ.get("SAGE_HIP_LIBRARY") or os.path.join(_HERE, "libsage_hip.so")   # the in-tree build unless told otherwise
BINDING_PATH = os.path.join(_HERE, "_binding.so")           # argument marshalling in native code (csrc/python_binding.cpp)
MAX_NODES = 64
F32, BF16 = 0, 1
STATUS = {0: "OK", 1: "INVALID_ARG", 2: "UNSUPPORTED", 3: "WORKSPACE_TOO_SMALL", 4: "LAUNCH_FAILED"}


class SageError(RuntimeError):
    def __init__(self, call: str, code: int):
        super().__init__(f"{call} -> {STATUS.get(code, code)}")
        self.code = code


class TreeParams(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("d_min", "d_max", "w_min", "w_max", "k", "n_max")]


_lib = None
_vp, _ci, _cl, _cf, _sz = ctypes.c_void_p, ctypes.c_int, ctypes.c_long, ctypes.c_float, ctypes.c_size_t


def lib():
    """Load the HIP library built in-tree by paper_2602_00523_amd.build; fail loudly when it is absent."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise SageError(f"{LIB_PATH} is missing: run `python -m paper_2602_00523_amd.build`", -1)
        L = ctypes.CDLL(LIB_PATH)
        L.sage_entropy_topk_workspace_bytes.restype = _sz
        L.sage_entropy_topk_workspace_bytes.argtypes = [_ci, _ci, _ci]
        L.sage_entropy_topk.restype = _ci
        L.sage_entropy_topk.argtypes = [_vp, _ci, _ci, _ci, _cl, _ci, _vp, _ci, _vp, _vp, _vp, _vp, _vp, _vp, _vp, _sz, _vp]
        L.sage_build_tree.restype = _ci
        L.sage_build_tree.argtypes = [_vp, _vp, _vp, _ci, _ci, ctypes.POINTER(TreeParams), _vp, _vp, _vp, _vp, _vp, _vp,
                                      _vp, _vp, _vp]
        L.sage_tree_attention_workspace_bytes.restype = _sz
        L.sage_tree_attention_workspace_bytes.argtypes = [_ci, _ci, _ci, _ci, _ci, _ci]
        L.sage_tree_attention.restype = _ci
        L.sage_tree_attention.argtypes = [_vp, _vp, _vp, _vp, _vp, _vp, _ci, _ci, _ci, _ci, _ci, _vp, _vp, _ci, _cl, _cl,
                                          _vp, _vp, _vp, _cf, _vp, _sz, _vp]
        L.sage_tree_attention_static_scratch_bytes.restype = _sz
        L.sage_tree_attention_static_scratch_bytes.argtypes = []
        L.sage_tree_attention_static.restype = _ci
        L.sage_tree_attention_static.argtypes = [_vp, _vp, _vp, _vp, _vp, _vp, _ci, _ci, _ci, _ci, _ci, _vp, _vp, _ci, _cl, _cl,
                                                 _vp, _vp, _cf, _vp]
        L.sage_tree_attention_with_plan.restype = _ci
        L.sage_tree_attention_with_plan.argtypes = (
            [_vp, _vp, _vp, _vp, _vp, _vp, _ci, _ci, _ci, _ci, _ci, _vp, _vp, _ci, _cl, _cl, _vp, _vp, _cf, _vp, _sz]
            + [_vp, _ci, _ci, ctypes.POINTER(TreeParams)] + [_vp] * 15)
        L.sage_verify_accept.restype = _ci
        L.sage_verify_accept.argtypes = [_vp, _vp, _vp, _vp, _vp, _vp, _ci, _ci, _vp, _vp, _vp, _vp, _vp]
        L.sage_commit_path.restype = _ci
        L.sage_commit_path.argtypes = [_vp, _vp, _vp, _vp, _ci, _ci, _ci, _ci, _vp, _vp, _ci, _cl, _cl, _vp, _vp, _ci, _vp]
        L.sage_advance_kv_len.restype = _ci
        L.sage_advance_kv_len.argtypes = [_vp, _vp, _ci, _ci, _vp]
        L.sage_update_history.restype = _ci
        L.sage_update_history.argtypes = [_vp, _ci, _ci, _cf, _cf, _ci, _ci, _vp, _vp, _vp, _vp, _vp]
        L.sage_lm_head_topk_workspace_bytes.restype = _sz
        L.sage_verify_accept_close_from_slices.restype = _ci
        L.sage_verify_accept_close_from_slices.argtypes = (
            [_vp, _ci, _vp, _vp, _vp, _vp, _vp, _ci, _ci] + [_vp] * 6 + [_vp, _vp, _vp, _vp, _ci, _ci, _ci, _vp, _vp, _ci, _cl, _cl,
                                                                       _ci, _cf, _cf, _ci, _ci, _vp, _vp, _vp, _vp, _vp, _vp])
        L.sage_close_step.restype = _ci
        L.sage_close_step.argtypes = [_vp, _vp, _vp, _vp, _ci, _ci, _ci, _ci, _vp, _vp, _ci, _cl, _cl, _vp, _vp, _ci, _ci, _cf, _cf,
                                      _ci, _ci, _vp, _vp, _vp, _vp, _vp, _vp]
        L.sage_entropy_topk_slices.restype = _ci
        L.sage_entropy_topk_slices.argtypes = [_vp, _ci, _ci, _ci, _cl, _ci, _vp, _ci, _vp, _sz, _vp]
        L.sage_entropy_topk_slices_pair.restype = _ci
        L.sage_entropy_topk_slices_pair.argtypes = [_vp, _ci, _cl, _vp, _ci, _vp, _sz, _vp, _ci, _cl, _ci, _vp, _sz, _ci, _ci, _vp]
        L.sage_build_tree_from_slices.restype = _ci
        L.sage_build_tree_from_slices.argtypes = [_vp, _ci, _ci, _ci, ctypes.POINTER(TreeParams)] + [_vp] * 15
        L.sage_verify_accept_from_slices.restype = _ci
        L.sage_verify_accept_from_slices.argtypes = [_vp, _ci, _vp, _vp, _vp, _vp, _vp, _ci, _ci] + [_vp] * 7
        L.sage_lm_head_topk_workspace_bytes.argtypes = [_ci, _ci, _ci]
        L.sage_lm_head_topk.restype = _ci
        L.sage_lm_head_topk.argtypes = [_vp, _vp, _ci, _ci, _ci, _ci, _cl, _cl, _ci, _vp, _ci, _vp, _vp, _vp, _vp, _vp, _vp,
                                        _vp, _sz, _vp]
        L.sage_build_info.restype = ctypes.c_char_p
        _lib = L
    return _lib


def tree_params(d_min, d_max, w_min, w_max, k, n_max) -> TreeParams:
    return TreeParams(d_min, d_max, w_min, w_max, k, n_max)


def sage_entropy_topk_workspace_bytes(rows: int, vocab: int, k: int) -> int:
    return int(lib().sage_entropy_topk_workspace_bytes(rows, vocab, k))


def sage_lm_head_topk_workspace_bytes(rows: int, vocab: int, k: int = 1) -> int:
    return int(lib().sage_lm_head_topk_workspace_bytes(rows, vocab, k))


def sage_tree_attention_workspace_bytes(dtype_code: int, B: int, Hq: int, Hkv: int, d: int, max_kv_len: int) -> int:
    return int(lib().sage_tree_attention_workspace_bytes(dtype_code, B, Hq, Hkv, d, max_kv_len))


# ---- the calls: Python parameters, and where each C argument comes from ------------------------------------
# Items of the second string, one per C argument in the order of include/sage.h: ptr (a tensor's address; None = null),
# nbytes, dtype (float32 / bfloat16), sizeN / strideN of a tensor, int, float, struct, stream (None = the current one);
# dimN, unitN, sameN and sametype only check.  csrc/python_binding.cpp turns them into native calls.

_ATT = "Q Kc Vc Kt Vt O kv_start kv_len max_kv_len kv_token_stride kv_head_stride anc_mask n_nodes scale"
_ATT_HEAD = ("dim4:Q ptr:Q ptr:Kc ptr:Vc ptr:Kt ptr:Vt ptr:O dtype:Q size0:Q size2:Q size2:Kt size3:Q ptr:kv_start ptr:kv_len "
             "int:max_kv_len int:kv_token_stride int:kv_head_stride ptr:anc_mask ptr:n_nodes ")
_ROW = "entropy topk_idx topk_prob topk_renorm topk_entropy alpha"
_ROW_PTRS = " ".join(f"ptr:{n}" for n in _ROW.split()) + " "
_TREE = "n_nodes parent depth rank anc_mask cum_prob=None"
_TREE_PTRS = "ptr:n_nodes ptr:parent ptr:depth ptr:rank ptr:anc_mask ptr:cum_prob ptr:node_token "
_CACHE = "Kt Vt Kc Vc kv_start kv_len kv_capacity kv_token_stride kv_head_stride"
_CACHE_PTRS = "ptr:Kt ptr:Vt ptr:Kc ptr:Vc dtype:Kt "
_CACHE_POS = "ptr:kv_start ptr:kv_len int:kv_capacity int:kv_token_stride int:kv_head_stride "
_ACC_PTRS = "ptr:accept_len ptr:best_node ptr:path_nodes ptr:out_tokens "
_SLICES_VERIFY = ("slices vocab token parent depth anc_mask n_nodes path_cap entropy target_argmax accept_len best_node path_nodes "
                  "out_tokens")
_SLICES_VERIFY_PTRS = ("ptr:slices int:vocab ptr:token ptr:parent ptr:depth ptr:anc_mask ptr:n_nodes size0:n_nodes int:path_cap "
                       "ptr:entropy ptr:target_argmax " + _ACC_PTRS)
_HISTORY_TAIL = "ptr:hist ptr:count ptr:d_max_in ptr:d_max_out ptr:avg_out stream:stream"
_LOGITS = "dim2:logits unit1:logits ptr:logits dtype:logits size0:logits size1:logits stride0:logits int:k "

_CALLS = {
    "sage_entropy_topk": (
        f"logits k {_ROW} workspace n_valid=None rows_per_group=1 stream=None",
        _LOGITS + "ptr:n_valid int:rows_per_group " + _ROW_PTRS + "ptr:workspace nbytes:workspace stream:stream"),
    "sage_entropy_topk_slices": (
        "logits k workspace n_valid=None rows_per_group=1 stream=None",
        _LOGITS + "ptr:n_valid int:rows_per_group ptr:workspace nbytes:workspace stream:stream"),
    "sage_entropy_topk_slices_pair": (
        "logits_a n_valid_a rows_per_group_a workspace_a logits_b k_b workspace_b stream=None",
        "dim2:logits_a dim2:logits_b same1:logits_a,logits_b sametype:logits_a,logits_b unit1:logits_a unit1:logits_b "
        "ptr:logits_a size0:logits_a stride0:logits_a ptr:n_valid_a int:rows_per_group_a ptr:workspace_a nbytes:workspace_a "
        "ptr:logits_b size0:logits_b stride0:logits_b int:k_b ptr:workspace_b nbytes:workspace_b dtype:logits_a size1:logits_a "
        "stream:stream"),
    "sage_build_tree": (
        f"topk_renorm alpha params {_TREE} topk_idx=None node_token=None stream=None d_max_seq=None",
        "dim2:topk_renorm ptr:topk_renorm ptr:alpha ptr:topk_idx size0:topk_renorm size1:topk_renorm struct:params ptr:d_max_seq "
        + _TREE_PTRS + "stream:stream"),
    "sage_build_tree_from_slices": (
        f"slices vocab params {_ROW} {_TREE} node_token=None stream=None d_max_seq=None",
        "dim2:topk_idx ptr:slices int:vocab size0:topk_idx size1:topk_idx struct:params ptr:d_max_seq " + _ROW_PTRS + _TREE_PTRS
        + "stream:stream"),
    "sage_tree_attention": (
        f"{_ATT} workspace stream=None first_node=None",
        _ATT_HEAD + "ptr:first_node float:scale ptr:workspace nbytes:workspace stream:stream"),
    "sage_tree_attention_static": (f"{_ATT} stream=None", _ATT_HEAD + "float:scale stream:stream"),
    "sage_tree_attention_with_plan": (                     # one draft row per sequence: the batch size travels once
        f"{_ATT} workspace slices vocab params {_ROW} next_n_nodes next_parent next_depth next_rank next_anc_mask next_cum_prob=None "
        "next_node_token=None stream=None d_max_seq=None",
        _ATT_HEAD + "float:scale ptr:workspace nbytes:workspace dim2:topk_idx same0:Q,topk_idx ptr:slices int:vocab size1:topk_idx "
        "struct:params ptr:d_max_seq " + _ROW_PTRS + "ptr:next_n_nodes ptr:next_parent ptr:next_depth ptr:next_rank "
        "ptr:next_anc_mask ptr:next_cum_prob ptr:next_node_token stream:stream"),
    "sage_verify_accept": (
        "token target_argmax parent depth anc_mask n_nodes path_cap accept_len best_node path_nodes out_tokens stream=None",
        "ptr:token ptr:target_argmax ptr:parent ptr:depth ptr:anc_mask ptr:n_nodes size0:n_nodes int:path_cap " + _ACC_PTRS
        + "stream:stream"),
    "sage_verify_accept_from_slices": (f"{_SLICES_VERIFY} stream=None", _SLICES_VERIFY_PTRS + "stream:stream"),
    "sage_verify_accept_close_from_slices": (
        f"{_SLICES_VERIFY} {_CACHE} hist count d_max_in d_max_out lo hi d_floor d_cap avg_out=None stream=None",
        _SLICES_VERIFY_PTRS + "dim4:Kt " + _CACHE_PTRS + "size2:Kt size3:Kt " + _CACHE_POS
        + "size1:hist float:lo float:hi int:d_floor int:d_cap " + _HISTORY_TAIL),
    "sage_commit_path": (
        f"{_CACHE} path_nodes accept_len stream=None",
        "dim4:Kt " + _CACHE_PTRS + "size0:Kt size2:Kt size3:Kt " + _CACHE_POS + "ptr:path_nodes ptr:accept_len size1:path_nodes "
        "stream:stream"),
    "sage_advance_kv_len": (
        "kv_len accept_len kv_capacity stream=None",
        "ptr:kv_len ptr:accept_len size0:kv_len int:kv_capacity stream:stream"),
    "sage_update_history": (
        "accept_len hist count d_max lo hi d_floor d_cap avg_out=None stream=None",
        "dim2:hist ptr:accept_len size0:hist size1:hist float:lo float:hi int:d_floor int:d_cap ptr:hist ptr:count ptr:d_max "
        "ptr:avg_out stream:stream"),
    "sage_close_step": (
        f"{_CACHE} path_nodes accept_len hist count d_max_in d_max_out lo hi d_floor d_cap avg_out=None stream=None",
        "dim4:Kt " + _CACHE_PTRS + "size0:Kt size2:Kt size3:Kt " + _CACHE_POS + "ptr:path_nodes ptr:accept_len "
        "size1:path_nodes size1:hist float:lo float:hi int:d_floor int:d_cap " + _HISTORY_TAIL),
    "sage_lm_head_topk": (
        f"hidden weight k {_ROW} workspace n_valid=None rows_per_group=1 stream=None",
        "dim2:hidden ptr:hidden ptr:weight dtype:hidden size0:hidden size1:hidden size0:weight stride0:hidden stride0:weight int:k "
        "ptr:n_valid int:rows_per_group " + _ROW_PTRS + "ptr:workspace nbytes:workspace stream:stream"),
}

_native = {}


def _doc(name: str) -> str:
    return f"{name}({', '.join(_CALLS[name][0].split())}): see include/sage.h"


def _signature(name: str) -> inspect.Signature:
    def parameter(word: str) -> inspect.Parameter:
        n, _, default = word.partition("=")
        default = inspect.Parameter.empty if not default else None if default == "None" else int(default)
        return inspect.Parameter(n, inspect.Parameter.POSITIONAL_OR_KEYWORD, default=default)
    return inspect.Signature([parameter(w) for w in _CALLS[name][0].split()])


def _load_native(name: str):
    """The native call `name` (all of them are made on first use, then stand in this module under their own names)."""
    if not _native:
        if not os.path.exists(BINDING_PATH):
            raise SageError(f"{BINDING_PATH} is missing: run `python -m paper_2602_00523_amd.build`", -1)
        from . import _binding
        L = lib()
        made = {n: _binding.make(n, ctypes.cast(getattr(L, n), ctypes.c_void_p).value, params, args, SageError, __name__, _doc(n), _signature(n))
                for n, (params, args) in _CALLS.items()}
        # (a name that the program has given to something else in the meantime, a wrapper say, stays with that)
        globals().update({n: call for n, call in made.items() if globals().get(n) is _first[n]})
        _native.update(made)
    return _native[name]


def _first_use(name: str):
    def call(*a, **kw):
        return _load_native(name)(*a, **kw)
    call.__name__ = call.__qualname__ = name
    call.__doc__ = _doc(name)
    call.__signature__ = _signature(name)
    return call


_first = {_name: _first_use(_name) for _name in _CALLS}
globals().update(_first)


def sage_tree_attention_static_scratch_bytes() -> int:
    return int(lib().sage_tree_attention_static_scratch_bytes())


def prepare(name: str, *a, **kw):
    """Marshal the arguments of call `name` once and return a zero-argument callable that enqueues it.

    For loops that issue the same call on the same buffers and stream many times: what is left per call is the launch.
    The callable keeps its arguments alive.
    """
    if name not in _CALLS:
        raise AttributeError(f"the library has no call {name!r}")
    return _load_native(name).bind(*a, **kw)


def sage_build_info() -> str:
    return lib().sage_build_info().decode()
