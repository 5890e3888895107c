"""Thin Python binding of the C ABI in include/vlut.h (argument marshalling only).

Device buffers are torch tensors on a ROCm device; this module passes their raw
pointers and the current HIP stream to libvlut.so.  Every step of the path runs
inside the library's kernels; there is no fallback: if the library is missing or
a call fails, an exception is raised.
"""
from __future__ import annotations

import ctypes
import importlib.util
import os
import sys
from typing import Optional, Tuple

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libvlut.so")
NATIVE_PATH = os.path.join(_HERE, "_vlut_torch.so")

VLUT_OK = 0
VLUT_ERR_NULL, VLUT_ERR_SHAPE, VLUT_ERR_SMALL_BUFFER = -1, -2, -3
VLUT_ERR_VALUE, VLUT_ERR_DEVICE, VLUT_ERR_UNSUPPORTED = -4, -5, -6

EXPORTS = [
    "vlut_status_string", "vlut_version", "vlut_packed_weight_bytes", "vlut_packed_offset", "vlut_act_bytes",
    "vlut_lut_bytes",
    "vlut_workspace_bytes", "vlut_pack_weights", "vlut_quantize_act", "vlut_build_lut", "vlut_mpgemm",
    "vlut_mpgemm_rows", "vlut_mpgemm_mfma", "vlut_mfma_workspace_bytes", "vlut_set_plan", "vlut_query_plan",
    "vlut_packed_weight_bytes_g5", "vlut_packed_offset_g5", "vlut_workspace_bytes_g5", "vlut_pack_weights_g5",
    "vlut_mpgemm_g5", "vlut_set_plan_g5", "vlut_query_plan_g5",
    "vlut_workspace_bytes_f32", "vlut_query_plan_f32", "vlut_mpgemm_f32",
    "vlut_build_lut_token_outer", "vlut_mpgemm_token_outer",
    "vlut_mixed_k5", "vlut_packed_weight_bytes_mixed", "vlut_workspace_bytes_mixed", "vlut_pack_weights_mixed",
    "vlut_mpgemm_mixed", "vlut_static_scratch_bytes", "vlut_mpgemm_static", "vlut_query_lookup_waves",
    "vlut_query_kernel", "vlut_query_matrix_plan", "vlut_workspace_used", "vlut_workspace_used_g5", "vlut_workspace_used_mixed",
    "vlut_mpgemm_lean", "vlut_mpgemm_g5_lean", "vlut_mpgemm_mixed_lean",
]

_lib = None


class VlutError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = status
        super().__init__(f"{where}: {status_string(status)}")


def lib() -> ctypes.CDLL:
    """Loads libvlut.so; building it is the job of __graft_entry__.build() / paper_2512_06443_amd.build."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise FileNotFoundError(f"{LIB_PATH} is missing: build it with `python -m paper_2512_06443_amd.build`")
        L = ctypes.CDLL(LIB_PATH)
        i64, sz, p, ci, cf = ctypes.c_int64, ctypes.c_size_t, ctypes.c_void_p, ctypes.c_int, ctypes.c_float
        L.vlut_status_string.argtypes, L.vlut_status_string.restype = [ci], ctypes.c_char_p
        L.vlut_version.argtypes, L.vlut_version.restype = [], ci
        L.vlut_packed_weight_bytes.argtypes, L.vlut_packed_weight_bytes.restype = [i64, i64], sz
        L.vlut_packed_offset.argtypes, L.vlut_packed_offset.restype = [i64, i64, i64, i64], sz
        L.vlut_act_bytes.argtypes, L.vlut_act_bytes.restype = [i64, i64], sz
        L.vlut_lut_bytes.argtypes, L.vlut_lut_bytes.restype = [i64, i64], sz
        L.vlut_workspace_bytes.argtypes, L.vlut_workspace_bytes.restype = [i64, i64, i64], sz
        L.vlut_mfma_workspace_bytes.argtypes, L.vlut_mfma_workspace_bytes.restype = [i64, i64, i64], sz
        L.vlut_pack_weights.argtypes, L.vlut_pack_weights.restype = [p, i64, i64, p, sz, p], ci
        L.vlut_quantize_act.argtypes, L.vlut_quantize_act.restype = [p, i64, i64, i64, p, p, p], ci
        L.vlut_build_lut.argtypes, L.vlut_build_lut.restype = [p, i64, i64, p, sz, p], ci
        gemm_args = [p, cf, p, p, p, i64, i64, i64, p, i64, p, p, sz, p]
        L.vlut_mpgemm.argtypes, L.vlut_mpgemm.restype = gemm_args, ci
        L.vlut_mpgemm_mfma.argtypes, L.vlut_mpgemm_mfma.restype = gemm_args, ci
        L.vlut_mpgemm_lean.argtypes, L.vlut_mpgemm_lean.restype = gemm_args, ci
        for f in (L.vlut_workspace_used, L.vlut_workspace_used_g5, L.vlut_workspace_used_mixed):
            f.argtypes, f.restype = [i64, i64, i64], sz
        for f in (L.vlut_mpgemm_g5_lean, L.vlut_mpgemm_mixed_lean):
            f.argtypes, f.restype = [p, cf, p, p, i64, i64, i64, p, i64, p, p, sz, p], ci
        L.vlut_mpgemm_rows.argtypes, L.vlut_mpgemm_rows.restype = [p, p] + list(gemm_args[2:]), ci
        L.vlut_packed_weight_bytes_g5.argtypes, L.vlut_packed_weight_bytes_g5.restype = [i64, i64], sz
        L.vlut_packed_offset_g5.argtypes, L.vlut_packed_offset_g5.restype = [i64, i64, i64, i64], sz
        L.vlut_workspace_bytes_g5.argtypes, L.vlut_workspace_bytes_g5.restype = [i64, i64, i64], sz
        L.vlut_pack_weights_g5.argtypes, L.vlut_pack_weights_g5.restype = [p, i64, i64, p, sz, p], ci
        L.vlut_mpgemm_g5.argtypes, L.vlut_mpgemm_g5.restype = [p, cf, p, p, i64, i64, i64, p, i64, p, p, sz, p], ci
        L.vlut_set_plan_g5.argtypes, L.vlut_set_plan_g5.restype = [ci, ci], ci
        L.vlut_query_plan_g5.argtypes, L.vlut_query_plan_g5.restype = [i64, i64, i64, ctypes.POINTER(ci)], ci
        L.vlut_mixed_k5.argtypes, L.vlut_mixed_k5.restype = [i64], i64
        L.vlut_packed_weight_bytes_mixed.argtypes, L.vlut_packed_weight_bytes_mixed.restype = [i64, i64], sz
        L.vlut_workspace_bytes_mixed.argtypes, L.vlut_workspace_bytes_mixed.restype = [i64, i64, i64], sz
        L.vlut_pack_weights_mixed.argtypes, L.vlut_pack_weights_mixed.restype = [p, i64, i64, p, sz, p], ci
        L.vlut_mpgemm_mixed.argtypes, L.vlut_mpgemm_mixed.restype = [p, cf, p, p, i64, i64, i64, p, i64, p, p, sz, p], ci
        L.vlut_build_lut_token_outer.argtypes, L.vlut_build_lut_token_outer.restype = [p, i64, i64, p, sz, p], ci
        L.vlut_mpgemm_token_outer.argtypes = [p, cf, p, p, i64, i64, i64, p, i64, p, p]
        L.vlut_mpgemm_token_outer.restype = ci
        L.vlut_workspace_bytes_f32.argtypes, L.vlut_workspace_bytes_f32.restype = [i64, i64, i64], sz
        L.vlut_query_plan_f32.argtypes, L.vlut_query_plan_f32.restype = [i64, i64, i64, ctypes.POINTER(ci)], ci
        L.vlut_mpgemm_f32.argtypes = [p, cf, p, p, i64, i64, i64, i64, p, i64, p, p, p, sz, p]
        L.vlut_mpgemm_f32.restype = ci
        L.vlut_query_lookup_waves.argtypes, L.vlut_query_lookup_waves.restype = [i64, i64, i64], ci
        L.vlut_query_kernel.argtypes, L.vlut_query_kernel.restype = [ci, i64, i64, i64], ci
        L.vlut_query_matrix_plan.argtypes, L.vlut_query_matrix_plan.restype = [ci, i64, i64, i64, ctypes.POINTER(ci)], ci
        L.vlut_static_scratch_bytes.argtypes, L.vlut_static_scratch_bytes.restype = [], sz
        L.vlut_mpgemm_static.argtypes, L.vlut_mpgemm_static.restype = [p, cf, p, p, i64, i64, i64, p, i64, p, p], ci
        L.vlut_set_plan.argtypes, L.vlut_set_plan.restype = [ci, ci, ci, ci], ci
        L.vlut_query_plan.argtypes, L.vlut_query_plan.restype = [i64, i64, i64, ctypes.POINTER(ci)], ci
        _load_native(L)
        _lib = L
    return _lib


# The frequent calls as native code (csrc/torch_calls.cpp): the same arguments, outputs and library call without ctypes and without
# torch's Python layer.  Each returns None for arguments it leaves to the Python form below it (which also raises every
# error), an int status or the tuple of outputs.  None here: not built, or built for another torch; the Python form serves then.
# The products take the lean form of the call: no workspace is allocated where the kernel leaves it alone (0.75 us each).
# Host time of a call, Python / native form, us (640 x 2560, four tokens; the launch alone is 2.2): quantize_act 7.9 / 4.9,
# mpgemm 7.6 / 4.4, with y and workspace given 5.5 / 3.4, mpgemm_g5 and mpgemm_mixed 4.5, mpgemm_f32 7.6 / 4.4; with a workspace for
# each call, a launch by <<< >>> and the rules worked out anew 5.3, 4.6, 3.6, 5.9 and 4.5 (hosts differ: the native forms 4.5, 3.8, 2.9, 3.9
# and 3.8 on another; with a layer's four matrices in turn within 0.2 of that).
_native = None
_NATIVE_ORDER = ("vlut_quantize_act", "vlut_mpgemm_lean", "vlut_workspace_used", "vlut_mpgemm_f32", "vlut_workspace_bytes_f32", "vlut_mpgemm_g5_lean",
                 "vlut_workspace_used_g5", "vlut_mpgemm_mixed_lean", "vlut_workspace_used_mixed", "vlut_pack_weights",
                 "vlut_packed_weight_bytes", "vlut_pack_weights_g5", "vlut_packed_weight_bytes_g5", "vlut_pack_weights_mixed",
                 "vlut_packed_weight_bytes_mixed")


def built_for() -> str:
    """What NATIVE_PATH is compiled against: it holds layouts and key numbers of torch's headers, and a file for others may load all the same."""
    return f"torch {torch.__version__} {getattr(torch.version, 'git_version', '')} python {sys.version_info[0]}.{sys.version_info[1]}"


def _load_native(L: ctypes.CDLL) -> None:
    global _native
    if not os.path.exists(NATIVE_PATH) or not hasattr(torch._C, "_cuda_getCurrentRawStream"):
        return
    try:
        spec = importlib.util.spec_from_file_location("_vlut_torch", NATIVE_PATH)
        mod = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(mod)
    except ImportError:                 # built for another torch
        return
    if getattr(mod, "built_for", None) != built_for():      # (whose symbols are all here)
        return
    mod.bind(*[ctypes.cast(getattr(L, f), ctypes.c_void_p).value for f in _NATIVE_ORDER])
    _native = mod


def status_string(status: int) -> str:
    return lib().vlut_status_string(status).decode()


def _check(status: int, where: str) -> None:
    if status != VLUT_OK:
        raise VlutError(status, where)


# The raw handle of the current device's current stream.  torch.cuda.current_stream() builds a Stream object around the same
# handle, 2.7 us of a call that takes 8.7; asking for the handle itself takes 0.1.  The two functions are private names of torch:
# where a build does not have them (one without a GPU, on which the size helpers still work) the public call serves.
if hasattr(torch._C, "_cuda_getCurrentRawStream") and hasattr(torch._C, "_cuda_getDevice"):
    _raw_stream, _device = torch._C._cuda_getCurrentRawStream, torch._C._cuda_getDevice

    def _stream() -> int:
        return _raw_stream(_device())
else:
    def _stream() -> int:
        return torch.cuda.current_stream().cuda_stream


def _outputs(r, where: str):
    """What a native call returned: the outputs, or the status of a call that was refused."""
    if type(r) is tuple:
        return r
    raise VlutError(r, where)


def _ptr(t: Optional[torch.Tensor]) -> Optional[int]:
    return None if t is None else t.data_ptr()


def packed_weight_bytes(M: int, K: int) -> int:
    return lib().vlut_packed_weight_bytes(M, K)


def packed_offset(M: int, K: int, m: int, kg: int) -> int:
    return lib().vlut_packed_offset(M, K, m, kg)


def act_bytes(K: int, N: int) -> int:
    return lib().vlut_act_bytes(K, N)


def act_chunked_to_kn(a_q: torch.Tensor, N: int) -> torch.Tensor:
    """View helper for checks: token-chunked int8 [ceil(N/8)][K][8] -> plain [K][N] (a copy)."""
    C, K, _ = a_q.shape
    return a_q.permute(1, 0, 2).reshape(K, C * 8)[:, :N].contiguous()


def lut_bytes(K: int, N: int) -> int:
    return lib().vlut_lut_bytes(K, N)


def workspace_bytes(M: int, K: int, N: int) -> int:
    return lib().vlut_workspace_bytes(M, K, N)


def set_plan(J: int = 0, R: int = 0, waves: int = 0, split_k: int = 0) -> None:
    _check(lib().vlut_set_plan(J, R, waves, split_k), "vlut_set_plan")


def query_plan(M: int, K: int, N: int) -> Tuple[int, int, int, int]:
    out = (ctypes.c_int * 4)()
    _check(lib().vlut_query_plan(M, K, N, out), "vlut_query_plan")
    return out[0], out[1], out[2], out[3]


def pack_weights(w_ternary: torch.Tensor) -> torch.Tensor:
    """int8 [M][K] on the GPU -> packed uint8 blob (opaque tile layout) on the GPU."""
    if _native is not None:
        r = _native.pack_weights(w_ternary)
        if r is not None:
            return _outputs(r, "vlut_pack_weights")[0]
    assert w_ternary.is_cuda and w_ternary.dtype == torch.int8 and w_ternary.is_contiguous()
    M, K = w_ternary.shape
    nbytes = packed_weight_bytes(M, K)
    if nbytes == 0:
        raise VlutError(VLUT_ERR_SHAPE, "vlut_packed_weight_bytes")
    packed = torch.empty(nbytes, dtype=torch.uint8, device=w_ternary.device)
    _check(lib().vlut_pack_weights(_ptr(w_ternary), M, K, _ptr(packed), nbytes, _stream()), "vlut_pack_weights")
    return packed


def quantize_act(x: torch.Tensor, a_q: Optional[torch.Tensor] = None, a_scale: Optional[torch.Tensor] = None):
    """fp32 [N][K] (row stride >= K) -> (int8 token-chunked [ceil(N/8)][K][8], fp32 [N])."""
    if _native is not None:
        r = _native.quantize_act(x, a_q, a_scale)
        if r is not None:
            return _outputs(r, "vlut_quantize_act")
    assert x.is_cuda and x.dtype == torch.float32 and x.dim() == 2 and x.stride(1) == 1
    N, K = x.shape
    if a_q is None:
        a_q = torch.empty(((N + 7) // 8, K, 8), dtype=torch.int8, device=x.device)
    if a_scale is None:
        a_scale = torch.empty(N, dtype=torch.float32, device=x.device)
    _check(lib().vlut_quantize_act(_ptr(x), N, K, x.stride(0), _ptr(a_q), _ptr(a_scale), _stream()), "vlut_quantize_act")
    return a_q, a_scale


def build_lut(a_q: torch.Tensor, N: int, lut: Optional[torch.Tensor] = None) -> torch.Tensor:
    assert a_q.is_cuda and a_q.dtype == torch.int8 and a_q.is_contiguous() and a_q.dim() == 3
    K = a_q.shape[1]
    assert a_q.shape[0] == (N + 7) // 8
    if lut is None:
        lut = torch.empty((K // 4, 81, N), dtype=torch.int16, device=a_q.device)
    _check(lib().vlut_build_lut(_ptr(a_q), K, N, _ptr(lut), lut.numel() * 2, _stream()), "vlut_build_lut")
    return lut


def mpgemm(packed: torch.Tensor, w_scale: float, a_q: torch.Tensor, a_scale: torch.Tensor, M: int,
           y: Optional[torch.Tensor] = None, acc: Optional[torch.Tensor] = None, lut: Optional[torch.Tensor] = None,
           workspace: Optional[torch.Tensor] = None, want_acc: bool = False, mfma: bool = False):
    """Runs vlut_mpgemm (or the MFMA comparison path).  Returns (y fp32 [N][M], acc int32 [M][N] or None)."""
    if _native is not None and lut is None and not mfma:
        r = _native.mpgemm(packed, w_scale, a_q, a_scale, M, y, acc, want_acc, workspace)
        if r is not None:
            return _outputs(r, "vlut_mpgemm")
    K, N = a_q.shape[1], a_scale.shape[0]
    dev = a_q.device
    if y is None:
        y = torch.empty((N, M), dtype=torch.float32, device=dev)
    if acc is None and want_acc:
        acc = torch.empty((M, N), dtype=torch.int32, device=dev)
    ws_bytes = lib().vlut_mfma_workspace_bytes(M, K, N) if mfma else workspace_bytes(M, K, N)
    if workspace is None and ws_bytes:
        workspace = torch.empty(ws_bytes, dtype=torch.uint8, device=dev)
    fn = lib().vlut_mpgemm_mfma if mfma else lib().vlut_mpgemm
    rc = fn(_ptr(packed), float(w_scale), _ptr(a_q), _ptr(a_scale), _ptr(lut), M, K, N, _ptr(y), y.stride(0),
            _ptr(acc), _ptr(workspace), 0 if workspace is None else workspace.numel() * workspace.element_size(),
            _stream())
    _check(rc, "vlut_mpgemm_mfma" if mfma else "vlut_mpgemm")
    return y, acc


def query_lookup_waves(M: int, K: int, N: int) -> int:
    """Lookup waves per workgroup (12 or 14) of the plan query_plan reports; 0 for the few-token kernel."""
    w = lib().vlut_query_lookup_waves(M, K, N)
    if w < 0:
        raise VlutError(w, "vlut_query_lookup_waves")
    return w


_FORMS = {"codes": 0, "f32": 1, "g5": 2, "mixed": 3}
_KERNELS = {1: "lookup", 2: "few_tokens", 3: "matrix", 4: "matrix_few_tokens"}


def query_kernel(form: str, M: int, K: int, N: int) -> str:
    """The kernel that computes the product of `mpgemm` ("codes"), `mpgemm_f32` ("f32"), `mpgemm_g5` ("g5") or
    `mpgemm_mixed` ("mixed"): "lookup", "few_tokens", "matrix" or "matrix_few_tokens" (VLUT_KERNEL_* of the header).
    From INT8 codes both "few_tokens" and "matrix" can be the matrix-core kernel for a few tokens: query_matrix_plan tells."""
    k = lib().vlut_query_kernel(_FORMS[form], M, K, N)
    if k < 0:
        raise VlutError(k, "vlut_query_kernel")
    return _KERNELS[k]


def query_matrix_plan(form: str, M: int, K: int, N: int) -> Optional[Tuple[int, int, int, int]]:
    """(rows, tokens, parts of K) of a workgroup and the number of workgroups of the matrix-core kernel that computes the
    product of such a call; up to 16 tokens: a kernel for a few tokens.  None where a kernel that looks up tables runs."""
    out = (ctypes.c_int * 4)()
    rc = lib().vlut_query_matrix_plan(_FORMS[form], M, K, N, out)
    if rc == VLUT_ERR_UNSUPPORTED and lib().vlut_query_kernel(_FORMS[form], M, K, N) > 0:
        return None
    _check(rc, "vlut_query_matrix_plan")
    return out[0], out[1], out[2], out[3]


def static_scratch_bytes() -> int:
    return lib().vlut_static_scratch_bytes()


def mpgemm_static(packed: torch.Tensor, w_scale: float, a_q: torch.Tensor, a_scale: torch.Tensor, M: int,
                  y: torch.Tensor, acc: Optional[torch.Tensor] = None):
    """Runs vlut_mpgemm_static: the caller passes inputs and outputs only, the split-K scratch is the library's own
    static device array; neither this wrapper nor the call allocates anything."""
    K, N = a_q.shape[1], a_scale.shape[0]
    rc = lib().vlut_mpgemm_static(_ptr(packed), float(w_scale), _ptr(a_q), _ptr(a_scale), M, K, N, _ptr(y), y.stride(0),
                                  _ptr(acc), _stream())
    _check(rc, "vlut_mpgemm_static")
    return y, acc


def mpgemm_rows(packed: torch.Tensor, w_scale_rows: torch.Tensor, a_q: torch.Tensor, a_scale: torch.Tensor, M: int,
                y: Optional[torch.Tensor] = None, want_acc: bool = False, workspace: Optional[torch.Tensor] = None):
    """Runs vlut_mpgemm_rows: stacked weight matrices, one weight scale per output row (fp32 [M] on the GPU)."""
    assert w_scale_rows.is_cuda and w_scale_rows.dtype == torch.float32 and w_scale_rows.numel() == M
    K, N = a_q.shape[1], a_scale.shape[0]
    dev = a_q.device
    if y is None:
        y = torch.empty((N, M), dtype=torch.float32, device=dev)
    acc = torch.empty((M, N), dtype=torch.int32, device=dev) if want_acc else None
    ws_bytes = workspace_bytes(M, K, N)
    if workspace is None and ws_bytes:
        workspace = torch.empty(ws_bytes, dtype=torch.uint8, device=dev)
    rc = lib().vlut_mpgemm_rows(_ptr(packed), _ptr(w_scale_rows), _ptr(a_q), _ptr(a_scale), None, M, K, N, _ptr(y),
                                y.stride(0), _ptr(acc), _ptr(workspace),
                                0 if workspace is None else workspace.numel() * workspace.element_size(), _stream())
    _check(rc, "vlut_mpgemm_rows")
    return y, acc


def build_lut_token_outer(a_q: torch.Tensor, N: int) -> torch.Tensor:
    """The table with the token index outermost, int16 [N][K/4][81] (layout ablation)."""
    assert a_q.is_cuda and a_q.dtype == torch.int8 and a_q.is_contiguous() and a_q.dim() == 3
    K = a_q.shape[1]
    lut = torch.empty((N, K // 4, 81), dtype=torch.int16, device=a_q.device)
    _check(lib().vlut_build_lut_token_outer(_ptr(a_q), K, N, _ptr(lut), lut.numel() * 2, _stream()),
           "vlut_build_lut_token_outer")
    return lut


def mpgemm_token_outer(packed: torch.Tensor, w_scale: float, a_scale: torch.Tensor, lut: torch.Tensor, M: int,
                       want_acc: bool = False):
    """Runs vlut_mpgemm_token_outer on a table from build_lut_token_outer.  Returns (y [N][M], acc or None)."""
    N, G, _ = lut.shape
    y = torch.empty((N, M), dtype=torch.float32, device=lut.device)
    acc = torch.empty((M, N), dtype=torch.int32, device=lut.device) if want_acc else None
    _check(lib().vlut_mpgemm_token_outer(_ptr(packed), float(w_scale), _ptr(a_scale), _ptr(lut), M, 4 * G, N, _ptr(y),
                                         y.stride(0), _ptr(acc), _stream()), "vlut_mpgemm_token_outer")
    return y, acc


def query_plan_f32(M: int, K: int, N: int) -> Tuple[int, int, int, int, bool]:
    """(J, R, split_k, workgroups, one launch) of vlut_mpgemm_f32 for this shape; query_kernel names the kernel."""
    out = (ctypes.c_int * 5)()
    _check(lib().vlut_query_plan_f32(M, K, N, out), "vlut_query_plan_f32")
    return out[0], out[1], out[2], out[3], bool(out[4])


def mpgemm_f32(packed: torch.Tensor, w_scale, x: torch.Tensor, M: int, y: Optional[torch.Tensor] = None,
               want_acc: bool = False, want_scales: bool = False, workspace: Optional[torch.Tensor] = None):
    """Runs vlut_mpgemm_f32 on fp32 activations x [N][K] (row stride >= K).  w_scale: a float, or an fp32 [M]
    tensor on the GPU with one weight scale per output row.  Returns (y [N][M], acc or None, a_scale or None)."""
    if _native is not None:
        r = _native.mpgemm_f32(packed, w_scale, x, M, y, want_acc, want_scales, workspace)
        if r is not None:
            return _outputs(r, "vlut_mpgemm_f32")
    assert x.is_cuda and x.dtype == torch.float32 and x.dim() == 2 and x.stride(1) == 1
    L = _lib or lib()
    N, K = x.shape
    rows = w_scale if isinstance(w_scale, torch.Tensor) else None
    if rows is not None:
        assert rows.is_cuda and rows.dtype == torch.float32 and rows.numel() == M
    if y is None:
        y = torch.empty((N, M), dtype=torch.float32, device=x.device)
    acc = torch.empty((M, N), dtype=torch.int32, device=x.device) if want_acc else None
    scales = torch.empty(N, dtype=torch.float32, device=x.device) if want_scales else None
    if workspace is None:
        ws_bytes = L.vlut_workspace_bytes_f32(M, K, N)
        if ws_bytes:
            workspace = torch.empty(ws_bytes, dtype=torch.uint8, device=x.device)
    else:
        ws_bytes = workspace.numel() * workspace.element_size()
    rc = L.vlut_mpgemm_f32(_ptr(packed), 1.0 if rows is not None else float(w_scale), _ptr(rows), x.data_ptr(), x.stride(0),
                           M, K, N, y.data_ptr(), y.stride(0), _ptr(acc), _ptr(scales), _ptr(workspace), ws_bytes, _stream())
    if rc != VLUT_OK:
        raise VlutError(rc, "vlut_mpgemm_f32")
    return y, acc, scales


# ---- 1.60-bit packing (g = 5)
def pack_weights_g5(w_ternary: torch.Tensor) -> torch.Tensor:
    """int8 [M][K] (K % 5 == 0) on the GPU -> 1.60-bit packed blob on the GPU."""
    if _native is not None:
        r = _native.pack_weights_g5(w_ternary)
        if r is not None:
            return _outputs(r, "vlut_pack_weights_g5")[0]
    assert w_ternary.is_cuda and w_ternary.dtype == torch.int8 and w_ternary.is_contiguous()
    M, K = w_ternary.shape
    nbytes = lib().vlut_packed_weight_bytes_g5(M, K)
    if nbytes == 0:
        raise VlutError(VLUT_ERR_SHAPE, "vlut_packed_weight_bytes_g5")
    packed = torch.empty(nbytes, dtype=torch.uint8, device=w_ternary.device)
    _check(lib().vlut_pack_weights_g5(_ptr(w_ternary), M, K, _ptr(packed), nbytes, _stream()), "vlut_pack_weights_g5")
    return packed


def pack_weights_mixed(w_ternary: torch.Tensor) -> torch.Tensor:
    """int8 [M][K] (K % 4 == 0) on the GPU -> blob of the mixed 1.60-bit / 2-bit packing on the GPU."""
    if _native is not None:
        r = _native.pack_weights_mixed(w_ternary)
        if r is not None:
            return _outputs(r, "vlut_pack_weights_mixed")[0]
    assert w_ternary.is_cuda and w_ternary.dtype == torch.int8 and w_ternary.is_contiguous()
    M, K = w_ternary.shape
    nbytes = lib().vlut_packed_weight_bytes_mixed(M, K)
    if nbytes == 0:
        raise VlutError(VLUT_ERR_SHAPE, "vlut_packed_weight_bytes_mixed")
    packed = torch.empty(nbytes, dtype=torch.uint8, device=w_ternary.device)
    _check(lib().vlut_pack_weights_mixed(_ptr(w_ternary), M, K, _ptr(packed), nbytes, _stream()), "vlut_pack_weights_mixed")
    return packed


def mpgemm_mixed(packed: torch.Tensor, w_scale: float, a_q: torch.Tensor, a_scale: torch.Tensor, M: int,
                 y: Optional[torch.Tensor] = None, want_acc: bool = False):
    """Runs vlut_mpgemm_mixed on a blob from pack_weights_mixed.  Returns (y [N][M], acc or None)."""
    if _native is not None:
        r = _native.mpgemm_mixed(packed, w_scale, a_q, a_scale, M, y, None, want_acc, None)
        if r is not None:
            return _outputs(r, "vlut_mpgemm_mixed")
    K, N = a_q.shape[1], a_scale.shape[0]
    dev = a_q.device
    if y is None:
        y = torch.empty((N, M), dtype=torch.float32, device=dev)
    acc = torch.empty((M, N), dtype=torch.int32, device=dev) if want_acc else None
    ws = torch.empty(max(lib().vlut_workspace_bytes_mixed(M, K, N), 16), dtype=torch.uint8, device=dev)
    _check(lib().vlut_mpgemm_mixed(_ptr(packed), float(w_scale), _ptr(a_q), _ptr(a_scale), M, K, N, _ptr(y), y.stride(0),
                                   _ptr(acc), _ptr(ws), ws.numel(), _stream()), "vlut_mpgemm_mixed")
    return y, acc


def set_plan_g5(R: int = 0, split_k: int = 0) -> None:
    _check(lib().vlut_set_plan_g5(R, split_k), "vlut_set_plan_g5")


def query_plan_g5(M: int, K: int, N: int) -> Tuple[int, int, int]:
    out = (ctypes.c_int * 3)()
    _check(lib().vlut_query_plan_g5(M, K, N, out), "vlut_query_plan_g5")
    return out[0], out[1], out[2]


def mpgemm_g5(packed: torch.Tensor, w_scale: float, a_q: torch.Tensor, a_scale: torch.Tensor, M: int,
              y: Optional[torch.Tensor] = None, want_acc: bool = False, workspace: Optional[torch.Tensor] = None):
    """Runs vlut_mpgemm_g5.  Returns (y fp32 [N][M], acc int32 [M][N] or None)."""
    if _native is not None:
        r = _native.mpgemm_g5(packed, w_scale, a_q, a_scale, M, y, None, want_acc, workspace)
        if r is not None:
            return _outputs(r, "vlut_mpgemm_g5")
    K, N = a_q.shape[1], a_scale.shape[0]
    dev = a_q.device
    if y is None:
        y = torch.empty((N, M), dtype=torch.float32, device=dev)
    acc = torch.empty((M, N), dtype=torch.int32, device=dev) if want_acc else None
    ws_bytes = lib().vlut_workspace_bytes_g5(M, K, N)
    if workspace is None and ws_bytes:
        workspace = torch.empty(ws_bytes, dtype=torch.uint8, device=dev)
    rc = lib().vlut_mpgemm_g5(_ptr(packed), float(w_scale), _ptr(a_q), _ptr(a_scale), M, K, N, _ptr(y), y.stride(0),
                              _ptr(acc), _ptr(workspace),
                              0 if workspace is None else workspace.numel() * workspace.element_size(), _stream())
    _check(rc, "vlut_mpgemm_g5")
    return y, acc
