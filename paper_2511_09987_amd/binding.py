"""ctypes binding of libcyclotron_mm.so.  Same names as the C ABI (include/cyclotron_mm.h).

PyTorch appears here only as the owner of device memory and streams.  There is no
fallback: if the shared library is missing, the first call raises ImportError.
"""
from __future__ import annotations

import ctypes
import os

CYC_BF16_F32 = 0
CYC_I8_I32 = 1
CYC_OK = 0
CYC_ERR_WORKSPACE = 6

_HERE = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(_HERE, "libcyclotron_mm.so")


def lib_path() -> str:
    return _LIB_PATH


def _load() -> ctypes.CDLL:
    if not os.path.exists(_LIB_PATH):
        raise ImportError(f"{_LIB_PATH} is not built; run `python -m paper_2511_09987_amd.build` "
                          "(needs hipcc, cross-compiles for gfx950)")
    lib = ctypes.CDLL(_LIB_PATH)
    i64, ptr, cint = ctypes.c_int64, ctypes.c_void_p, ctypes.c_int
    lib.cyc_recurrence_matmul.argtypes = [ptr, ptr, ptr, i64, i64, i64, cint, ptr]
    lib.cyc_recurrence_matmul.restype = cint
    lib.cyc_recurrence_matmul_noalloc.argtypes = [ptr, ptr, ptr, i64, i64, i64, cint, ptr]
    lib.cyc_recurrence_matmul_noalloc.restype = cint
    lib.cyc_recurrence_matmul_batched.argtypes = [ptr, ptr, ptr, i64, i64, i64, i64, i64, i64, i64, cint, ptr]
    lib.cyc_recurrence_matmul_batched.restype = cint
    lib.cyc_recurrence_matmul_in.argtypes = [ptr, ptr, ptr, i64, i64, i64, cint, ptr, i64, ptr]
    lib.cyc_recurrence_matmul_in.restype = cint
    lib.cyc_matmul_workspace.argtypes = [ptr, ptr, ptr, i64, i64, i64, cint]
    lib.cyc_matmul_workspace.restype = i64
    lib.cyc_recurrence_trsm.argtypes = [ptr, ptr, ptr, ptr, i64, i64, i64, ptr]
    lib.cyc_recurrence_trsm.restype = cint
    lib.cyc_recurrence_cholesky.argtypes = [ptr, ptr, ptr, i64, i64, ptr]
    lib.cyc_recurrence_cholesky.restype = cint
    lib.cyc_recurrence_trsm_in.argtypes = [ptr, ptr, ptr, ptr, i64, i64, i64, ptr, i64, ptr]
    lib.cyc_recurrence_trsm_in.restype = cint
    lib.cyc_trsm_workspace.argtypes = [ptr, ptr, ptr, i64, i64, i64]
    lib.cyc_trsm_workspace.restype = i64
    lib.cyc_recurrence_cholesky_in.argtypes = [ptr, ptr, ptr, i64, i64, ptr, i64, ptr]
    lib.cyc_recurrence_cholesky_in.restype = cint
    lib.cyc_cholesky_workspace.argtypes = [ptr, ptr, ptr, i64, i64]
    lib.cyc_cholesky_workspace.restype = i64
    lib.cyc_recurrence_attention.argtypes = [ptr, ptr, ptr, ptr, i64, i64, i64, i64, ptr]
    lib.cyc_recurrence_attention.restype = cint
    lib.cyc_recurrence_attention_split.argtypes = [ptr, ptr, ptr, ptr, i64, i64, i64, i64, ptr, i64, ptr]
    lib.cyc_recurrence_attention_split.restype = cint
    lib.cyc_attention_workspace.argtypes = [i64, i64, i64, i64]
    lib.cyc_attention_workspace.restype = i64
    lib.cyc_status_string.argtypes = [cint]
    lib.cyc_status_string.restype = ctypes.c_char_p
    lib.cyc_version.argtypes = []
    lib.cyc_version.restype = cint
    lib.cyc_kernel_name.argtypes = [ptr, ptr, ptr, i64, i64, i64, i64, i64, i64, i64, cint]
    lib.cyc_kernel_name.restype = ctypes.c_char_p
    lib.cyc_kernel_variant.argtypes = lib.cyc_kernel_name.argtypes
    lib.cyc_kernel_variant.restype = ctypes.c_char_p
    lib.cyc_force_kernel.argtypes = [ctypes.c_char_p]
    lib.cyc_force_kernel.restype = cint
    lib.cyc_diag_mfma_ceiling.argtypes = [cint, cint, i64, ptr, ctypes.POINTER(ctypes.c_double), ptr]
    lib.cyc_diag_mfma_ceiling.restype = cint
    lib.cyc_diag_issue_mix.argtypes = [cint, cint, cint, cint, i64, ptr, ctypes.POINTER(ctypes.c_double), ptr]
    lib.cyc_diag_issue_mix.restype = cint
    lib.cyc_diag_mfma_f32_tiles.argtypes = [ptr, ptr, ptr, ptr, i64, ptr]
    lib.cyc_diag_mfma_f32_tiles.restype = cint
    lib.cyc_diag_pivots.argtypes = [cint, i64, i64, ptr, ptr]
    lib.cyc_diag_pivots.restype = cint
    lib.cyc_diag_set_wait_limit.argtypes = [i64]
    lib.cyc_diag_set_wait_limit.restype = cint
    lib.cyc_diag_clock.argtypes = [ptr, i64, ptr]
    lib.cyc_diag_clock.restype = cint
    return lib


_cached = None


def _lib() -> ctypes.CDLL:
    """The loaded library; loading is deferred to first use so that the build module can be
    imported before the library exists.  Raises ImportError if it is not built."""
    global _cached
    if _cached is None:
        _cached = _load()
    return _cached


def _stream_handle(tensor, stream) -> int:
    """The handle of `stream`, or of the current stream of the tensor's device.  torch.cuda.current_stream builds an object
    around it, which takes 1.8 us of the 9 us that a small call spends on the host; asking for the handle takes 0.1."""
    import torch
    if stream is not None:
        return stream.cuda_stream
    raw = getattr(torch._C, "_cuda_getCurrentRawStream", None)
    return raw(tensor.device.index) if raw else torch.cuda.current_stream(tensor.device).cuda_stream


def _memory(wanted: int, tensor, stream):
    """`wanted` bytes from the allocator's pool of the stream that a call runs on, or None.  They go back to that pool when the
    caller drops them: whoever gets them next is ordered after the call.  Under capture they belong to the graph."""
    import torch
    try:
        if stream is None:
            return torch.empty(wanted, dtype=torch.uint8, device=tensor.device)
        if isinstance(stream, torch.cuda.Stream) and stream.device == tensor.device:
            with torch.cuda.stream(stream):
                return torch.empty(wanted, dtype=torch.uint8, device=tensor.device)
    except torch.OutOfMemoryError:
        pass
    return None


class CycError(RuntimeError):
    def __init__(self, status: int):
        self.status = status
        super().__init__(cyc_status_string(status))


def cyc_status_string(status: int) -> str:
    return _lib().cyc_status_string(int(status)).decode()


def cyc_version() -> int:
    return int(_lib().cyc_version())


def cyc_recurrence_matmul(A: int, B: int, C: int, M: int, K: int, N: int, dtype: int, stream: int = 0) -> int:
    """Raw call: device addresses as ints, returns the cyc_status."""
    return int(_lib().cyc_recurrence_matmul(A, B, C, M, K, N, dtype, stream))


def cyc_recurrence_matmul_noalloc(A: int, B: int, C: int, M: int, K: int, N: int, dtype: int, stream: int = 0) -> int:
    """Raw call of the allocation-free variant: device addresses as ints, returns the cyc_status."""
    return int(_lib().cyc_recurrence_matmul_noalloc(A, B, C, M, K, N, dtype, stream))


def cyc_recurrence_matmul_batched(A: int, B: int, C: int, batch: int, M: int, K: int, N: int,
                                  strideA: int, strideB: int, strideC: int, dtype: int, stream: int = 0) -> int:
    return int(_lib().cyc_recurrence_matmul_batched(A, B, C, batch, M, K, N, strideA, strideB, strideC,
                                                  dtype, stream))


def cyc_matmul_workspace(A: int, B: int, C: int, M: int, K: int, N: int, dtype: int) -> int:
    """Bytes of workspace that cyc_recurrence_matmul_in wants for this problem."""
    return int(_lib().cyc_matmul_workspace(A, B, C, M, K, N, dtype))


def cyc_recurrence_matmul_in(A: int, B: int, C: int, M: int, K: int, N: int, dtype: int, workspace: int, workspace_bytes: int,
                             stream: int = 0) -> int:
    """Raw call: device addresses as ints, returns the cyc_status."""
    return int(_lib().cyc_recurrence_matmul_in(A, B, C, M, K, N, dtype, workspace, workspace_bytes, stream))


def cyc_recurrence_trsm(L: int, B: int, X: int, Xh: int, n: int, nrhs: int, nb: int, stream: int = 0) -> int:
    """Raw call: device addresses as ints, returns the cyc_status."""
    return int(_lib().cyc_recurrence_trsm(L, B, X, Xh, n, nrhs, nb, stream))


def cyc_trsm_workspace(L: int, X: int, Xh: int, n: int, nrhs: int, nb: int) -> int:
    """Bytes of workspace that cyc_recurrence_trsm_in wants for this system."""
    return int(_lib().cyc_trsm_workspace(L, X, Xh, n, nrhs, nb))


def cyc_recurrence_trsm_in(L: int, B: int, X: int, Xh: int, n: int, nrhs: int, nb: int, workspace: int, workspace_bytes: int,
                           stream: int = 0) -> int:
    """Raw call: device addresses as ints, returns the cyc_status."""
    return int(_lib().cyc_recurrence_trsm_in(L, B, X, Xh, n, nrhs, nb, workspace, workspace_bytes, stream))


def cyc_recurrence_attention(Q: int, K: int, V: int, O: int, batch: int, N: int, M: int, d: int, stream: int = 0) -> int:
    """Raw call: device addresses as ints, returns the cyc_status."""
    return int(_lib().cyc_recurrence_attention(Q, K, V, O, batch, N, M, d, stream))


def cyc_attention_workspace(batch: int, N: int, M: int, d: int) -> int:
    """Bytes of workspace that cyc_recurrence_attention_split wants for these extents."""
    return int(_lib().cyc_attention_workspace(batch, N, M, d))


def cyc_recurrence_attention_split(Q: int, K: int, V: int, O: int, batch: int, N: int, M: int, d: int, workspace: int,
                                   workspace_bytes: int, stream: int = 0) -> int:
    """Raw call: device addresses as ints, returns the cyc_status."""
    return int(_lib().cyc_recurrence_attention_split(Q, K, V, O, batch, N, M, d, workspace, workspace_bytes, stream))


def cyc_kernel_name(A: int, B: int, C: int, batch: int, M: int, K: int, N: int,
                    strideA: int, strideB: int, strideC: int, dtype: int) -> str:
    return _lib().cyc_kernel_name(A, B, C, batch, M, K, N, strideA, strideB, strideC, dtype).decode()


def cyc_kernel_variant(A: int, B: int, C: int, batch: int, M: int, K: int, N: int,
                       strideA: int, strideB: int, strideC: int, dtype: int) -> str:
    """The kernel that runs, where cyc_kernel_name says whose part of the dispatch the problem falls into."""
    return _lib().cyc_kernel_variant(A, B, C, batch, M, K, N, strideA, strideB, strideC, dtype).decode()


def cyc_force_kernel(name) -> int:
    """Force a kernel by name (None or "": back to the dispatcher); returns the cyc_status."""
    return int(_lib().cyc_force_kernel((name or "").encode()))


def cyc_diag_mfma_ceiling(dtype: int, mfma_shape: int, iters: int, sink: int, stream: int = 0):
    """Raw call; returns (cyc_status, operations of the launch)."""
    ops = ctypes.c_double(0.0)
    st = int(_lib().cyc_diag_mfma_ceiling(dtype, mfma_shape, iters, sink, ctypes.byref(ops), stream))
    return st, ops.value


def cyc_diag_issue_mix(mfma_shape: int, other_kind: int, others_per_round: int, waves_per_simd: int, iters: int, sink: int,
                       stream: int = 0):
    """Raw call; returns (cyc_status, MFMA operations of the launch)."""
    ops = ctypes.c_double(0.0)
    st = int(_lib().cyc_diag_issue_mix(mfma_shape, other_kind, others_per_round, waves_per_simd, iters, sink, ctypes.byref(ops), stream))
    return st, ops.value


def cyc_diag_mfma_f32_tiles(A: int, B: int, C: int, D: int, tiles: int, stream: int = 0) -> int:
    return int(_lib().cyc_diag_mfma_f32_tiles(A, B, C, D, tiles, stream))


def cyc_diag_pivots(what: int, first: int, count: int, bad: int, stream: int = 0) -> int:
    return int(_lib().cyc_diag_pivots(what, first, count, bad, stream))


def cyc_diag_set_wait_limit(polls: int) -> int:
    return int(_lib().cyc_diag_set_wait_limit(polls))


def cyc_diag_clock(out: int, microseconds: int, stream: int = 0) -> int:
    return int(_lib().cyc_diag_clock(out, microseconds, stream))


def recurrence_matmul(A, B, out=None, stream=None):
    """Tensor-level convenience: C = weight-stationary recurrence of A against B.

    A: (M,K) or (batch,M,K); B: (K,N) or (batch,K,N); contiguous CUDA tensors, both
    torch.bfloat16 (C float32) or both torch.int8 (C int32).  Only allocates C and, under
    stream capture, memory for the partial products of a long k, and forwards pointers to the
    C ABI on the current (or given) stream.  (Where no memory is to be had for those, fewer
    slices of k or none are taken, and the fp32 sums are added in another order.)
    """
    import torch
    if not (A.is_cuda and B.is_cuda):
        raise ValueError("A and B must be device tensors; there is no CPU path")
    if A.dtype != B.dtype or A.dtype not in (torch.bfloat16, torch.int8):
        raise ValueError("A and B must both be bfloat16 or both int8")
    if A.dim() != B.dim() or A.dim() not in (2, 3) or not (A.is_contiguous() and B.is_contiguous()):
        raise ValueError("A and B must be contiguous and both 2-D or both 3-D")
    dtype = CYC_BF16_F32 if A.dtype == torch.bfloat16 else CYC_I8_I32
    batch = A.shape[0] if A.dim() == 3 else 1
    M, K = A.shape[-2:]
    K2, N = B.shape[-2:]
    if K != K2 or (A.dim() == 3 and B.shape[0] != batch):
        raise ValueError(f"shape mismatch: A {tuple(A.shape)}, B {tuple(B.shape)}")
    cshape = (batch, M, N) if A.dim() == 3 else (M, N)
    cdtype = torch.float32 if dtype == CYC_BF16_F32 else torch.int32
    if out is None:
        out = torch.empty(cshape, dtype=cdtype, device=A.device)
    elif tuple(out.shape) != cshape or out.dtype != cdtype or not out.is_contiguous() or out.device != A.device:
        raise ValueError("out has the wrong shape, dtype, layout or device")
    s = _stream_handle(A, stream)
    if batch == 1:
        args = A.data_ptr(), B.data_ptr(), out.data_ptr(), M, K, N, dtype
        st = cyc_recurrence_matmul_in(*args, 0, 0, s)
        if st == CYC_ERR_WORKSPACE:               # under capture: partial sums in memory of the graph's own
            wanted = cyc_matmul_workspace(*args)
            for size in (wanted, min(wanted, 16 << 20)):      # (what fewer slices need, where there is not all of it)
                work = _memory(size, A, stream) if size else None
                if work is not None:
                    st = cyc_recurrence_matmul_in(*args, work.data_ptr(), size, s)
                    break
            if st == CYC_ERR_WORKSPACE:
                st = cyc_recurrence_matmul(*args, s)
    else:
        st = cyc_recurrence_matmul_batched(A.data_ptr(), B.data_ptr(), out.data_ptr(), batch, M, K, N,
                                           M * K, K * N, M * N, dtype, s)
    if st != CYC_OK:
        raise CycError(st)
    return out


def cyc_recurrence_cholesky(A: int, L: int, Lh: int, n: int, nb: int, stream: int = 0) -> int:
    """Raw C-ABI call: device pointers as integers, returns the status code."""
    return int(_lib().cyc_recurrence_cholesky(A, L, Lh, n, nb, stream))


def cyc_cholesky_workspace(A: int, L: int, Lh: int, n: int, nb: int) -> int:
    """Bytes of workspace that cyc_recurrence_cholesky_in wants for this matrix."""
    return int(_lib().cyc_cholesky_workspace(A, L, Lh, n, nb))


def cyc_recurrence_cholesky_in(A: int, L: int, Lh: int, n: int, nb: int, workspace: int, workspace_bytes: int, stream: int = 0) -> int:
    """Raw call: device addresses as ints, returns the cyc_status."""
    return int(_lib().cyc_recurrence_cholesky_in(A, L, Lh, n, nb, workspace, workspace_bytes, stream))


def recurrence_cholesky(A, nb: int = 64, out=None, out_bf16=None, stream=None):
    """Tensor-level convenience: (L, Lh) with A = L L^T factored tile by tile (tiles of nb).

    A: (n,n) torch.float32 contiguous CUDA tensor, symmetric positive definite (its lower triangle is what counts).
    Allocates L (fp32, zero above the diagonal) and Lh (bf16, both triangles filled) unless given, and memory for
    the padded copy of an unaligned matrix or under stream capture, and forwards pointers to the C ABI on the
    current (or given) stream.  (Where that memory is not to be had an unaligned matrix is factored in place, more
    slowly and with other last bits.)
    """
    import torch
    if not A.is_cuda:
        raise ValueError("A must be a device tensor; there is no CPU path")
    if A.dtype != torch.float32 or A.dim() != 2 or A.shape[0] != A.shape[1] or not A.is_contiguous():
        raise ValueError(f"A must be a contiguous square float32 matrix, got {tuple(A.shape)} {A.dtype}")
    n = A.shape[0]
    if out is None:
        out = torch.empty((n, n), dtype=torch.float32, device=A.device)
    if out_bf16 is None:
        out_bf16 = torch.empty((n, n), dtype=torch.bfloat16, device=A.device)
    for t, dt in ((out, torch.float32), (out_bf16, torch.bfloat16)):
        if tuple(t.shape) != (n, n) or t.dtype != dt or not t.is_contiguous() or t.device != A.device:
            raise ValueError("out / out_bf16 has the wrong shape, dtype, layout or device")
    s = _stream_handle(A, stream)
    args = A.data_ptr(), out.data_ptr(), out_bf16.data_ptr(), n, nb
    st = cyc_recurrence_cholesky_in(*args, 0, 0, s)
    if st == CYC_ERR_WORKSPACE:                   # unaligned, or under capture: in memory that the caller brings
        wanted = cyc_cholesky_workspace(*args)
        work = _memory(wanted, A, stream) if wanted else None
        st = cyc_recurrence_cholesky(*args, s) if work is None else cyc_recurrence_cholesky_in(*args, work.data_ptr(), wanted, s)
    if st != CYC_OK:
        raise CycError(st)
    return out, out_bf16


def recurrence_trsm(L, B, nb: int = 64, out=None, out_bf16=None, stream=None):
    """Tensor-level convenience: (X, Xh) with L X = B solved tile by tile (tiles of nb rows).

    L: (n,n) torch.bfloat16, B: (n,nrhs) torch.float32, contiguous CUDA tensors.  Allocates X (fp32)
    and Xh (bf16) unless given, and memory for the padded copy of an unaligned system or under stream
    capture, and forwards pointers to the C ABI on the current (or given) stream.  (Where that memory is
    not to be had an unaligned system is solved in place, more slowly and with other last bits.)
    """
    import torch
    if not (L.is_cuda and B.is_cuda):
        raise ValueError("L and B must be device tensors; there is no CPU path")
    if L.dtype != torch.bfloat16 or B.dtype != torch.float32:
        raise ValueError("L must be bfloat16 and B float32")
    if L.dim() != 2 or B.dim() != 2 or L.shape[0] != L.shape[1] or B.shape[0] != L.shape[0]:
        raise ValueError(f"shape mismatch: L {tuple(L.shape)}, B {tuple(B.shape)}")
    if not (L.is_contiguous() and B.is_contiguous()):
        raise ValueError("L and B must be contiguous")
    n, nrhs = B.shape
    if out is None:
        out = torch.empty((n, nrhs), dtype=torch.float32, device=L.device)
    if out_bf16 is None:
        out_bf16 = torch.empty((n, nrhs), dtype=torch.bfloat16, device=L.device)
    for t, dt in ((out, torch.float32), (out_bf16, torch.bfloat16)):
        if tuple(t.shape) != (n, nrhs) or t.dtype != dt or not t.is_contiguous() or t.device != L.device:
            raise ValueError("out / out_bf16 has the wrong shape, dtype, layout or device")
    s = _stream_handle(L, stream)
    args = L.data_ptr(), B.data_ptr(), out.data_ptr(), out_bf16.data_ptr(), n, nrhs, nb
    st = cyc_recurrence_trsm_in(*args, 0, 0, s)
    if st == CYC_ERR_WORKSPACE:                   # unaligned, or under capture: in memory that the caller brings
        wanted = cyc_trsm_workspace(args[0], *args[2:])
        work = _memory(wanted, L, stream) if wanted else None
        st = cyc_recurrence_trsm(*args, s) if work is None else cyc_recurrence_trsm_in(*args, work.data_ptr(), wanted, s)
    if st != CYC_OK:
        raise CycError(st)
    return out, out_bf16


def recurrence_attention(Q, K, V, out=None, stream=None):
    """Tensor-level convenience: O = softmax(Q K^T / sqrt(d)) V by the tile recurrence.

    Q: (N,d) or (batch,N,d); K, V: (M,d) or (batch,M,d); contiguous torch.bfloat16 CUDA tensors, d 64 or 128.
    Allocates O (float32) unless given and forwards pointers to the C ABI on the current (or given) stream.
    """
    import torch
    if not (Q.is_cuda and K.is_cuda and V.is_cuda):
        raise ValueError("Q, K and V must be device tensors; there is no CPU path")
    if not (Q.dtype == K.dtype == V.dtype == torch.bfloat16):
        raise ValueError("Q, K and V must be bfloat16")
    if Q.dim() not in (2, 3) or K.dim() != Q.dim() or K.shape != V.shape or Q.shape[-1] != K.shape[-1]:
        raise ValueError(f"shape mismatch: Q {tuple(Q.shape)}, K {tuple(K.shape)}, V {tuple(V.shape)}")
    if Q.dim() == 3 and Q.shape[0] != K.shape[0]:
        raise ValueError("batch extents differ")
    if not (Q.is_contiguous() and K.is_contiguous() and V.is_contiguous()):
        raise ValueError("Q, K and V must be contiguous")
    batch = Q.shape[0] if Q.dim() == 3 else 1
    N, d = Q.shape[-2:]
    M = K.shape[-2]
    if out is None:
        out = torch.empty(tuple(Q.shape), dtype=torch.float32, device=Q.device)
    elif tuple(out.shape) != tuple(Q.shape) or out.dtype != torch.float32 or not out.is_contiguous() or out.device != Q.device:
        raise ValueError("out has the wrong shape, dtype, layout or device")
    s = _stream_handle(Q, stream)
    # The library splits no key list below 512.  Without memory the keys are not split, which is slower and adds the fp32 sums in
    # another order.
    wanted = cyc_attention_workspace(batch, N, M, d) if M >= 512 else 0
    work = _memory(wanted, Q, stream) if wanted else None
    if work is None:
        st = cyc_recurrence_attention(Q.data_ptr(), K.data_ptr(), V.data_ptr(), out.data_ptr(), batch, N, M, d, s)
    else:
        st = cyc_recurrence_attention_split(Q.data_ptr(), K.data_ptr(), V.data_ptr(), out.data_ptr(), batch, N, M, d, work.data_ptr(),
                                            wanted, s)
    if st != CYC_OK:
        raise CycError(st)
    return out
