"""Solves and factorisations whose rows are not 16-byte aligned, through copies that are: sizes one off a multiple of 8 and of a
tile, pointers off by one element, against the fp64 recurrences, with everything around the results untouched.

The bounds are those of tests/test_gpu_trsm.py and tests/test_gpu_cholesky.py: X (L) enters products rounded to bfloat16.
"""
import numpy as np
import pytest
import scipy.linalg
import torch

from datagen import ws_inputs
from helpers import bits_to_f64, torch_bf16_to_bits

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def guarded(shape, dtype, shift):
    """A tensor of this shape that starts `shift` elements past an aligned address, and the memory around it."""
    size = shape[0] * shape[1]
    around = torch.full((size + 64,), -77.0, dtype=dtype, device=DEV)
    return around[16 + shift:16 + shift + size].view(shape), around


def untouched(around, shift, size):
    return bool((around[:16 + shift] == -77.0).all()) and bool((around[16 + shift + size:] == -77.0).all())


@pytest.mark.parametrize("n,nrhs,shift", [(513, 8, 0), (519, 1, 0), (512, 61, 0), (577, 130, 0), (1333, 28, 1), (1024, 64, 1), (1087, 65, 3)])
def test_solve(n, nrhs, shift):
    import paper_2511_09987_amd as lib
    L, _ = guarded((n, n), torch.bfloat16, shift)
    L.copy_(ws_inputs.tri_lower_bf16(n, 50 + n, 0, DEV, upper=float("nan")))
    B, _ = guarded((n, nrhs), torch.float32, shift)
    B.copy_(ws_inputs.normal_f32((n, nrhs), 1.0, 50 + n, 1, DEV))
    X, Xa = guarded((n, nrhs), torch.float32, shift)
    Xh, Xha = guarded((n, nrhs), torch.bfloat16, shift)
    lib.recurrence_trsm(L, B, 64, out=X, out_bf16=Xh)
    assert untouched(Xa, shift, n * nrhs) and untouched(Xha, shift, n * nrhs)
    assert torch.equal(Xh, X.to(torch.bfloat16))
    L64 = np.tril(bits_to_f64(torch_bf16_to_bits(L)))
    ref = scipy.linalg.solve_triangular(L64, B.cpu().numpy().astype(np.float64), lower=True)
    Linv = scipy.linalg.solve_triangular(L64, np.eye(n), lower=True)
    skeel = float(np.max(np.sum(np.abs(Linv) @ np.abs(L64), axis=1)))
    assert np.max(np.abs(X.cpu().numpy() - ref)) <= 2.0 * 2.0 ** -9 * skeel * np.max(np.abs(ref))
    Xagain, _ = lib.recurrence_trsm(L, B, 64)
    assert torch.equal(X, Xagain)


@pytest.mark.parametrize("n,shift", [(129, 0), (191, 0), (193, 0), (585, 0), (1001, 1), (1033, 0), (1152, 1), (1280, 2)])
def test_factorisation(n, shift):
    import paper_2511_09987_amd as lib
    A, _ = guarded((n, n), torch.float32, shift)
    A.copy_(ws_inputs.spd_f32(n, 200 + n, 0, DEV))
    ref = np.linalg.cholesky(A.cpu().numpy().astype(np.float64))
    A[torch.triu(torch.ones(n, n, dtype=torch.bool, device=DEV), 1)] = float("nan")
    L, La = guarded((n, n), torch.float32, shift)
    Lh, Lha = guarded((n, n), torch.bfloat16, shift)
    lib.recurrence_cholesky(A, 64, out=L, out_bf16=Lh)
    assert untouched(La, shift, n * n) and untouched(Lha, shift, n * n)
    assert torch.equal(L, L.tril()) and torch.equal(Lh, Lh.t())
    assert torch.equal(Lh.tril(), L.to(torch.bfloat16))
    err = np.abs(L.cpu().numpy() - ref)
    scale = np.abs(ref).max()
    assert err.max() <= 4 * 2.0 ** -9 * scale and err.mean() <= 2.0 ** -12 * scale
    Lagain, _ = lib.recurrence_cholesky(A, 64)
    assert torch.equal(L, Lagain)


def test_under_capture():
    """On a stream without memory for the copies the calls take the direct way."""
    import paper_2511_09987_amd as lib
    n, nrhs = 777, 13
    L = ws_inputs.tri_lower_bf16(n, 50, 0, DEV)
    B = ws_inputs.normal_f32((n, nrhs), 1.0, 50, 1, DEV)
    want, _ = lib.recurrence_trsm(L, B, 64)
    stream = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        X, _ = lib.recurrence_trsm(L, B, 64)
    for _ in range(3):
        X.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert bool((X - want).abs().max() <= 2.0 ** -9 * want.abs().max())
