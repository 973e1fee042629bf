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


@pytest.mark.parametrize("bad", (float("inf"), float("-inf"), float("nan"), 3.0e38))
@pytest.mark.parametrize("n,nrhs", [(1333, 28), (1087, 65)])
def test_infinities_and_nans_spoil_no_row_above_them(n, nrhs, bad):
    """Row r of a column depends on the rows up to r: above the first bad right-hand side the solution is what it is without it (the
    tile of the bad row by substitution instead of through the inverse, so to the bounds of test_solve there, and to the
    bit in the tiles before and in all other columns), and from there on finite exactly where the direct way's is."""
    import paper_2511_09987_amd as lib
    L = ws_inputs.tri_lower_bf16(n, 50 + n, 0, DEV)
    B = ws_inputs.normal_f32((n, nrhs), 1.0, 50 + n, 1, DEV)
    clean, _ = lib.recurrence_trsm(L, B, 64)
    spots = {0: 0, 3: 1, 5: 31, 7: 32, 9: 63, 11: 64 + 17, 12: 5 * 64 + 40, 17: 8 * 64, 20: 10 * 64 + 63, 25: n - 30, nrhs - 1: n - 1}
    Bbad = B.clone()
    for col, row in spots.items():
        Bbad[row, col] = bad
    X, Xh = lib.recurrence_trsm(L, Bbad, 64)
    assert torch.equal(Xh.view(torch.int16)[X == X], X.to(torch.bfloat16).view(torch.int16)[X == X])
    direct, direct_h = torch.empty_like(X), torch.empty_like(Xh)
    assert lib.cyc_recurrence_trsm(L.data_ptr(), Bbad.data_ptr(), direct.data_ptr(), direct_h.data_ptr(), n, nrhs, 64,
                                   torch.cuda.current_stream().cuda_stream) == 0
    if bad != 3.0e38:                                          # (a large finite value overflows where its sums happen to)
        assert torch.equal(X.isfinite(), direct.isfinite())
    for col in range(nrhs):
        row = spots.get(col, n)
        tile = row // 64 * 64
        assert torch.equal(X[:tile, col], clean[:tile, col])
        assert bool(X[:row, col].isfinite().all())
        assert bool((X[tile:row, col] - clean[tile:row, col]).abs().le(2.0 ** -9 * clean.abs().max()).all())


@pytest.mark.parametrize("n,nrhs", [(777, 13), (776, 16)])
def test_under_capture(n, nrhs):
    """Captured solves and factorisations, aligned and not, have memory of their graph's own and give the eager call's bits: first
    calls on a stream, two graphs replayed on two streams at once, eager calls on the stream that they were captured on."""
    import paper_2511_09987_amd as lib
    stream, other = torch.cuda.Stream(), torch.cuda.Stream()
    sets = [(ws_inputs.tri_lower_bf16(n, 50 + i, 0, DEV), ws_inputs.normal_f32((n, nrhs), 1.0, 50 + i, 1, DEV), ws_inputs.spd_f32(n, 60 + i, 0, DEV))
            for i in range(2)]
    work = lambda L, B, A, **on: (*lib.recurrence_trsm(L, B, 64, **on), *lib.recurrence_cholesky(A, 64, **on))
    want = [work(*s) for s in sets]
    torch.cuda.synchronize()
    graphs, outs = [], []
    for s in sets:
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            outs.append(work(*s))
        graphs.append(graph)
    for _ in range(3):
        for out in outs:
            for t in out:
                t.zero_()
        torch.cuda.synchronize()
        for graph, on in zip(graphs, (stream, other)):
            with torch.cuda.stream(on):
                graph.replay()
        eager = work(*sets[0], stream=stream)
        torch.cuda.synchronize()
        for got, ref in ((outs[0], want[0]), (outs[1], want[1]), (eager, want[0])):
            assert all(torch.equal(g, r) for g, r in zip(got, ref))


def test_a_workspace_that_the_caller_brings():
    """Asked for, refused when too small, misaligned or overlapping, not written past; the plain entry points take none and give
    the direct way's bits whatever the workspaces of the library hold."""
    import paper_2511_09987_amd as lib
    n, nrhs = 777, 13
    L, B, A = ws_inputs.tri_lower_bf16(n, 50, 0, DEV), ws_inputs.normal_f32((n, nrhs), 1.0, 50, 1, DEV), ws_inputs.spd_f32(n, 60, 0, DEV)
    X, Xh = torch.zeros((n, nrhs), device=DEV), torch.zeros((n, nrhs), dtype=torch.bfloat16, device=DEV)
    F, Fh = torch.zeros((n, n), device=DEV), torch.zeros((n, n), dtype=torch.bfloat16, device=DEV)
    stream = torch.cuda.current_stream().cuda_stream
    trsm, chol = (L.data_ptr(), B.data_ptr(), X.data_ptr(), Xh.data_ptr(), n, nrhs, 64), (A.data_ptr(), F.data_ptr(), Fh.data_ptr(), n, 64)
    for call, args, wanted, results, tensor_level in (
            (lib.cyc_recurrence_trsm_in, trsm, lib.cyc_trsm_workspace(trsm[0], *trsm[2:]), (X, Xh), lambda: lib.recurrence_trsm(L, B, 64)),
            (lib.cyc_recurrence_cholesky_in, chol, lib.cyc_cholesky_workspace(*chol), (F, Fh), lambda: lib.recurrence_cholesky(A, 64))):
        around = torch.full((wanted + 4096,), 77, dtype=torch.uint8, device=DEV)
        assert wanted > 0 and call(*args, 0, 0, stream) == 6 and call(*args, around.data_ptr(), wanted - 1, stream) == 6
        assert call(*args, around.data_ptr() + 8, wanted, stream) == 2 and call(*args, args[0], wanted, stream) == 4
        torch.cuda.synchronize()
        assert bool((results[0] == 0).all()) and bool((around == 77).all())
        assert call(*args, around.data_ptr(), wanted, stream) == 0
        assert bool((around[wanted:] == 77).all()) and all(torch.equal(a, b) for a, b in zip(results, tensor_level()))
    for call, args, result in ((lib.cyc_recurrence_trsm, trsm, X), (lib.cyc_recurrence_cholesky, chol, F)):
        cold, warm = torch.cuda.Stream(), torch.cuda.current_stream()
        torch.cuda.synchronize()
        assert call(*args, cold.cuda_stream) == 0
        cold.synchronize()
        first = result.clone()
        lib.recurrence_cholesky(ws_inputs.spd_f32(1024, 60, 0, DEV), 64)             # the current stream has a workspace now
        assert call(*args, warm.cuda_stream) == 0
        assert torch.equal(result, first)


def test_sizes_that_need_no_copy_want_no_more_than_before():
    import paper_2511_09987_amd as lib
    at = 1 << 20
    assert lib.cyc_trsm_workspace(at, at, at, 511, 8, 64) == lib.cyc_trsm_workspace(at, at, at, 1001, 8, 32) == 0
    assert lib.cyc_trsm_workspace(at, at, at, 1024, 64, 64) == 16 * (64 * 64 * 4 + 56 * 1024 + 4)
    assert lib.cyc_trsm_workspace(at, at, at, 8191, 8191, 64) == 0 and lib.cyc_cholesky_workspace(at, at, at, 127, 64) == 0
