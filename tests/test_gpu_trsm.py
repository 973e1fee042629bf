"""GPU parity of the tiled triangular solve (cyc_recurrence_trsm, through the C ABI) against the
CPU oracle (oracle/tri_oracle.c).

What can be compared how:
  * Integer systems (small-integer L with power-of-two diagonal, integer X, B = L X): every
    intermediate of any schedule is an exact integer, so X and Xh must match the oracle bit for bit.
  * Real data: inside a tile the library either runs the oracle's chain in the oracle's order (bit
    for bit the oracle's rows in the first tile) or, for tiles of 64 rows that its check finds well
    conditioned, multiplies by the tile's inverse in fp32, whose rows of the first tile agree with
    the oracle's within the fp32 bound of such a product, 64 * 2^-24 * (kappa^2 + kappa) max |X| with
    kappa = || |L_11^-1||L_11| ||_inf.  Later tiles go through GEMMs whose fp32 summation
    order differs from the oracle's tile-by-tile order; a last-bit difference can tip the bfloat16
    rounding of an X that later rows consume, so from the second tile on the two are compared
    against the bound both obey against the fp64 recurrence: 2 * 2^-9 * || |L^-1||L| ||_inf
    relative to max |X| (the bfloat16 rounding of X is the only error of that size).
"""
import os

import numpy as np
import pytest
import scipy.linalg
import torch

from datagen import ws_inputs
from helpers import bits_to_f64, to_bf16_bits, torch_bf16_to_bits

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def lib():
    import paper_2511_09987_amd as pkg
    assert os.path.exists(pkg.lib_path()), "libcyclotron_mm.so must be built in-tree"
    return pkg


@pytest.fixture(scope="module")
def tri():
    from oracle import tri_oracle
    return tri_oracle


def integer_system(n, nrhs, seed, density=0.2, device=DEV):
    """L (bf16), X_true (int64), B = L X_true (fp32, exact) on the device; see the pins for why
    such a system is exact in every arithmetic."""
    g = torch.Generator(device="cpu").manual_seed(seed)
    L = torch.randint(-1, 2, (n, n), generator=g) * (torch.rand((n, n), generator=g) < density)
    L = torch.tril(L, -1)
    d = torch.tensor([1, 2, -1, 4, -2])[torch.randint(0, 5, (n,), generator=g)]
    L = L + torch.diag(d)
    X = torch.randint(-8, 9, (n, nrhs), generator=g)
    L, X = L.to(device), X.to(device)
    B = (L.double() @ X.double())
    assert float(B.abs().max()) < 2 ** 20
    return L.to(torch.bfloat16), X, B.float()


SHAPES = [(64, 64, 64), (256, 128, 64), (1000, 72, 64), (1024, 512, 128), (520, 200, 32), (1032, 264, 8),
          (37, 5, 8), (130, 33, 16), (100, 40, 10), (1, 1, 64), (1, 70, 64), (200, 1, 64), (129, 64, 128),
          # panels of 5, 7, 8 tiles, 9 = 5 + 4 and 13 = 7 + 6 tiles in the four-wave kernel (nrhs a multiple of 8, the
          # last slab partly filled); 3 and 6 tiles in the one-wave kernel (nrhs not a multiple of 8)
          (320, 72, 64), (448, 136, 64), (512, 64, 64), (576, 80, 64), (832, 200, 64), (192, 70, 64), (384, 61, 64),
          # 16 and 32 tiles: two and four full panels with the smallest products between them, a partly filled last slab
          (1024, 72, 64), (1024, 200, 64), (2048, 40, 64)]


@pytest.mark.parametrize("n,nrhs,nb", SHAPES)
def test_integer_systems_bit_exact(lib, tri, n, nrhs, nb):
    L, Xtrue, B = integer_system(n, nrhs, seed=1000 + n + nb)
    X, Xh = lib.recurrence_trsm(L, B, nb)
    torch.cuda.synchronize()
    Xo, Xho = tri.tri_tiled(torch_bf16_to_bits(L), B.cpu().numpy(), nb)
    assert np.array_equal(Xo, Xtrue.cpu().numpy().astype(np.float32)), "the oracle itself must be exact here"
    assert np.array_equal(X.cpu().numpy(), Xo), f"{int((X.cpu().numpy() != Xo).sum())} elements of X differ"
    assert np.array_equal(torch_bf16_to_bits(Xh), Xho)


def skeel(L64):
    Linv = scipy.linalg.solve_triangular(L64, np.eye(L64.shape[0]), lower=True)
    return float(np.max(np.sum(np.abs(Linv) @ np.abs(np.tril(L64)), axis=1)))


@pytest.mark.parametrize("n,nrhs,nb", [(512, 256, 64), (1024, 512, 128), (300, 100, 32), (1000, 136, 64), (77, 19, 16),
                                       (448, 72, 64), (576, 264, 64), (384, 70, 64),
                                       (1024, 264, 64), (1024, 40, 64), (2048, 72, 64)])   # full panels through the inverses with products between them
def test_real_data_against_oracle(lib, tri, n, nrhs, nb):
    L = ws_inputs.tri_lower_bf16(n, 50 + n, 0, DEV, upper=float("nan"))     # NaN above the diagonal: never read
    B = ws_inputs.normal_f32((n, nrhs), 1.0, 50 + n, 1, DEV)
    X, Xh = lib.recurrence_trsm(L, B, nb)
    torch.cuda.synchronize()
    X, Xh = X.cpu().numpy(), torch_bf16_to_bits(Xh)
    bits = torch_bf16_to_bits(L)
    Xo, Xho = tri.tri_tiled(bits, B.cpu().numpy(), nb)
    assert np.all(np.isfinite(X))
    first = min(nb, n)
    L64 = np.tril(bits_to_f64(bits))
    if not np.array_equal(X[:first], Xo[:first]):
        # only the product with the inverse may differ from the oracle's chain inside a tile, and only this much
        assert nb == 64 and n >= 64 and nrhs % 8 == 0, "this shape is solved by substitution: first tile must match bitwise"
        kappa = skeel(L64[:first, :first])
        assert np.max(np.abs(X[:first] - Xo[:first])) <= 64 * 2.0 ** -24 * (kappa * kappa + kappa) * np.max(np.abs(Xo[:first]))
    else:
        assert np.array_equal(Xh[:first], Xho[:first])
    assert np.array_equal(Xh, to_bf16_bits(X)), "Xh must be X rounded to bfloat16"
    ref = tri.tri_scalar(L64, B.cpu().numpy())
    bound = 2.0 * 2.0 ** -9 * skeel(L64) * np.max(np.abs(ref))
    assert np.max(np.abs(X - ref)) <= bound
    assert np.max(np.abs(X - Xo)) <= bound
    # the bulk agrees far better than the bound: a tipped rounding is rare
    assert np.median(np.abs(X - Xo)) <= 2.0 ** -16 * np.max(np.abs(ref))


def test_two_calls_give_identical_bits_and_inputs_are_untouched(lib):
    n, nrhs, nb = 768, 320, 64
    L = ws_inputs.tri_lower_bf16(n, 7, 0, DEV)
    B = ws_inputs.normal_f32((n, nrhs), 1.0, 7, 1, DEV)
    L0, B0 = L.clone(), B.clone()
    X1, Xh1 = lib.recurrence_trsm(L, B, nb)
    X2, Xh2 = lib.recurrence_trsm(L, B, nb)
    torch.cuda.synchronize()
    assert torch.equal(X1, X2) and torch.equal(Xh1.view(torch.int16), Xh2.view(torch.int16))
    assert torch.equal(L.view(torch.int16), L0.view(torch.int16)) and torch.equal(B, B0)


def test_tile_size_changes_where_x_is_rounded(lib, tri):
    """The hand-worked rounding case of the pins, on the GPU: nb = 1 feeds the rounded X_0 to row 1,
    nb = 2 the unrounded one."""
    L = torch.tensor([[1.0, 0.0], [1.0, 1.0]], dtype=torch.bfloat16, device=DEV)
    B = torch.tensor([[1.0 + 2.0 ** -10], [0.0]], dtype=torch.float32, device=DEV)
    X, _ = lib.recurrence_trsm(L, B, 1)
    assert X.cpu().tolist() == [[1.0 + 2.0 ** -10], [-1.0]]
    X, Xh = lib.recurrence_trsm(L, B, 2)
    assert X.cpu().tolist() == [[1.0 + 2.0 ** -10], [-(1.0 + 2.0 ** -10)]]
    assert Xh.float().cpu().tolist() == [[1.0], [-1.0]]


def test_full_size_integer_system_and_sampled_columns(lib, tri):
    """n = nrhs = 8192 in the configuration the benchmark times: an integer system checked on every
    element, and real data checked on sampled columns (columns are independent, so the oracle can
    solve just those)."""
    n = nrhs = 8192
    nb = 64
    L, Xtrue, B = integer_system(n, nrhs, seed=4242, density=0.02)
    X, Xh = lib.recurrence_trsm(L, B, nb)
    torch.cuda.synchronize()
    assert torch.equal(X, Xtrue.float()), "integer system: X differs from the exact solution"
    assert torch.equal(Xh.float(), Xtrue.float())
    cols = [0, 1, 63, 64, 4095, 8191]
    Xo, _ = tri.tri_tiled(torch_bf16_to_bits(L), B[:, cols].cpu().numpy(), nb)
    assert np.array_equal(X[:, cols].cpu().numpy(), Xo)
    del L, Xtrue, B, X, Xh

    L = ws_inputs.tri_lower_bf16(n, 99, 0, DEV)
    B = ws_inputs.normal_f32((n, nrhs), 1.0, 99, 1, DEV)
    X, Xh = lib.recurrence_trsm(L, B, nb)
    torch.cuda.synchronize()
    cols = [0, 31, 64, 1000, 4097, 8191, 5555, 77]
    Bs = B[:, cols].cpu().numpy()
    bits = torch_bf16_to_bits(L)
    Xo, Xho = tri.tri_tiled(bits, Bs, nb)
    Xs = X[:, cols].cpu().numpy()
    L64 = np.tril(bits_to_f64(bits))
    # these diagonal tiles are well conditioned (diagonal in [1, 2), off-diagonal entries of size 0.006), so the first
    # tile is a product with its inverse in fp32: within that product's bound of the oracle's chain
    kappa = skeel(L64[:nb, :nb])
    assert kappa < 2.0
    assert np.max(np.abs(Xs[:nb] - Xo[:nb])) <= 64 * 2.0 ** -24 * (kappa * kappa + kappa) * np.max(np.abs(Xo[:nb]))
    ref = tri.tri_scalar(L64, Bs)
    # || |L^-1||L| ||_inf at this size, from the solve of |L| against its own row sums (L^-1 >= 0 is not
    # given, so take the bound from the sampled columns instead): compare both to fp64 and to each other
    scale = np.max(np.abs(ref))
    err_gpu, err_orc = np.max(np.abs(Xs - ref)) / scale, np.max(np.abs(Xo - ref)) / scale
    assert err_gpu <= 4.0 * max(err_orc, 2.0 ** -9), (err_gpu, err_orc)
    assert np.max(np.abs(Xs - Xo)) / scale <= 4.0 * max(err_orc, 2.0 ** -9)
    assert np.array_equal(torch_bf16_to_bits(Xh[:, cols]), to_bf16_bits(Xs))
    # and the system is solved: residual of the fp64 check on the sampled columns
    res = np.max(np.abs(L64 @ Xs.astype(np.float64) - Bs)) / (np.max(np.abs(Bs)) + scale)
    assert res <= 2.0 ** -7, res


def test_panels_with_ill_conditioned_tiles_fall_back_to_substitution(lib, tri):
    """Tiles of 64 rows are solved through their inverses only where the library's check finds them well conditioned;
    a panel (eight tiles) that holds one ill-conditioned diagonal tile is solved by substitution as a whole.  Here
    tile 2 of a well-conditioned L gets a unit lower-triangular block of ones (its inverse has entries up to 2^62):
    the rows of the first panel, substitution all through, match the oracle bit for bit up to the first GEMM, and
    the whole solve obeys the usual bound."""
    n, nrhs, nb = 1024, 136, 64
    L = ws_inputs.tri_lower_bf16(n, 321, 0, DEV)
    bad = torch.tril(torch.ones((64, 64), dtype=torch.bfloat16, device=DEV))
    L[128:192, 128:192] = bad
    B = ws_inputs.normal_f32((n, nrhs), 1.0, 321, 1, DEV)
    X, Xh = lib.recurrence_trsm(L, B, nb)
    torch.cuda.synchronize()
    X = X.cpu().numpy()
    bits = torch_bf16_to_bits(L)
    Xo, _ = tri.tri_tiled(bits, B.cpu().numpy(), nb)
    assert np.all(np.isfinite(X))
    assert np.array_equal(X[:64], Xo[:64]), "first tile of a panel solved by substitution must match bitwise"
    L64 = np.tril(bits_to_f64(bits))
    ref = tri.tri_scalar(L64, B.cpu().numpy())
    bound = 2.0 * 2.0 ** -9 * skeel(L64) * np.max(np.abs(ref))
    assert np.max(np.abs(X - ref)) <= bound and np.max(np.abs(X - Xo)) <= bound
    assert np.array_equal(torch_bf16_to_bits(Xh), to_bf16_bits(X))


def test_zero_on_the_diagonal_gives_ieee_infinities_not_an_error(lib):
    """A zero pivot makes the tile's inverse non-finite, which the library's check rejects: the tile is solved by
    substitution and the division by zero shows as IEEE infinities or NaNs from that row on, in that tile's columns."""
    n, nrhs, nb = 512, 64, 64
    L = ws_inputs.tri_lower_bf16(n, 77, 0, DEV)
    L[70, 70] = 0.0
    B = ws_inputs.normal_f32((n, nrhs), 1.0, 77, 1, DEV)
    X, _ = lib.recurrence_trsm(L, B, nb)
    torch.cuda.synchronize()
    X = X.cpu().numpy()
    assert np.all(np.isfinite(X[:70])), "rows before the zero pivot are unaffected"
    assert not np.any(np.isfinite(X[70])), "the row of the zero pivot is a division by zero in every column"


@pytest.mark.parametrize("n,nrhs,nb", [(62, 23, 64), (61, 70, 64), (32, 17, 32), (16, 64, 16), (13, 65, 16), (128, 80, 128), (100, 9, 128), (65, 64, 128)])
@pytest.mark.parametrize("case", ["plain", "negative", "large", "small", "tiny", "zeros"])
def test_quotients_from_reciprocals_are_the_divisions(lib, tri, n, nrhs, nb, case):
    """One tile on one launch: the quotients come from reciprocals of the diagonal where everything that comes out lies in
    [2^-50, 2^50] or is zero and the diagonal is positive, and from divisions elsewhere: bit for bit the oracle's chain on
    either side of that line (full tiles of 64 aligned rows have a kernel of their own, without reciprocals: see the next test)."""
    L = ws_inputs.tri_lower_bf16(n, 90 + n, 0, DEV)
    B = ws_inputs.normal_f32((n, nrhs), 1.0, 90 + n, 1, DEV)
    if case == "negative":
        L[:, ::3] *= -1
    elif case in ("large", "small"):
        B *= 2.0 ** (55 if case == "large" else -55)
    elif case == "tiny":
        L *= 2.0 ** -30
        L[n // 2] *= 2.0 ** -30
    elif case == "zeros":
        B[::2, ::3] = -0.0
        B[:, 1::3] = 0.0
        L.tril_()[:, 1::2] *= torch.eye(n, device=DEV, dtype=L.dtype)[:, 1::2]
    X, Xh = lib.recurrence_trsm(L, B, nb)
    torch.cuda.synchronize()
    Xo, Xho = tri.tri_tiled(torch_bf16_to_bits(L), B.cpu().numpy(), nb)
    assert np.all(np.isfinite(Xo))
    assert np.array_equal(X.cpu().numpy().view(np.int32), Xo.astype(np.float32).view(np.int32))
    assert np.array_equal(torch_bf16_to_bits(Xh), Xho)


@pytest.mark.parametrize("case", ["plain", "negative", "large", "small", "tiny", "zeros"])
def test_quotients_in_a_full_tile_at_an_unaligned_address(lib, tri, case):
    """The same for a tile of 64 rows: at an address that is no multiple of 16 bytes, through the entry point that makes no copy."""
    n, nrhs = 64, 24
    L = ws_inputs.tri_lower_bf16(n, 190, 0, DEV)
    B = ws_inputs.normal_f32((n, nrhs), 1.0, 190, 1, DEV)
    if case == "negative":
        L[:, ::3] *= -1
    elif case in ("large", "small"):
        B *= 2.0 ** (55 if case == "large" else -55)
    elif case == "tiny":
        L *= 2.0 ** -30
        L[n // 2] *= 2.0 ** -30
    elif case == "zeros":
        B[::2, ::3] = -0.0
        B[:, 1::3] = 0.0
    at = torch.empty(n * n + 8, dtype=torch.bfloat16, device=DEV)[1:1 + n * n].view(n, n)
    at.copy_(L)
    assert at.data_ptr() % 16 == 2
    X, Xh = torch.empty_like(B), torch.empty((n, nrhs), dtype=torch.bfloat16, device=DEV)
    assert lib.cyc_recurrence_trsm(at.data_ptr(), B.data_ptr(), X.data_ptr(), Xh.data_ptr(), n, nrhs, 64, torch.cuda.current_stream().cuda_stream) == 0
    Xo, Xho = tri.tri_tiled(torch_bf16_to_bits(L), B.cpu().numpy(), 64)
    assert np.array_equal(X.cpu().numpy().view(np.int32), Xo.astype(np.float32).view(np.int32))
    assert np.array_equal(torch_bf16_to_bits(Xh), Xho)


@pytest.mark.parametrize("n,nrhs", [(512, 64), (1024, 136)])
def test_the_inverse_by_divisions_is_the_one_by_reciprocals(lib, n, nrhs):
    """A negative diagonal entry sends the inverse of its tile to the pass with divisions, which has to be the same inverse up to
    signs, and used: every second column of L and row of X negated leaves the other rows of X as they were, in every bit."""
    L = ws_inputs.tri_lower_bf16(n, 191, 0, DEV)
    B = ws_inputs.normal_f32((n, nrhs), 1.0, 191, 1, DEV)
    X, Xh = lib.recurrence_trsm(L, B, 64)
    signs = torch.ones(n, device=DEV)
    signs[::2] = -1
    Xs, Xhs = lib.recurrence_trsm(L * signs.to(L.dtype)[None, :], B, 64)
    assert torch.equal(Xs, X * signs[:, None]) and torch.equal(Xhs.float(), Xh.float() * signs[:, None])
    # (the product with the inverse, not the chain: that differs from it in last bits)
    bad = L.clone()
    bad[:64, :64] = torch.tril(torch.ones((64, 64), dtype=L.dtype, device=DEV))
    Xb, _ = lib.recurrence_trsm(bad, torch.cat((bad[:64, :64].float() @ X[:64], B[64:])).contiguous(), 64)
    assert bool(torch.isfinite(Xb).all()) and not torch.equal(Xb[64:128], X[64:128])


@pytest.mark.parametrize("n,nb", [(64, 64), (61, 64), (30, 32), (16, 16), (128, 128)])
@pytest.mark.parametrize("divisor,result", [(0, -70), (0, -90), (0, -115), (-23, -74), (-26, -60), (-45, -55), (30, -60)])
def test_small_results_are_the_divisions(lib, tri, n, nb, divisor, result):
    """Results below 2^-50 with a diagonal above and below 2^-24 (powers of two: divisor, result), either side of the lines between
    quotients from reciprocals and divisions: bit for bit the oracle's chain.  At an unaligned address, without a copy."""
    nrhs = 40
    L = ws_inputs.tri_lower_bf16(n, 290 + n, 0, DEV) * 2.0 ** divisor
    B = ws_inputs.normal_f32((n, nrhs), 1.0, 290 + n, 1, DEV)
    B = torch.where(torch.arange(nrhs, device=DEV)[None, :] % 2 == 0, B, B * 2.0 ** 10) * 2.0 ** (divisor + result)
    at = torch.empty(n * n + 8, dtype=torch.bfloat16, device=DEV)[1:1 + n * n].view(n, n)
    at.copy_(L)
    X, Xh = torch.empty_like(B), torch.empty((n, nrhs), dtype=torch.bfloat16, device=DEV)
    assert lib.cyc_recurrence_trsm(at.data_ptr(), B.data_ptr(), X.data_ptr(), Xh.data_ptr(), n, nrhs, nb, torch.cuda.current_stream().cuda_stream) == 0
    Xo, Xho = tri.tri_tiled(torch_bf16_to_bits(at), B.cpu().numpy(), nb)
    assert np.array_equal(X.cpu().numpy().view(np.int32), Xo.astype(np.float32).view(np.int32))
    assert np.array_equal(torch_bf16_to_bits(Xh), Xho)


@pytest.mark.parametrize("case", ["negative", "small"])
def test_signs_and_small_results_do_not_double_the_time(lib, case):
    """A diagonal with negative entries goes to divisions without a pass of quotients before them, and results down to 2^-76 to one
    pass of quotients alone: sixteen tiles one after the other, at an unaligned address and without a copy.  1.07 and 1.03 times the time
    of the plain system, 1.29 and 1.26 with two passes."""
    n, nrhs = 1024, 24
    L = ws_inputs.tri_lower_bf16(n, 390, 0, DEV)
    B = ws_inputs.normal_f32((n, nrhs), 1.0, 390, 1, DEV)
    signs = torch.where(torch.arange(n, device=DEV) % 3 == 0, -1.0, 1.0).to(L.dtype)
    plain, other = (torch.empty(n * n + 8, dtype=torch.bfloat16, device=DEV)[1:1 + n * n].view(n, n) for _ in range(2))
    plain.copy_(L)
    other.copy_(L * signs[None, :] if case == "negative" else L)
    Bo = B * 2.0 ** -58 if case == "small" else B
    X, Xh = torch.empty_like(B), torch.empty((n, nrhs), dtype=torch.bfloat16, device=DEV)
    stream = torch.cuda.current_stream().cuda_stream

    def time(L, B):
        begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        begin.record()
        for _ in range(20):
            assert lib.cyc_recurrence_trsm(L.data_ptr(), B.data_ptr(), X.data_ptr(), Xh.data_ptr(), n, nrhs, 64, stream) == 0
        end.record()
        end.synchronize()
        return begin.elapsed_time(end)
    time(plain, B), time(other, Bo)
    pairs = [(time(plain, B), time(other, Bo)) for _ in range(9)]
    assert sorted(b / a for a, b in pairs)[4] < 1.18
