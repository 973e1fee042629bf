"""Products whose rows start at any byte address, on the matrix cores, against the CPU oracle.

Small-integer data: every sum is exact, so results are compared bit for bit.  Normal data: within K * 2^-23 of
sum |a||b|, what a correct fp32 accumulation of K terms stays below in any order.
"""
import numpy as np
import pytest
import torch

from datagen import ws_inputs
from helpers import bits_to_f64, rel_err, torch_bf16_to_bits

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

# rows and columns that end inside, at and just past the blocks of each of the four shapes (32 x 32, 64 x 64, 96 x 128,
# 256 x 128), with k extents around one 16-byte chunk, one k-tile (64 bf16, 128 int8) and one round of eight k-tiles
EXTENTS = [(1, 16), (33, 17), (31, 65), (64, 33), (1001, 1003), (961, 1025), (1501, 1403), (1345, 1409), (2047, 2049), (1793, 1921)]
KS = [16, 17, 63, 65, 127, 129, 193]
BLOCKS = ("uneven256", "uneven96", "uneven64", "uneven32")


@pytest.fixture(scope="module")
def lib():
    import paper_2511_09987_amd as pkg
    return pkg


def embedded(flat, offset, mode):
    """The elements of `flat` at an odd address inside a buffer whose other elements would be seen if they were used."""
    pad = torch.full((flat.numel() + offset + 64,), float("nan") if mode == "bf16" else 111, dtype=flat.dtype, device=DEV)
    pad[offset:offset + flat.numel()] = flat.reshape(-1)
    return pad, pad.data_ptr() + offset * flat.element_size()


def product(lib, mode, A, B, M, K, N, offset):
    keepA, pa = embedded(A, offset, mode)
    keepB, pb = embedded(B, offset, mode)
    C = torch.full((M * N + 32,), -7, dtype=torch.int32 if mode == "i8" else torch.float32, device=DEV)
    dt = lib.CYC_I8_I32 if mode == "i8" else lib.CYC_BF16_F32
    assert lib.cyc_kernel_name(pa, pb, C.data_ptr(), 1, M, K, N, 0, 0, 0, dt) in ("generic",) + BLOCKS
    assert lib.cyc_kernel_variant(pa, pb, C.data_ptr(), 1, M, K, N, 0, 0, 0, dt) in BLOCKS, "not on the matrix cores"
    assert lib.cyc_recurrence_matmul(pa, pb, C.data_ptr(), M, K, N, dt, torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    assert torch.all(C[M * N:] == -7)
    return C[:M * N].view(M, N).cpu().numpy()


@pytest.mark.parametrize("mode", ("i8", "bf16"))
@pytest.mark.parametrize("M,N", EXTENTS)
def test_any_alignment(lib, oracle, mode, M, N):
    for n, K in enumerate(KS if M < 1000 else KS[M % 3::3]):
        if mode == "i8":
            A, B = ws_inputs.uniform_int((M, K), 127, 50 + n, 0, DEV), ws_inputs.uniform_int((K, N), 127, 50 + n, 1, DEV)
            Ah, Bh = A.cpu().numpy(), B.cpu().numpy()
        else:
            A, B = ws_inputs.small_int_bf16((M, K), 8, 50 + n, 0, DEV), ws_inputs.small_int_bf16((K, N), 8, 50 + n, 1, DEV)
            Ah, Bh = torch_bf16_to_bits(A), torch_bf16_to_bits(B)
        C = product(lib, mode, A, B, M, K, N, 1 + n % 3)
        assert np.array_equal(C, oracle.ws_rowchain(Ah, Bh, mode)), (M, K, N)


@pytest.mark.parametrize("mode", ("i8", "bf16"))
@pytest.mark.parametrize("block", BLOCKS)
def test_every_block_at_its_edges(lib, oracle, mode, block):
    """Each block shape whatever the dispatcher would choose: one short of, at and one past a block and a pair of blocks."""
    rows = int(block[6:])
    cols = {256: 128, 96: 128, 64: 64, 32: 32}[rows]
    assert lib.cyc_force_kernel(block) == 0
    try:
        for n, (M, N, K) in enumerate([(rows - 1, cols + 1, 65), (rows, cols, 128), (rows + 1, cols - 1, 17), (2 * rows + 1, 2 * cols + 1, 129),
                                       (1, 16, 193), (3 * rows, cols + 3, 1025)]):
            make = (lambda s, t: ws_inputs.uniform_int(s, 127, 60 + n, t, DEV)) if mode == "i8" else (lambda s, t: ws_inputs.small_int_bf16(s, 8, 60 + n, t, DEV))
            A, B = make((M, K), 0), make((K, N), 1)
            h = [t.cpu().numpy() if mode == "i8" else torch_bf16_to_bits(t) for t in (A, B)]
            assert np.array_equal(product(lib, mode, A, B, M, K, N, n % 4), oracle.ws_rowchain(h[0], h[1], mode)), (M, K, N)
    finally:
        assert lib.cyc_force_kernel(None) == 0


@pytest.mark.parametrize("shape", [(1, 512, 512, 512), (1, 201, 203, 205), (1, 1500, 999, 1403), (2, 4096, 1024, 7), (1, 20, 4000, 1000), (3, 300, 520, 200)])
def test_forcing_the_variant_gives_the_same_bits(lib, shape):
    batch, M, K, N = shape
    A, B = ws_inputs.normal_bf16((batch, M, K), 1.0, 91, 0, DEV), ws_inputs.normal_bf16((batch, K, N), 1.0, 91, 1, DEV)
    own = lib.recurrence_matmul(A, B)
    variant = lib.cyc_kernel_variant(A.data_ptr(), B.data_ptr(), own.data_ptr(), batch, M, K, N, M * K, K * N, M * N, lib.CYC_BF16_F32)
    assert lib.cyc_force_kernel(variant) == 0
    try:
        assert torch.equal(lib.recurrence_matmul(A, B).view(torch.int32), own.view(torch.int32)), variant
    finally:
        assert lib.cyc_force_kernel(None) == 0


@pytest.mark.parametrize("M,K,N", [(74, 787, 27), (999, 515, 1001), (1501, 131, 1403), (2047, 67, 2049)])
def test_normal_data(lib, oracle, M, K, N):
    A, B = ws_inputs.normal_bf16((M, K), 1.0, 71, 0, DEV), ws_inputs.normal_bf16((K, N), 1.0, 71, 1, DEV)
    Ah, Bh = torch_bf16_to_bits(A), torch_bf16_to_bits(B)
    C = product(lib, "bf16", A, B, M, K, N, 1)
    assert rel_err(C, oracle.ws_rowchain(Ah, Bh, "bf16"), bits_to_f64(Ah), bits_to_f64(Bh)) <= K * 2.0 ** -23


@pytest.mark.parametrize("mode", ("i8", "bf16"))
def test_batch_at_odd_strides(lib, oracle, mode):
    b, M, K, N = 3, 50, 77, 39
    gen = (lambda s, t: ws_inputs.uniform_int(s, 127, 81, t, DEV)) if mode == "i8" else (lambda s, t: ws_inputs.small_int_bf16(s, 8, 81, t, DEV))
    A, B = gen((b, M, K), 0), gen((b, K, N), 1)
    C = lib.recurrence_matmul(A, B).cpu().numpy()
    for x in range(b):
        h = [t[x].cpu().numpy() if mode == "i8" else torch_bf16_to_bits(t[x].contiguous()) for t in (A, B)]
        assert np.array_equal(C[x], oracle.ws_rowchain(h[0], h[1], mode))
