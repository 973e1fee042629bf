"""Products in blocks of 192 x 192, forced at their edges and as the dispatcher takes them, against 64-bit sums (int8 exact; bf16: K
roundings of 2^-24 of the sum of magnitudes at the most), with guard elements around the result."""
import pytest
import torch

from datagen import ws_inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (batch, M, K, N), K and N in 16-byte chunks: less than a block and a k-tile; whole blocks; one row and one chunk past and short of
# a block; one, two and three k-tiles and a last one of a single chunk; batches; and the size at which it is taken
SHAPES = [(1, 1, 1, 1), (1, 192, 16, 24), (1, 384, 24, 48), (1, 193, 17, 25), (1, 191, 9, 23), (1, 400, 8, 49), (2, 577, 41, 71), (3, 50, 33, 24)]

TAKEN = 0                             # 2944 columns of either type, which the dispatcher gives to these blocks


@pytest.mark.parametrize("dtype", (torch.bfloat16, torch.int8))
@pytest.mark.parametrize("batch,M,kc,nc", SHAPES + [(1, 2900, 40, TAKEN)])
def test_products(dtype, batch, M, kc, nc):
    import paper_2511_09987_amd as lib
    chunk = 16 if dtype == torch.int8 else 8
    K, N = kc * chunk, nc * chunk or 2944
    make = (lambda shape, t: ws_inputs.uniform_int(shape, 127, M + K, t, DEV)) if dtype == torch.int8 else \
        (lambda shape, t: ws_inputs.normal_bf16(shape, 1.0, M + K, t, DEV))
    A, B = make((batch, M, K), 0), make((batch, K, N), 1)
    guard = torch.full((batch * M * N + 64,), -77, dtype=torch.int32 if dtype == torch.int8 else torch.float32, device=DEV)
    C = guard[32:32 + batch * M * N].view(batch, M, N)
    ask = (A.data_ptr(), B.data_ptr(), C.data_ptr(), batch, M, K, N, M * K, K * N, M * N, lib.CYC_I8_I32 if dtype == torch.int8 else lib.CYC_BF16_F32)
    forced = (batch, M, kc, nc) in SHAPES
    assert lib.cyc_force_kernel("mfma192" if forced else None) == 0
    try:
        assert lib.cyc_kernel_variant(*ask) == "mfma192"
        lib.recurrence_matmul(A, B, out=C)
    finally:
        lib.cyc_force_kernel(None)
    assert bool((guard[:32] == -77).all()) and bool((guard[-32:] == -77).all())
    for b in range(batch):
        ref = torch.matmul(A[b].double(), B[b].double())
        if dtype == torch.int8:
            assert torch.equal(C[b].double(), ref)
        else:
            bound = K * 2.0 ** -24 * torch.matmul(A[b].double().abs(), B[b].double().abs())
            assert bool(((C[b].double() - ref).abs() <= bound).all())
