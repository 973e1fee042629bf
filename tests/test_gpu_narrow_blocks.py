"""Few columns of B against many rows of A in blocks of 32 rows, down to rows of B shorter than a 16-byte chunk."""
import pytest
import torch

from datagen import ws_inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (batch, M, K, N); rows of B of 1 element to a chunk and one more; one and two k-tiles; M past a block
SHAPES = [(1, 4096, 1024, 1), (1, 4097, 1040, 3), (2, 4100, 2048, 7), (1, 8192, 1024, 8), (1, 4096, 1072, 9), (3, 1400, 1024, 15), (1, 8192, 4096, 16),
          (1, 40, 144, 1), (1, 33, 80, 7), (2, 70, 208, 5)]


@pytest.mark.parametrize("dtype", (torch.bfloat16, torch.int8))
@pytest.mark.parametrize("batch,M,K,N", SHAPES)
def test_few_columns(dtype, batch, M, K, N):
    import paper_2511_09987_amd as lib
    make = (lambda s, i: ws_inputs.uniform_int(s, 127, M + K, i, DEV)) if dtype == torch.int8 else (lambda s, i: ws_inputs.normal_bf16(s, 1.0, M + K, i, DEV))
    A, B = make((batch, M, K), 0), make((batch, K, N), 1)
    # B between NaNs (the largest bytes): nothing of what lies around it may show
    size = batch * K * N
    around = torch.full((size + 64,), 127 if dtype == torch.int8 else float("nan"), dtype=dtype, device=DEV)
    inside = around[32:32 + size].view(batch, K, N)
    inside.copy_(B)
    C = lib.recurrence_matmul(A, inside)
    for a, b, c in zip(A, B, C):
        ref = torch.matmul(a.double(), b.double())
        if dtype == torch.int8:
            assert torch.equal(c.double(), ref)
        else:                                                   # K roundings of 2^-24 of the sum of magnitudes at the most
            assert bool(((c.double() - ref).abs() <= K * 2.0 ** -24 * torch.matmul(a.double().abs(), b.double().abs())).all())
