"""Small products with 16-byte aligned rows: blocks of 64 x 64, and of 32 x 32 with eight teams along k, against 64-bit sums.

int8 is exact.  bf16: products are exact in fp32 and every sum of K of them is rounded at most K times, each time by at most
2^-24 of the sum of the magnitudes.
"""
import pytest
import torch

from datagen import ws_inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (batch, M, K, N): one block and less; one past a block; fewer k-tiles than teams, one more, and a last k-tile of one chunk;
# blocks on every compute unit; batches
SHAPES = [(1, 16, 16, 16), (1, 64, 64, 64), (1, 65, 80, 32), (1, 33, 1024, 48), (1, 129, 1040, 272), (1, 48, 4080, 2048), (1, 511, 528, 496),
          (1, 1000, 400, 2000), (5, 100, 208, 112), (16, 64, 2048, 64), (2, 33, 4096, 2048), (3, 40, 6000, 1008)]


@pytest.mark.parametrize("dtype", (torch.bfloat16, torch.int8))
@pytest.mark.parametrize("batch,M,K,N", SHAPES)
def test_small_products(dtype, batch, M, K, N):
    import paper_2511_09987_amd as lib
    make = (lambda shape, t: ws_inputs.uniform_int(shape, 127, M + K, t, DEV)) if dtype == torch.int8 else \
        (lambda shape, t: ws_inputs.normal_bf16(shape, 1.0, M + K, t, DEV))
    A, B = make((batch, M, K), 0), make((batch, K, N), 1)
    guard = torch.full((batch * M * N + 64,), -77, dtype=torch.int32 if dtype == torch.int8 else torch.float32, device=DEV)
    C = guard[32:32 + batch * M * N].view(batch, M, N)
    lib.recurrence_matmul(A, B, out=C)
    assert bool((guard[:32] == -77).all()) and bool((guard[-32:] == -77).all())
    for b in range(batch):
        ref = torch.matmul(A[b].double(), B[b].double())
        if dtype == torch.int8:
            assert torch.equal(C[b].double(), ref)
        else:
            bound = K * 2.0 ** -24 * torch.matmul(A[b].double().abs(), B[b].double().abs())
            assert bool(((C[b].double() - ref).abs() <= bound).all())
    again = torch.empty_like(C)
    lib.recurrence_matmul(A, B, out=again)
    assert torch.equal(again.view(torch.int32), C.view(torch.int32))
