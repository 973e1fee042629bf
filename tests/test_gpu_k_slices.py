"""k in space over any number of k-slices, the last of them shorter, and few rows of A over a B of few columns."""
import pytest
import torch

from datagen import ws_inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def operands(dtype, batch, M, K, N):
    if dtype == torch.int8:
        return [ws_inputs.uniform_int((batch,) + s, 127, M + K, i, DEV) for i, s in enumerate(((M, K), (K, N)))]
    return [ws_inputs.normal_bf16((batch,) + s, 1.0, M + K, i, DEV) for i, s in enumerate(((M, K), (K, N)))]


# (batch, M, K, N): as many slices as fit; k-tiles that do not divide among them; a last k-tile of one 16-byte chunk; ragged
# blocks; then few rows (blocks of 32 columns, one and two to a compute unit; k in space; M below a block of MFMA rows)
SHAPES = [(1, 40, 17280, 784), (1, 130, 8640, 272), (1, 128, 4112, 128), (1, 300, 9232, 144), (1, 64, 65600, 64), (1, 18, 17280, 784),
          (1, 1, 17280, 256), (1, 20, 4000, 1008), (1, 16, 8192, 1024), (4, 32, 1040, 4096), (3, 5, 2048, 528), (1, 32, 2048, 8192)]


@pytest.mark.parametrize("dtype", (torch.bfloat16, torch.int8))
@pytest.mark.parametrize("batch,M,K,N", SHAPES)
def test_products(dtype, batch, M, K, N):
    import paper_2511_09987_amd as lib
    A, B = operands(dtype, batch, M, K, N)
    if batch == 1:
        A, B = A[0], B[0]
    C = lib.recurrence_matmul(A, B)
    assert torch.equal(C.view(torch.int32), lib.recurrence_matmul(A, B).view(torch.int32))
    for a, b, c in zip(A.view(batch, M, K), B.view(batch, K, N), C.view(batch, M, N)):
        ref = torch.matmul(a.double(), b.double())
        if dtype == torch.int8:
            assert torch.equal(c.double(), ref)
        else:                                                   # K roundings of 2^-24 of the sum of magnitudes at the most
            assert bool(((c.double() - ref).abs() <= K * 2.0 ** -24 * torch.matmul(a.double().abs(), b.double().abs())).all())


# slices in blocks of 256 x 256 (more than 19 k-tiles each, unequal, whole and ragged blocks, a ragged last k-tile) and in twice
# as many blocks of 128 x 128 (more than 27), on either side of both lines; slices start at different k-tiles of their range
@pytest.mark.parametrize("dtype", (torch.bfloat16, torch.int8))
@pytest.mark.parametrize("M,tiles,N,slices", [(512, 64 * 19, 512, 32), (512, 64 * 19 + 1, 512, 61), (1000, 16 * 23 + 5, 1008, 16), (64, 64 * 27, 1008, 32),
                                              (64, 64 * 28 - 3, 1008, 64), (128, 256 * 27 + 3, 128, 247), (130, 6 * 27 + 128, 784, 18)])
def test_long_slices(dtype, M, tiles, N, slices):
    import paper_2511_09987_amd as lib
    bke = 128 if dtype == torch.int8 else 64
    for K in (tiles * bke, tiles * bke - 16):
        A, B = (t[0] for t in operands(dtype, 1, M, K, N))
        C = lib.recurrence_matmul(A, B)
        assert lib.cyc_matmul_workspace(A.data_ptr(), B.data_ptr(), C.data_ptr(), M, K, N, lib.CYC_I8_I32 if dtype == torch.int8 else lib.CYC_BF16_F32) == 4 * slices * M * N, K
        assert torch.equal(C.view(torch.int32), lib.recurrence_matmul(A, B).view(torch.int32))
        ref = torch.matmul(A.double(), B.double())
        if dtype == torch.int8:
            assert torch.equal(C.double(), ref)
        else:                                                   # K roundings of 2^-24 of the sum of magnitudes at the most
            assert bool(((C.double() - ref).abs() <= K * 2.0 ** -24 * torch.matmul(A.double().abs(), B.double().abs())).all())


@pytest.mark.parametrize("M,K,N", [(18, 17280, 784), (40, 17280, 784), (256, 8192, 256)])
def test_captured_and_eager_calls_give_the_same_bits(M, K, N):
    """A captured product keeps its partial sums in memory of its graph's own: on a stream without a workspace and on one that has
    one, replayed on two streams at once and beside eager calls on the stream that it was captured on."""
    import paper_2511_09987_amd as lib
    stream, other = torch.cuda.Stream(), torch.cuda.Stream()
    sets = [[t[0] for t in operands(torch.bfloat16, 1, M, K, N + 16 * i)] for i in range(2)]
    want = [lib.recurrence_matmul(A, B) for A, B in sets]
    torch.cuda.synchronize()
    graphs, outs = [], []
    for A, B in sets:
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            outs.append(lib.recurrence_matmul(A, B))
        graphs.append(graph)
        with torch.cuda.stream(stream):
            lib.recurrence_matmul(A, B)
    for _ in range(4):
        for out in outs:
            out.zero_()
        torch.cuda.synchronize()
        for graph, s in zip(graphs, (stream, other)):
            with torch.cuda.stream(s):
                graph.replay()
        eager = lib.recurrence_matmul(*sets[0], stream=stream)
        torch.cuda.synchronize()
        assert torch.equal(outs[0], want[0]) and torch.equal(outs[1], want[1]) and torch.equal(eager, want[0])


@pytest.mark.parametrize("mode", ("global", "thread_local", "relaxed"))
def test_plain_entry_points_under_capture_on_a_fresh_stream(mode):
    """The per-stream workspace can be had under a capture of any mode; the bits are the eager call's."""
    import paper_2511_09987_amd as lib
    M, K, N, n, nrhs = 256, 8192, 256, 512, 64
    A, B = (t[0] for t in operands(torch.bfloat16, 1, M, K, N))
    L, R, S = ws_inputs.tri_lower_bf16(n, 50, 0, DEV), ws_inputs.normal_f32((n, nrhs), 1.0, 50, 1, DEV), ws_inputs.spd_f32(n, 60, 0, DEV)
    want = (lib.recurrence_matmul(A, B), *lib.recurrence_trsm(L, R, 64), *lib.recurrence_cholesky(S, 64))
    C, X, Xh, F, Fh = got = [torch.empty_like(t) for t in want]
    torch.cuda.synchronize()
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream, capture_error_mode=mode):
        assert lib.cyc_recurrence_matmul(A.data_ptr(), B.data_ptr(), C.data_ptr(), M, K, N, lib.CYC_BF16_F32, stream.cuda_stream) == 0
        assert lib.cyc_recurrence_trsm(L.data_ptr(), R.data_ptr(), X.data_ptr(), Xh.data_ptr(), n, nrhs, 64, stream.cuda_stream) == 0
        assert lib.cyc_recurrence_cholesky(S.data_ptr(), F.data_ptr(), Fh.data_ptr(), n, 64, stream.cuda_stream) == 0
    for _ in range(3):
        for t in got:
            t.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(g, w) for g, w in zip(got, want))


def test_a_workspace_that_the_caller_brings():
    """Refused when it is too small, misaligned or overlaps an operand; nothing past it is touched, and the bits are those of the
    library's own."""
    import paper_2511_09987_amd as lib
    M, K, N = 40, 17280, 784
    A, B = (t[0] for t in operands(torch.bfloat16, 1, M, K, N))
    C = torch.full((M, N), 5.0, device=DEV)
    args = A.data_ptr(), B.data_ptr(), C.data_ptr(), M, K, N, lib.CYC_BF16_F32
    wanted, stream = lib.cyc_matmul_workspace(*args), torch.cuda.current_stream().cuda_stream
    around = torch.full((wanted + 4096,), 77, dtype=torch.uint8, device=DEV)
    call = lambda work, size: lib.cyc_recurrence_matmul_in(*args, work, size, stream)
    assert wanted > 0 and call(around.data_ptr(), wanted - 1) == 6
    assert call(around.data_ptr() + 8, wanted) == 2 and call(A.data_ptr(), wanted) == 4
    torch.cuda.synchronize()
    assert bool((C == 5.0).all()) and bool((around == 77).all())
    assert call(around.data_ptr(), wanted) == 0
    assert torch.equal(C, lib.recurrence_matmul(A, B)) and bool((around[wanted:] == 77).all())
    for shape in ((512, 512, 512), (17, 33, 5), (16, 4096, 2048)):
        assert lib.cyc_matmul_workspace(A.data_ptr(), B.data_ptr(), C.data_ptr(), *shape, lib.CYC_BF16_F32) == 0


def test_first_call_on_a_stream_under_capture():
    """Captured products have memory of their own, whether or not the stream has a workspace, and whatever a later call needs."""
    import paper_2511_09987_amd as lib
    A, B = (t[0] for t in operands(torch.int8, 1, 64, 16384, 64))
    A2, B2 = (t[0] for t in operands(torch.int8, 1, 500, 32768, 496))
    want = torch.matmul(A.double(), B.double())
    stream = torch.cuda.Stream()
    cold, warm = torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(cold, stream=stream):
        C1 = lib.recurrence_matmul(A, B)
    with torch.cuda.stream(stream):
        lib.recurrence_matmul(A, B)
    torch.cuda.synchronize()
    with torch.cuda.graph(warm, stream=stream):
        C2 = lib.recurrence_matmul(A, B)
    with torch.cuda.stream(stream):
        C3 = lib.recurrence_matmul(A2, B2)                      # more slices of more elements
    for _ in range(3):
        C1.zero_()
        C2.zero_()
        cold.replay()
        warm.replay()
        torch.cuda.synchronize()
        assert torch.equal(C1.double(), want) and torch.equal(C2.double(), want)
    assert torch.equal(C3.double(), torch.matmul(A2.double(), B2.double()))


@pytest.mark.parametrize("dtype", (torch.bfloat16, torch.int8))
@pytest.mark.parametrize("M,K,N", [(1000, 24000, 1008), (512, 64 * 64 * 20 + 64, 512), (128, 64 * 64 * 28 - 16, 1024), (700, 96000, 528)])
def test_a_workspace_of_16_mib_takes_the_slices_that_fit(dtype, M, K, N):
    """Callers that bring the 16 MiB that slices of any length once needed at the most are served, by fewer of them; with no memory at
    all the call is refused."""
    import paper_2511_09987_amd as lib
    K *= 2 if dtype == torch.int8 else 1
    A, B = (t[0] for t in operands(dtype, 1, M, K, N))
    C = torch.full((M, N), 5, dtype=torch.int32 if dtype == torch.int8 else torch.float32, device=DEV)
    args = A.data_ptr(), B.data_ptr(), C.data_ptr(), M, K, N, lib.CYC_I8_I32 if dtype == torch.int8 else lib.CYC_BF16_F32
    size, stream = 16 << 20, torch.cuda.current_stream().cuda_stream
    assert lib.cyc_matmul_workspace(*args) > size
    around = torch.full((size + 4096,), 77, dtype=torch.uint8, device=DEV)
    assert lib.cyc_recurrence_matmul_in(*args, around.data_ptr(), 0, stream) == 6 and bool((C == 5).all())
    assert lib.cyc_recurrence_matmul_in(*args, around.data_ptr(), size, stream) == 0
    assert bool((around[size:] == 77).all())
    ref = torch.matmul(A.double(), B.double())
    if dtype == torch.int8:
        assert torch.equal(C.double(), ref)
    else:                                                       # K roundings of 2^-24 of the sum of magnitudes at the most
        assert bool(((C.double() - ref).abs() <= K * 2.0 ** -24 * torch.matmul(A.double().abs(), B.double().abs())).all())
