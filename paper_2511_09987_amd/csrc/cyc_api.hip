// cyc_api.hip -- the C ABI declared in include/cyclotron_mm.h: argument checks and
// the choice of kernel.  No device work happens here except the launches.
#include "../../include/cyclotron_mm.h"
#include "cyc_internal.h"

#include <cstdlib>
#include <cstring>
#include <atomic>

namespace {

constexpr int64_t kMaxElems = (int64_t)1 << 46;   // keeps every byte offset far inside int64

bool mul_ok(int64_t a, int64_t b, int64_t *out)
{
    if (a == 0 || b == 0) { *out = 0; return true; }
    if (a > kMaxElems / b) return false;
    *out = a * b;
    return true;
}

bool overlaps(const void *p, int64_t pbytes, const void *q, int64_t qbytes)
{
    if (!p || !q || pbytes <= 0 || qbytes <= 0) return false;
    uintptr_t a = (uintptr_t)p, b = (uintptr_t)q;
    return a < b + (uintptr_t)qbytes && b < a + (uintptr_t)pbytes;
}

// what a caller may bring as a workspace
bool workspace_ok(const void *workspace, int64_t bytes) { return ((uintptr_t)workspace & 15) == 0 && bytes >= 0; }

enum Kernel { K_NONE, K_ZERO, K_GENERIC, K_UNEVEN256, K_UNEVEN96, K_UNEVEN64, K_UNEVEN32, K_MFMA256, K_MFMA192, K_MFMA128, K_MFMA256X32, K_MFMA128X32, K_MFMAK, K_NARROW, K_NARROWM };

const char *kernel_label(Kernel k)
{
    switch (k) {
        case K_NONE: return "none";
        case K_ZERO: return "zero";
        case K_GENERIC: return "generic";
        case K_UNEVEN256: return "uneven256";
        case K_UNEVEN96: return "uneven96";
        case K_UNEVEN64: return "uneven64";
        case K_UNEVEN32: return "uneven32";
        case K_MFMA256: return "mfma256";
        case K_MFMA192: return "mfma192";
        case K_MFMA128: return "mfma128";
        case K_MFMA256X32: return "mfma256x32";
        case K_MFMA128X32: return "mfma128x32";
        case K_MFMAK: return "mfmak";
        case K_NARROW: return "narrow";
        case K_NARROWM: return "narrowm";
    }
    return "none";
}

Kernel uneven_kernel(int block) { return block == 256 ? K_UNEVEN256 : block == 96 ? K_UNEVEN96 : block == 64 ? K_UNEVEN64 : K_UNEVEN32; }
int uneven_block(Kernel k) { return k == K_UNEVEN256 ? 256 : k == K_UNEVEN96 ? 96 : k == K_UNEVEN64 ? 64 : 32; }

// The kernel forced by cyc_force_kernel(), or by the environment variable CYC_FORCE_KERNEL, which is read once
// (at the first call that gets as far as choosing a kernel) as the initial value.  K_NONE: the dispatcher decides.
Kernel kernel_by_name(const char *name)
{
    if (!name) return K_NONE;
    for (Kernel k : {K_GENERIC, K_UNEVEN256, K_UNEVEN96, K_UNEVEN64, K_UNEVEN32, K_MFMA256, K_MFMA192, K_MFMA128, K_MFMA256X32, K_MFMA128X32, K_MFMAK, K_NARROW, K_NARROWM})
        if (!std::strcmp(name, kernel_label(k))) return k;
    return K_NONE;
}
std::atomic<int> &forced_kernel()
{
    static std::atomic<int> forced{(int)kernel_by_name(std::getenv("CYC_FORCE_KERNEL"))};
    return forced;
}

std::atomic<int> &wait_limit_value()
{
    static std::atomic<int> v{1 << 20};
    return v;
}

// Validates and fills `p`.  Returns CYC_OK with *k == K_NONE when there is nothing to do.  *family: the kernel whose part of
// the dispatch the problem falls into; *k: the kernel that runs (blocks of cyc_uneven.hip stand in for several families).
// split: filled in for K_MFMAK; any_slices: k may be cut into slices of any number and length (see KSplit), which the entry points
// without a workspace argument do not do; memory: what there is for them (choose_ksplit).
constexpr int64_t UNLIMITED = INT64_MAX;
int plan(const void *A, const void *B, const void *C, int64_t batch, int64_t M, int64_t K, int64_t N,
         int64_t strideA, int64_t strideB, int64_t strideC, int dtype, cyc::Problem *p, Kernel *k, Kernel *family, cyc::KSplit *split, bool any_slices,
         int64_t memory = UNLIMITED)
{
    *k = *family = K_NONE;
    if (dtype != CYC_BF16_F32 && dtype != CYC_I8_I32) return CYC_ERR_DTYPE;
    if (batch < 0 || M < 0 || K < 0 || N < 0 || strideA < 0 || strideB < 0 || strideC < 0) return CYC_ERR_SHAPE;
    int64_t mk, kn, mn;
    if (!mul_ok(M, K, &mk) || !mul_ok(K, N, &kn) || !mul_ok(M, N, &mn)) return CYC_ERR_SHAPE;
    if (batch > 1) {
        int64_t t;
        if (strideC < mn) return CYC_ERR_SHAPE;
        if (!mul_ok(batch, strideA > mk ? strideA : mk, &t) || !mul_ok(batch, strideB > kn ? strideB : kn, &t) ||
            !mul_ok(batch, strideC, &t))
            return CYC_ERR_SHAPE;
        if ((strideA != 0 && strideA < mk) || (strideB != 0 && strideB < kn)) return CYC_ERR_SHAPE;
    }
    if (batch == 0 || M == 0 || N == 0) return CYC_OK;
    if (!C) return CYC_ERR_NULL;
    if (K > 0 && (!A || !B)) return CYC_ERR_NULL;

    const bool i8 = dtype == CYC_I8_I32;
    const int64_t es = i8 ? 1 : 2;
    const int64_t spanA = ((batch - 1) * strideA + mk) * es, spanB = ((batch - 1) * strideB + kn) * es;
    const int64_t spanC = ((batch - 1) * strideC + mn) * 4;
    if (K > 0 && (overlaps(C, spanC, A, spanA) || overlaps(C, spanC, B, spanB))) return CYC_ERR_ALIAS;

    p->A = A; p->B = B; p->C = const_cast<void *>(C);
    p->batch = batch; p->M = M; p->K = K; p->N = N;
    p->strideA = strideA; p->strideB = strideB; p->strideC = strideC;
    p->i8 = i8;

    auto take = [&](Kernel f, Kernel kernel) { *family = f; *k = kernel; return CYC_OK; };
    if (K == 0) return take(K_ZERO, K_ZERO);

    // a forced kernel overrides the heuristic when it supports the problem (testing and benchmarking aid).  The x32
    // names are the MFMA kernels built on the 32x32 instruction shape, which the dispatcher never picks by itself.
    const Kernel force = (Kernel)forced_kernel().load(std::memory_order_relaxed);
    auto splits = [&]() { return (*split = cyc::choose_ksplit(*p, any_slices, memory)).slices > 1; };
    switch (force) {
        case K_GENERIC: return take(force, force);
        case K_UNEVEN256: case K_UNEVEN96: case K_UNEVEN64: case K_UNEVEN32: if (cyc::supports_uneven(*p)) return take(force, force); break;
        case K_MFMA256: case K_MFMA256X32: if (cyc::supports_mfma(*p, 256)) return take(force, force); break;
        case K_MFMA192: if (cyc::supports_mfma(*p, 192)) return take(K_MFMA256, force); break;
        case K_MFMA128: case K_MFMA128X32: if (cyc::supports_mfma(*p, 128)) return take(force, force); break;
        case K_NARROW: if (cyc::supports_narrow(*p)) return take(force, force); break;
        case K_NARROWM: if (cyc::supports_narrowm(*p)) return take(force, force); break;
        case K_MFMAK: if (splits()) return take(force, force); break;
        default: break;
    }
    if (cyc::prefers_narrow(*p)) {
        // Its workgroups keep all of B in registers, which they fill before they stream: up to 512 blocks of 32 rows with eight
        // teams along k are done before that has paid (bf16, microseconds there / in blocks: 4096 x 2048 x 8 18.8 / 9.3,
        // 4100 x 1024 x 3 15.1 / 9.6, 4 x 4096 x 3000 x 16 23.9 / 21.6, i8 2 x 8192 x 8192 x 16 26.0 / 25.5); with more blocks (i8
        // 8 x 4096 x 4096 x 1 33.6 / 36.0) and past 128 MiB of A (2 x 8192 x 8192 x 16 48.7 / 49.7) it streams better
        const int64_t blocks = p->batch * ((p->M + 31) / 32), bytes = p->batch * mk * es;
        return take(K_NARROW, force == K_NONE && blocks <= 512 && bytes <= (128 << 20) && cyc::supports_uneven(*p) ? K_UNEVEN32 : K_NARROW);
    }
    if (cyc::prefers_narrowm(*p)) {
        // past 128 k-tiles k goes to space across workgroups (bf16 32 x 17280 x 784 144 us there, 39 in blocks, 17 so)
        const int64_t kt = p->K * es / 128;
        if (force == K_NONE && any_slices && kt > 128 && p->N <= 4096 && splits()) return take(K_MFMAK, K_MFMAK);
        return take(K_NARROWM, force == K_NONE && cyc::blocks_beat_narrowm(*p) && cyc::supports_uneven(*p) ? K_UNEVEN32 : K_NARROWM);
    }
    // few output blocks, long k: k goes to space (see choose_ksplit)
    if (force == K_NONE && splits()) return take(K_MFMAK, K_MFMAK);
    // MFMA kernels for everything with 16-byte aligned rows except slivers
    const int tile = cyc::choose_mfma_tile(*p);
    if (tile >= 192) return take(K_MFMA256, tile == 192 && force == K_NONE ? K_MFMA192 : K_MFMA256);
    if (tile == 128) {
        const int block = force == K_NONE ? cyc::choose_small_block(*p) : 0;
        return take(K_MFMA128, block ? uneven_kernel(block) : K_MFMA128);
    }
    // (thousands of tiny bf16 grids with a single k slab are bound by starting workgroups, which the vector-ALU kernel does with
    // less: 12000 x (20 x 9 x 20) 44 us there, 51 in blocks of 64; 60000 x (9 x 9 x 9) 166 / 191; 3000 x (9 x 9 x 9) 12.2 / 11.0)
    const bool tiny = !p->i8 && p->K <= 16 && p->M <= 32 && p->N <= 32 && p->batch >= 8192;
    return take(K_GENERIC, cyc::supports_uneven(*p) && !tiny ? uneven_kernel(cyc::choose_uneven_block(*p)) : K_GENERIC);
}

int run_chunk(const cyc::Problem &p, Kernel k, const cyc::KSplit &split, void *workspace, hipStream_t s)
{
    hipError_t e = hipSuccess;
    switch (k) {
        case K_NONE: return CYC_OK;
        case K_ZERO: e = cyc::launch_zero(p, s); break;
        case K_GENERIC: e = cyc::launch_generic(p, s); break;
        case K_UNEVEN256: case K_UNEVEN96: case K_UNEVEN64: case K_UNEVEN32: e = cyc::launch_uneven(p, uneven_block(k), s); break;
        case K_MFMA256: e = cyc::launch_mfma(p, 256, 16, s); break;
        case K_MFMA192: e = cyc::launch_mfma(p, 192, 16, s); break;
        case K_MFMA128: e = cyc::launch_mfma(p, 128, 16, s); break;
        case K_MFMA256X32: e = cyc::launch_mfma(p, 256, 32, s); break;
        case K_MFMA128X32: e = cyc::launch_mfma(p, 128, 32, s); break;
        case K_MFMAK: e = cyc::launch_mfma_ksplit(p, split, workspace, s); break;
        case K_NARROW: e = cyc::launch_narrow(p, s); break;
        case K_NARROWM: e = cyc::launch_narrowm(p, s); break;
    }
    return e == hipSuccess ? CYC_OK : CYC_ERR_LAUNCH;
}

// A grid's y extent ends at 65535, which is where a launch's share of the batch ends: longer batches take several
// launches of the same kernel (batch elements are independent).
constexpr int64_t kBatchPerLaunch = 65535;

// where the partial products of K_MFMAK go
enum Memory { CACHED, FIXED, GIVEN };    // the per-stream workspace, the library's fixed array, the caller's

int run(const cyc::Problem &p, Kernel k, const cyc::KSplit &split, hipStream_t s, Memory memory, void *given = nullptr, int64_t given_bytes = 0)
{
    void *workspace = nullptr;
    cyc::WorkspaceHold hold;
    if (k == K_MFMAK) {
        // everything that can fail before the first launch is settled before it
        const int64_t need = cyc::ksplit_workspace_bytes(p, split.slices);
        int64_t have = 0;
        if (memory == FIXED) workspace = cyc::static_workspace(&have);
        else if (memory == GIVEN) workspace = given, have = given_bytes;
        else workspace = hold.acquire(s, need), have = need;
        if (!workspace || need > have) return CYC_ERR_WORKSPACE;
    }
    if (p.batch <= kBatchPerLaunch) return run_chunk(p, k, split, workspace, s);
    const int64_t es = p.i8 ? 1 : 2;
    for (int64_t b0 = 0; b0 < p.batch; b0 += kBatchPerLaunch) {
        cyc::Problem q = p;
        q.batch = p.batch - b0 < kBatchPerLaunch ? p.batch - b0 : kBatchPerLaunch;
        q.A = (const char *)p.A + b0 * p.strideA * es;
        q.B = (const char *)p.B + b0 * p.strideB * es;
        q.C = (char *)p.C + b0 * p.strideC * 4;
        if (int st = run_chunk(q, k, split, workspace, s); st != CYC_OK) return st;
    }
    return CYC_OK;
}

// The memory of a solve or factorisation that needs `need` bytes, settled before its first launch.  in: the entry point for callers
// that bring it; copies: it is for padded copies, for which the library has none.  CYC_OK, or the status to return.
int memory_of(bool in, bool copies, int64_t need, void *given, int64_t given_bytes, hipStream_t s, cyc::WorkspaceHold &hold, void **workspace)
{
    *workspace = nullptr;
    if (need == 0) return CYC_OK;
    if (in && given) *workspace = given_bytes >= need ? given : nullptr;
    else if (!in || !(copies || cyc::is_capturing(s))) *workspace = hold.acquire(s, need);
    return *workspace ? CYC_OK : CYC_ERR_WORKSPACE;
}

int trsm(const void *L, const void *B, void *X, void *Xh, int64_t n, int64_t nrhs, int64_t nb, void *stream, bool in, void *given,
         int64_t given_bytes)
{
    if (n < 0 || nrhs < 0 || nb < 1 || nb > 128) return CYC_ERR_SHAPE;
    int64_t nn, nr;
    if (!mul_ok(n, n, &nn) || !mul_ok(n, nrhs, &nr)) return CYC_ERR_SHAPE;
    if (n == 0 || nrhs == 0) return CYC_OK;
    if (!L || !B || !X || !Xh) return CYC_ERR_NULL;
    if (!workspace_ok(given, given_bytes)) return CYC_ERR_SHAPE;
    if (overlaps(X, nr * 4, L, nn * 2) || overlaps(X, nr * 4, B, nr * 4) || overlaps(Xh, nr * 2, L, nn * 2) ||
        overlaps(Xh, nr * 2, B, nr * 4) || overlaps(X, nr * 4, Xh, nr * 2))
        return CYC_ERR_ALIAS;
    if (overlaps(given, given_bytes, L, nn * 2) || overlaps(given, given_bytes, B, nr * 4) || overlaps(given, given_bytes, X, nr * 4) ||
        overlaps(given, given_bytes, Xh, nr * 2))
        return CYC_ERR_ALIAS;
    const int64_t padded = in ? cyc::trsm_padded_bytes(L, X, Xh, n, nrhs, nb) : 0;
    const int64_t need = padded ? padded : cyc::trsm_workspace_bytes(L, X, Xh, n, nrhs, nb);
    cyc::WorkspaceHold hold;
    void *workspace;
    if (int st = memory_of(in, padded > 0, need, given, given_bytes, (hipStream_t)stream, hold, &workspace); st != CYC_OK) return st;
    const hipError_t e = padded ? cyc::launch_trsm_padded(L, B, X, Xh, n, nrhs, nb, workspace, (hipStream_t)stream)
                                : cyc::launch_trsm(L, B, X, Xh, n, nrhs, nb, workspace, (hipStream_t)stream);
    return e == hipSuccess ? CYC_OK : CYC_ERR_LAUNCH;
}

int cholesky(const void *A, void *L, void *Lh, int64_t n, int64_t nb, void *stream, bool in, void *given, int64_t given_bytes)
{
    if (n < 0 || nb < 1 || nb > 64 || n > (1 << 22)) return CYC_ERR_SHAPE;
    int64_t nn;
    if (!mul_ok(n, n, &nn)) return CYC_ERR_SHAPE;
    if (n == 0) return CYC_OK;
    if (!A || !L || !Lh) return CYC_ERR_NULL;
    if (((uintptr_t)A | (uintptr_t)L) & 3 || ((uintptr_t)Lh & 1) || !workspace_ok(given, given_bytes)) return CYC_ERR_SHAPE;
    if (overlaps(L, nn * 4, A, nn * 4) || overlaps(Lh, nn * 2, A, nn * 4) || overlaps(L, nn * 4, Lh, nn * 2)) return CYC_ERR_ALIAS;
    if (overlaps(given, given_bytes, A, nn * 4) || overlaps(given, given_bytes, L, nn * 4) || overlaps(given, given_bytes, Lh, nn * 2))
        return CYC_ERR_ALIAS;
    const int64_t padded = in ? cyc::chol_padded_bytes(A, L, Lh, n, nb) : 0, need = padded ? padded : cyc::chol_workspace_bytes(n, nb);
    cyc::WorkspaceHold hold;
    void *workspace;
    if (int st = memory_of(in, padded > 0, need, given, given_bytes, (hipStream_t)stream, hold, &workspace); st != CYC_OK) return st;
    const hipError_t e = padded ? cyc::launch_chol_padded(A, L, Lh, n, nb, workspace, (hipStream_t)stream)
                                : cyc::launch_chol(A, L, Lh, n, nb, workspace, (hipStream_t)stream);
    return e == hipSuccess ? CYC_OK : CYC_ERR_LAUNCH;
}

}  // namespace

namespace cyc {
int wait_limit() { return wait_limit_value().load(); }
}  // namespace cyc

extern "C" {

int cyc_recurrence_matmul_batched(const void *A, const void *B, void *C, int64_t batch, int64_t M, int64_t K,
                                  int64_t N, int64_t strideA, int64_t strideB, int64_t strideC, int dtype,
                                  void *stream)
{
    cyc::Problem p;
    Kernel k, family;
    cyc::KSplit split;
    int st = plan(A, B, C, batch, M, K, N, strideA, strideB, strideC, dtype, &p, &k, &family, &split, false);
    if (st != CYC_OK || k == K_NONE) return st;      // an error, or nothing to do (p is then not filled in)
    return run(p, k, split, (hipStream_t)stream, CACHED);
}

int cyc_recurrence_matmul(const void *A, const void *B, void *C, int64_t M, int64_t K, int64_t N, int dtype,
                          void *stream)
{
    return cyc_recurrence_matmul_batched(A, B, C, 1, M, K, N, 0, 0, 0, dtype, stream);
}

int cyc_recurrence_matmul_noalloc(const void *A, const void *B, void *C, int64_t M, int64_t K, int64_t N, int dtype,
                                  void *stream)
{
    cyc::Problem p;
    Kernel k, family;
    cyc::KSplit split;
    int st = plan(A, B, C, 1, M, K, N, 0, 0, 0, dtype, &p, &k, &family, &split, false);
    if (st != CYC_OK || k == K_NONE) return st;
    return run(p, k, split, (hipStream_t)stream, FIXED);
}

int64_t cyc_matmul_workspace(const void *A, const void *B, const void *C, int64_t M, int64_t K, int64_t N, int dtype)
{
    cyc::Problem p;
    Kernel k, family;
    cyc::KSplit split;
    if (plan(A, B, C, 1, M, K, N, 0, 0, 0, dtype, &p, &k, &family, &split, true) != CYC_OK || k != K_MFMAK) return 0;
    return cyc::ksplit_workspace_bytes(p, split.slices);
}

int cyc_recurrence_matmul_in(const void *A, const void *B, void *C, int64_t M, int64_t K, int64_t N, int dtype, void *workspace,
                             int64_t workspace_bytes, void *stream)
{
    cyc::Problem p;
    Kernel k, family;
    cyc::KSplit split;
    auto plan_for = [&](int64_t memory) { return plan(A, B, C, 1, M, K, N, 0, 0, 0, dtype, &p, &k, &family, &split, true, memory); };
    int st = plan_for(workspace && workspace_bytes >= 0 ? workspace_bytes : UNLIMITED);
    if (st != CYC_OK || k == K_NONE) return st;
    if (!workspace_ok(workspace, workspace_bytes)) return CYC_ERR_SHAPE;
    if (k != K_MFMAK) return run(p, k, split, (hipStream_t)stream, GIVEN);
    // (partial sums fit 64 MiB, 256 blocks of 256 x 256, which a stream's workspace may well keep; under a capture it
    // would be shared with other graphs, and asking torch for memory on every call costs 3 us of host time)
    if (!workspace) {
        if (cyc::is_capturing((hipStream_t)stream)) return CYC_ERR_WORKSPACE;
        st = run(p, k, split, (hipStream_t)stream, CACHED);
        if (st != CYC_ERR_WORKSPACE) return st;
        // the device has no such memory left: the slices that need least, if those are others
        const int slices = split.slices;
        st = plan_for(0);
        return st == CYC_OK && k == K_MFMAK && split.slices < slices ? run(p, k, split, (hipStream_t)stream, CACHED) : CYC_ERR_WORKSPACE;
    }
    const int64_t es = p.i8 ? 1 : 2;
    if (overlaps(workspace, workspace_bytes, A, M * K * es) || overlaps(workspace, workspace_bytes, B, K * N * es) ||
        overlaps(workspace, workspace_bytes, C, M * N * 4))
        return CYC_ERR_ALIAS;
    return run(p, k, split, (hipStream_t)stream, GIVEN, workspace, workspace_bytes);
}

int cyc_recurrence_trsm(const void *L, const void *B, void *X, void *Xh, int64_t n, int64_t nrhs, int64_t nb,
                        void *stream)
{
    return trsm(L, B, X, Xh, n, nrhs, nb, stream, false, nullptr, 0);
}

int64_t cyc_trsm_workspace(const void *L, void *X, void *Xh, int64_t n, int64_t nrhs, int64_t nb)
{
    int64_t t;
    if (n < 1 || nrhs < 1 || nb < 1 || nb > 128 || !mul_ok(n, n, &t) || !mul_ok(n, nrhs, &t)) return 0;
    const int64_t padded = cyc::trsm_padded_bytes(L, X, Xh, n, nrhs, nb);
    return padded ? padded : cyc::trsm_workspace_bytes(L, X, Xh, n, nrhs, nb);
}

int cyc_recurrence_trsm_in(const void *L, const void *B, void *X, void *Xh, int64_t n, int64_t nrhs, int64_t nb,
                           void *workspace, int64_t workspace_bytes, void *stream)
{
    return trsm(L, B, X, Xh, n, nrhs, nb, stream, true, workspace, workspace_bytes);
}

int cyc_recurrence_cholesky(const void *A, void *L, void *Lh, int64_t n, int64_t nb, void *stream)
{
    return cholesky(A, L, Lh, n, nb, stream, false, nullptr, 0);
}

int64_t cyc_cholesky_workspace(const void *A, void *L, void *Lh, int64_t n, int64_t nb)
{
    if (n < 1 || n > (1 << 22) || nb < 1 || nb > 64) return 0;
    const int64_t padded = cyc::chol_padded_bytes(A, L, Lh, n, nb);
    return padded ? padded : cyc::chol_workspace_bytes(n, nb);
}

int cyc_recurrence_cholesky_in(const void *A, void *L, void *Lh, int64_t n, int64_t nb, void *workspace, int64_t workspace_bytes,
                               void *stream)
{
    return cholesky(A, L, Lh, n, nb, stream, true, workspace, workspace_bytes);
}

int64_t cyc_attention_workspace(int64_t batch, int64_t N, int64_t M, int64_t d)
{
    int64_t nq, nk;
    if (batch < 1 || batch > 65535 || N < 1 || M < 1 || !cyc::supports_attention(N, M, d)) return 0;
    if (!mul_ok(N, d, &nq) || !mul_ok(M, d, &nk) || !mul_ok(batch, nq, &nq) || !mul_ok(batch, nk, &nk)) return 0;
    return cyc::attention_workspace_bytes(batch, N, M, d);
}

int cyc_recurrence_attention(const void *Q, const void *K, const void *V, void *O, int64_t batch, int64_t N, int64_t M,
                             int64_t d, void *stream)
{
    return cyc_recurrence_attention_split(Q, K, V, O, batch, N, M, d, nullptr, 0, stream);
}

int cyc_recurrence_attention_split(const void *Q, const void *K, const void *V, void *O, int64_t batch, int64_t N, int64_t M,
                                   int64_t d, void *workspace, int64_t workspace_bytes, void *stream)
{
    if (batch < 0 || N < 0 || M < 0 || d < 0) return CYC_ERR_SHAPE;
    if (batch == 0 || N == 0) return CYC_OK;
    int64_t nq, nk;
    if (!mul_ok(N, d, &nq) || !mul_ok(M, d, &nk) || !mul_ok(batch, nq, &nq) || !mul_ok(batch, nk, &nk)) return CYC_ERR_SHAPE;
    if (M == 0 || batch > 65535 || !cyc::supports_attention(N, M, d)) return CYC_ERR_SHAPE;
    if (!Q || !K || !V || !O) return CYC_ERR_NULL;
    if (((uintptr_t)Q | (uintptr_t)K | (uintptr_t)V | (uintptr_t)O) & 15) return CYC_ERR_SHAPE;
    if (overlaps(O, nq * 4, Q, nq * 2) || overlaps(O, nq * 4, K, nk * 2) || overlaps(O, nq * 4, V, nk * 2)) return CYC_ERR_ALIAS;
    if (!workspace || workspace_bytes < 0) workspace_bytes = 0;
    if ((uintptr_t)workspace & 15) return CYC_ERR_SHAPE;
    if (overlaps(workspace, workspace_bytes, Q, nq * 2) || overlaps(workspace, workspace_bytes, K, nk * 2) ||
        overlaps(workspace, workspace_bytes, V, nk * 2) || overlaps(workspace, workspace_bytes, O, nq * 4))
        return CYC_ERR_ALIAS;
    return cyc::launch_attention(Q, K, V, O, batch, N, M, d, workspace, workspace_bytes, (hipStream_t)stream) == hipSuccess ? CYC_OK
                                                                                                                        : CYC_ERR_LAUNCH;
}

const char *cyc_kernel_name(const void *A, const void *B, const void *C, int64_t batch, int64_t M, int64_t K,
                            int64_t N, int64_t strideA, int64_t strideB, int64_t strideC, int dtype)
{
    cyc::Problem p;
    Kernel k, family;
    cyc::KSplit split;
    if (plan(A, B, C, batch, M, K, N, strideA, strideB, strideC, dtype, &p, &k, &family, &split, false) != CYC_OK) return "none";
    return kernel_label(family);
}

const char *cyc_kernel_variant(const void *A, const void *B, const void *C, int64_t batch, int64_t M, int64_t K,
                               int64_t N, int64_t strideA, int64_t strideB, int64_t strideC, int dtype)
{
    cyc::Problem p;
    Kernel k, family;
    cyc::KSplit split;
    if (plan(A, B, C, batch, M, K, N, strideA, strideB, strideC, dtype, &p, &k, &family, &split, false) != CYC_OK) return "none";
    return kernel_label(k);
}

const char *cyc_status_string(int status)
{
    switch (status) {
        case CYC_OK: return "CYC_OK";
        case CYC_ERR_NULL: return "CYC_ERR_NULL: required pointer is NULL";
        case CYC_ERR_SHAPE: return "CYC_ERR_SHAPE: negative or overflowing extent or stride";
        case CYC_ERR_DTYPE: return "CYC_ERR_DTYPE: unknown element type";
        case CYC_ERR_ALIAS: return "CYC_ERR_ALIAS: C overlaps an input";
        case CYC_ERR_LAUNCH: return "CYC_ERR_LAUNCH: HIP launch failed";
        case CYC_ERR_WORKSPACE: return "CYC_ERR_WORKSPACE: workspace could not be allocated, or the problem needs more than the fixed workspace holds";
    }
    return "unknown cyc_status";
}

int cyc_version(void) { return 300; }

int cyc_diag_set_wait_limit(int64_t polls)
{
    if (polls < 0 || polls > (1 << 30)) return CYC_ERR_SHAPE;
    wait_limit_value().store(polls == 0 ? 1 << 20 : (int)polls);
    return CYC_OK;
}

int cyc_force_kernel(const char *name)
{
    if (!name || !*name) {
        forced_kernel().store((int)K_NONE);
        return CYC_OK;
    }
    const Kernel k = kernel_by_name(name);
    if (k == K_NONE) return CYC_ERR_SHAPE;
    forced_kernel().store((int)k);
    return CYC_OK;
}

}  // extern "C"
