// cyc_pad.hip -- triangular solves and Cholesky factorisations of systems whose rows are not 16-byte aligned.
//
// The tile kernels that go through the inverses of the diagonal tiles read and write whole 16-byte pieces of rows.  A
// system of any other size or address is embedded in one that has them, n and nrhs rounded up to multiples of 8,
//     [ L 0 ] [ X 0 ]   [ B 0 ]            [ A 0 ]
//     [ 0 I ] [ 0 0 ] = [ 0 0 ]    resp.   [ 0 I ],
// solved in memory that the caller brings and copied out.  The added rows and columns are zeros in every product, so the sums of the
// others are the same.  What bounds it is still the chain of tiles; the copies are two more passes over the operands in
// three launches.  Tile by tile / now, microseconds: solve 513 x 8 104 / 37, 1333 x 28 270 / 95, 1984 x 603
// 429 / 116, 2047 x 4001 681 / 179; Cholesky 133 53 / 42, 585 255 / 157, 1001 443 / 252, 2047 1014 / 522.
#include "cyc_internal.h"

namespace cyc {
namespace {

constexpr int64_t MAX_COPY_BYTES = (int64_t)256 << 20;   // what a call asks of its caller at most: no copies beyond this

inline int64_t up8(int64_t x) { return (x + 7) & ~(int64_t)7; }
inline int64_t up256(int64_t x) { return (x + 255) & ~(int64_t)255; }

// dst (rows_out x ld_out) <- src (rows x cols, row stride cols), zeros around it; lower: only what lies on and below the
// diagonal of src is read, zeros above it and ones on the diagonal of the rows past it.  One workgroup per 1024 columns
// of a row.
template <typename T>
__global__ __launch_bounds__(256) void pad_kernel(const T *__restrict__ src, T *__restrict__ dst, int64_t rows, int64_t cols, int64_t ld_out,
                                                  int lower, T one)
{
    const int64_t r = blockIdx.x;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t c = (int64_t)blockIdx.y * 1024 + i * 256 + threadIdx.x;
        if (c >= ld_out) return;
        T v = 0;
        if (r < rows && c < cols && (!lower || c <= r)) v = src[r * cols + c];
        else if (lower && r >= rows && c == r) v = one;
        dst[r * ld_out + c] = v;
    }
}

// dst (rows x cols, row stride cols) <- the upper left corner of src (row stride ld_in), in both precisions
__global__ __launch_bounds__(256) void unpad_kernel(const float *__restrict__ src, const uint16_t *__restrict__ src_h, float *__restrict__ dst,
                                                    uint16_t *__restrict__ dst_h, int64_t cols, int64_t ld_in)
{
    const int64_t r = blockIdx.x;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t c = (int64_t)blockIdx.y * 1024 + i * 256 + threadIdx.x;
        if (c >= cols) return;
        dst[r * cols + c] = src[r * ld_in + c];
        dst_h[r * cols + c] = src_h[r * ld_in + c];
    }
}

dim3 grid_of(int64_t rows, int64_t cols) { return dim3((unsigned)rows, (unsigned)((cols + 1023) / 1024)); }

struct TrsmCopies {
    int64_t n, nrhs, L, X, Xh, total;     // padded extents; sizes in bytes, multiples of 256
    TrsmCopies(int64_t n_, int64_t nrhs_) : n(up8(n_)), nrhs(up8(nrhs_))
    {
        L = up256(n * n * 2);
        X = up256(n * nrhs * 4);
        Xh = up256(n * nrhs * 2);
        total = L + X + Xh;
    }
};

struct CholCopies {
    int64_t n, A, Lh, total;
    explicit CholCopies(int64_t n_) : n(up8(n_))
    {
        A = up256(n * n * 4);
        Lh = up256(n * n * 2);
        total = 2 * A + Lh;
    }
};

// any place that is 16-byte aligned, to ask what a call on the copies would need
void *const ALIGNED = (void *)(uintptr_t)4096;

}  // namespace

int64_t trsm_padded_bytes(const void *L, void *X, void *Xh, int64_t n, int64_t nrhs, int64_t nb)
{
    // (a short chain of tiles is as fast by substitution: 200 x 9 46 us, 200 x 16 35)
    if (nb != 64 || n < 512 || n > (1 << 16) || nrhs > (1 << 20) || trsm_workspace_bytes(L, X, Xh, n, nrhs, nb) > 0) return 0;
    const TrsmCopies c(n, nrhs);
    if (c.total > MAX_COPY_BYTES) return 0;
    return c.total + trsm_workspace_bytes(ALIGNED, ALIGNED, ALIGNED, c.n, c.nrhs, nb);
}

hipError_t launch_trsm_padded(const void *L, const void *B, void *X, void *Xh, int64_t n, int64_t nrhs, int64_t nb, void *workspace, hipStream_t s)
{
    const TrsmCopies c(n, nrhs);
    char *w = (char *)workspace;
    uint16_t *Lp = (uint16_t *)w;
    float *Xp = (float *)(w + c.L);
    uint16_t *Xhp = (uint16_t *)(w + c.L + c.X);
    hipError_t e = launch_kernel(pad_kernel<uint16_t>, grid_of(c.n, c.n), dim3(256), s, (const uint16_t *)L, Lp, n, n, c.n, 1, (uint16_t)0x3f80);
    // (the solve reads a right-hand side before it writes that row of X, as it does with its own running right-hand sides)
    if (e == hipSuccess) e = launch_kernel(pad_kernel<float>, grid_of(c.n, c.nrhs), dim3(256), s, (const float *)B, Xp, n, nrhs, c.nrhs, 0, 0.0f);
    if (e == hipSuccess) e = launch_trsm(Lp, Xp, Xp, Xhp, c.n, c.nrhs, nb, w + c.total, s, true);
    if (e == hipSuccess) e = launch_kernel(unpad_kernel, grid_of(n, nrhs), dim3(256), s, (const float *)Xp, (const uint16_t *)Xhp, (float *)X, (uint16_t *)Xh, nrhs, c.nrhs);
    return e;
}

int64_t chol_padded_bytes(const void *A, void *L, void *Lh, int64_t n, int64_t nb)
{
    const bool aligned = n % 8 == 0 && (((uintptr_t)A | (uintptr_t)L | (uintptr_t)Lh) & 15) == 0;
    if (nb != 64 || n <= 128 || n > (1 << 16) || aligned) return 0;
    const CholCopies c(n);
    if (c.total > MAX_COPY_BYTES) return 0;
    return c.total + chol_workspace_bytes(c.n, nb);
}

hipError_t launch_chol_padded(const void *A, void *L, void *Lh, int64_t n, int64_t nb, void *workspace, hipStream_t s)
{
    const CholCopies c(n);
    char *w = (char *)workspace;
    float *Ap = (float *)w, *Lp = (float *)(w + c.A);
    uint16_t *Lhp = (uint16_t *)(w + 2 * c.A);
    hipError_t e = launch_kernel(pad_kernel<float>, grid_of(c.n, c.n), dim3(256), s, (const float *)A, Ap, n, n, c.n, 1, 1.0f);
    if (e == hipSuccess) e = launch_chol(Ap, Lp, Lhp, c.n, nb, w + c.total, s);
    if (e == hipSuccess) e = launch_kernel(unpad_kernel, grid_of(n, n), dim3(256), s, (const float *)Lp, (const uint16_t *)Lhp, (float *)L, (uint16_t *)Lh, n, c.n);
    return e;
}

}  // namespace cyc
