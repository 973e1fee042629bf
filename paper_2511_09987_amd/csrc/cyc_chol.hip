// cyc_chol.hip -- the tiled Cholesky recurrence  A = L L^T  on gfx950.
//
// Paper, "Cholesky Recurrence": with A cut into nb x nb tiles, for every panel (tile column) j
//     S_jj = A_jj - sum_{k<j} SYRK(L_jk),          L_jj = CHOL(S_jj),
//     S_ij = A_ij - sum_{k<j} GEMM(L_ik, L_jk),    L_ij = TRSM(S_ij, L_jj)      for the tiles i below j,
// where the scalar form ("Representative recurrences") is
//     L_ii = sqrt(A_ii - sum_{k<i} L_ik^2),        L_ij = (A_ij - sum_{k<j} L_ik L_jk) / L_jj.
//
// Mapping, on the caller's stream.  The SYRKs and GEMMs are products of the matrix-multiply recurrence of this
// library (bf16 operands, fp32 sums): rows of the finished factor times the transpose of other rows of it.  The
// transpose costs nothing because the bf16 copy of the factor, Lh, is kept with both triangles filled
// (Lh[c][r] = Lh[r][c]): a stationary operand is a window Lh[r0:, k0:k1], the streamed one the window
// Lh[k0:k1, c0:c1].  Panels are taken in groups of eight (see launch_chol):
//   1. at the first panel of a group, one launch of the GEMM kernel takes all tiles left of the group out of the
//      group's columns: epilogue A - product into L[g0:, g0:g0+512], which holds S until solved;
//   2. per panel, CHOL of the diagonal tile in LDS (factor_tile64 in cyc_wave.h);
//   3. per panel, TRSM of the rows below, 64 to a workgroup: rows do not depend on one another; the off-diagonal line of the
//      scalar recurrence against L_jj in LDS (solve_rows16), written as rows of L and of Lh and as mirrored columns of Lh.
//   Both tile kernels are workgroups of four waves, which first take the terms of the group's own earlier panels out of
//   the tile with MFMAs of their own (TileProduct), which is far cheaper than a launch of the
//   GEMM kernel for so short a k range; each wave then has sixteen rows of the tile.  Step 2 for panel j + 1 is done by
//   the first workgroup of step 3 for panel j (the rows that become tile (j+1, j)), in the same launch, also across
//   a group boundary: the chain diagonal tile - tile below it - next diagonal tile is what the whole factorisation
//   waits for.  On that chain the TRSM of the tile below a well-conditioned diagonal tile is a product with the diagonal
//   tile's inverse, which waves that are done with their rows compute beside the factorisation of the tile (InverseColumns).
// Inside a tile column everything is fp32 on unrounded values, in the order of the scalar recurrence:
// t = S_rc; t = fma(-L_rk, L_ck, t) for k ascending; then sqrt on the diagonal, IEEE division below it.  Four such steps
// are one v_mfma_f32_16x16x4_f32: that instruction adds its products in ascending k with one rounding each.
#include "cyc_internal.h"
#include "cyc_wave.h"

namespace cyc {
namespace {

constexpr int NBMAX = 64;      // largest tile
constexpr int LDT = NBMAX + 4; // row stride of the tiles in LDS: rows stay 16-byte aligned, and 16 consecutive rows
                               // spread over all banks for 16-byte reads
typedef float f32x4 __attribute__((ext_vector_type(4), may_alias));   // read from arrays written as floats

// fp32 -> bfloat16 bit pattern, round to nearest, ties to even; NaN stays NaN (the hardware conversion)
__device__ __forceinline__ uint16_t round_bf16(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
// two values rounded and packed (a in the low half) by one conversion instruction, where rounding them one by one and
// joining the halves takes four
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) { return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){a, b}, bf16x2_t)); }

constexpr int NT = 256;        // threads of a tile kernel: four waves

// A 64-row tile of a row-major fp32 matrix (row stride ld) into LDS, by the workgroup: rows 0..nrows-1 (rows past that
// repeat the last one), columns 0..cols-1, zeros right of them.  DIAGONAL: a tile of cols x cols, padded with the identity.  (Of up to 32 or 16 columns: to 32 or 16, all that is looked at.)  All
// loads of a thread are in flight together.
template <bool DIAGONAL>
__device__ __forceinline__ void load_tile(float (*dst)[LDT], const float *src, int64_t ld, int nrows, int cols, int tid)
{
    if (cols == NBMAX && ld % 4 == 0 && ((uintptr_t)src & 15) == 0) {
        constexpr int PASSES = NBMAX * 16 / NT;
        f32x4 v[PASSES];
#pragma unroll
        for (int i = 0; i < PASSES; ++i) {
            const int r = NT / 16 * i + (tid >> 4);
            v[i] = *(const f32x4 *)(src + (int64_t)(r < nrows ? r : nrows - 1) * ld + 4 * (tid & 15));
        }
#pragma unroll
        for (int i = 0; i < PASSES; ++i) *(f32x4 *)&dst[NT / 16 * i + (tid >> 4)][4 * (tid & 15)] = v[i];
    } else {
        // a row to 64 lanes, or to 32 or 16 where that is all of the tile that is looked at
        auto load = [&](auto width) __attribute__((always_inline)) {
            constexpr int WIDTH = decltype(width)::value, PASSES = NBMAX * WIDTH / NT;
            const int c = tid % WIDTH;
            float v[PASSES];
#pragma unroll
            for (int i = 0; i < PASSES; ++i) {
                const int r = NT / WIDTH * i + tid / WIDTH;
                v[i] = c < cols ? src[(int64_t)(r < nrows ? r : nrows - 1) * ld + c] : 0.0f;
            }
#pragma unroll
            for (int i = 0; i < PASSES; ++i) {
                const int r = NT / WIDTH * i + tid / WIDTH;
                dst[r][c] = DIAGONAL && (r >= cols || c >= cols) ? (r == c ? 1.0f : 0.0f) : v[i];
            }
        };
        if (cols > 32) load(std::integral_constant<int, 64>{});
        else if (cols > 16) load(std::integral_constant<int, 32>{});
        else load(std::integral_constant<int, 16>{});
    }
}

// The same in two steps for kernels that fetch several tiles: request() issues the loads of a thread, place() puts
// them into LDS.  With the steps of two tiles interleaved (all requests, then all placements) memory is waited for
// once; load_tile twice in a row waits for the first tile before it asks for the second.
struct TileLoad {
    static constexpr int PASSES = NBMAX * 16 / NT;
    f32x4 v[PASSES];
    bool whole;
    __device__ __forceinline__ void request(const float *src, int64_t ld, int nrows, int cols, int tid)
    {
        whole = cols == NBMAX && ld % 4 == 0 && ((uintptr_t)src & 15) == 0;             // uniform
        if (whole) {
#pragma unroll
            for (int i = 0; i < PASSES; ++i) {
                const int r = NT / 16 * i + (tid >> 4);
                v[i] = *(const f32x4 *)(src + (int64_t)(r < nrows ? r : nrows - 1) * ld + 4 * (tid & 15));
            }
        }
    }
    template <bool DIAGONAL = false>
    __device__ __forceinline__ void place(float (*dst)[LDT], const float *src, int64_t ld, int nrows, int cols, int tid)
    {
        if (whole) {
#pragma unroll
            for (int i = 0; i < PASSES; ++i) *(f32x4 *)&dst[NT / 16 * i + (tid >> 4)][4 * (tid & 15)] = v[i];
        } else {
            load_tile<DIAGONAL>(dst, src, ld, nrows, cols, tid);
        }
    }
};

// The reverse for a full-width tile held in LDS: rows 0..nrows-1 to the fp32 matrix L and, rounded, to the bfloat16
// matrix Lh (both with row stride ld), 16 bytes per thread and store.  False when shape or alignment do not allow it.
// LOWER: the tile is a diagonal tile; L gets zeros above the diagonal (Lh gets what the tile holds there).  PARTS: 1: L, 2: Lh,
// 3: both; FIRST: L from that row on only.
template <bool LOWER, int NTH = NT, int PARTS = 3, int FIRST = 0>
__device__ __forceinline__ bool store_tile(const float (*src)[LDT], float *L, uint16_t *Lh, int64_t ld, int nrows, int cols,
                                           int tid)
{
    if (cols != NBMAX || ld % 8 != 0 || ((uintptr_t)L & 15) != 0 || ((uintptr_t)Lh & 15) != 0) return false;
    // all LDS reads first, without conditions (rows past nrows hold copies of the last one), then the stores: a read
    // inside the row condition would be waited for on the spot, once per row group
    constexpr int PL = PARTS & 1 ? (NBMAX - FIRST) * 16 / NTH : 0, PH = PARTS & 2 ? NBMAX * 8 / NTH : 0;      // tid counts the NTH threads that take part
    f32x4 v[PL + 1];
#pragma unroll
    for (int i = 0; i < PL; ++i) {
        const int r = FIRST + NTH / 16 * i + (tid >> 4);
        v[i] = *(const f32x4 *)&src[r][4 * (tid & 15)];
        if (LOWER) {
#pragma unroll
            for (int q = 0; q < 4; ++q) v[i][q] = 4 * (tid & 15) + q <= r ? v[i][q] : 0.0f;
        }
    }
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    u32x4 h[PH + 1];
#pragma unroll
    for (int i = 0; i < PH; ++i) {
        const int r = NTH / 8 * i + (tid >> 3);
        const f32x4 a = *(const f32x4 *)&src[r][8 * (tid & 7)], b = *(const f32x4 *)&src[r][8 * (tid & 7) + 4];
        h[i][0] = pack_bf16(a[0], a[1]);
        h[i][1] = pack_bf16(a[2], a[3]);
        h[i][2] = pack_bf16(b[0], b[1]);
        h[i][3] = pack_bf16(b[2], b[3]);
    }
#pragma unroll
    for (int i = 0; i < PL; ++i) {
        const int r = FIRST + NTH / 16 * i + (tid >> 4);
        if (r < nrows) *(f32x4 *)(L + (int64_t)r * ld + 4 * (tid & 15)) = v[i];
    }
#pragma unroll
    for (int i = 0; i < PH; ++i) {
        const int r = NTH / 8 * i + (tid >> 3);
        if (r < nrows) *(u32x4 *)(Lh + (int64_t)r * ld + 8 * (tid & 7)) = h[i];
    }
    return true;
}

// The same for any shape and alignment, by all threads: a row to 64, 32 or 16 lanes.
template <bool LOWER>
__device__ __forceinline__ void store_rows(const float (*src)[LDT], float *L, uint16_t *Lh, int64_t ld, int nrows, int cols, int tid)
{
    auto store = [&](auto width) __attribute__((always_inline)) {
        constexpr int WIDTH = decltype(width)::value, PASSES = NBMAX * WIDTH / NT;
        const int c = tid % WIDTH;
        float v[PASSES];
#pragma unroll
        for (int i = 0; i < PASSES; ++i) v[i] = src[NT / WIDTH * i + tid / WIDTH][c];
        if (c >= cols) return;
#pragma unroll
        for (int i = 0; i < PASSES; ++i) {
            const int r = NT / WIDTH * i + tid / WIDTH;
            if (r < nrows) {
                L[(int64_t)r * ld + c] = LOWER && c > r ? 0.0f : v[i];
                Lh[(int64_t)r * ld + c] = round_bf16(v[i]);
            }
        }
    };
    if (cols > 32) store(std::integral_constant<int, 64>{});
    else if (cols > 16) store(std::integral_constant<int, 32>{});
    else store(std::integral_constant<int, 16>{});
}

// The mirror image of 64 finished rows (a tile in LDS) into the upper triangle of Lh, by NTH threads: thread (column c,
// part) gathers 64 * 4 / NTH rows of its column (the rows of the tile are LDT floats apart: 16 of them lie on distinct
// banks) and stores them as 16-byte pieces.  dst: entry (column 0, row 0); requires 16-byte aligned rows of Lh.
template <int NTH>
__device__ __forceinline__ void store_mirror(const float (*src)[LDT], uint16_t *dst, int64_t ld, int tid)
{
    constexpr int PARTS = NTH / 64, ROWS = 64 / PARTS;
    const int c = tid / PARTS, r0 = ROWS * (tid % PARTS);
    uint32_t packed[ROWS / 2];
#pragma unroll
    for (int i = 0; i < ROWS / 2; ++i)
        packed[i] = pack_bf16(src[r0 + 2 * i][c], src[r0 + 2 * i + 1][c]);
    uint4 *out = (uint4 *)(dst + (int64_t)c * ld + r0);
#pragma unroll
    for (int i = 0; i < ROWS / 8; ++i) out[i] = make_uint4(packed[4 * i], packed[4 * i + 1], packed[4 * i + 2], packed[4 * i + 3]);
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x2 __attribute__((ext_vector_type(2)));
#define CYC_LDS __attribute__((address_space(3)))
constexpr int KMAX = 7 * NBMAX;           // longest k range a tile kernel multiplies out by itself (a group's earlier panels)

// The update of a 64 x 64 tile by the earlier panels of its group, inside the tile's own kernel (four waves):
//     S[r][c] -= sum_{k0 <= k < k1} Lh[row0 + r][k] * Lh[k][j0 + c]          (the second factor is the mirror image)
// as bf16 MFMAs with fp32 sums, S being a tile in LDS; wave w computes rows 16 w .. 16 w + 15 (one wave alone would
// be bound by the MFMA rate of its one SIMD: 224 MFMAs for seven tiles of k).  The streamed operand,
// Lh[k0:k1, j0:j0+64], is staged in LDS ([k][column], 128 bytes per row, see staged_swizzle) and read through the transpose read; the
// stationary operand, the tile's own rows of Lh, goes from memory straight into operand registers, all k-steps at
// once.  Rows past `nrows` repeat the last one.  Requires 16-byte aligned rows of Lh (n, k0, j0 multiples of 8) and
// k1 - k0 a multiple of 64, at most KM.
// In two parts, so that a kernel can ask for the operands first, then for its tile, and wait for memory once.
// An MFMA operand fragment of k-step ks out of a staged operand ([k][64 columns] in LDS), through the transposing
// read: lane l gets column 16 c + l%16, k = 32 ks + 8 (l/16) .. +7.  As a streamed fragment that is column block c; where
// the staged operand is the mirror image of rows of Lh, the same words are the stationary fragment of row block c.
// Placement of a staged operand: row k (128 bytes: eight 16-byte chunks) at k * 128, its chunk q in slot
// q ^ staged_swizzle(k).  One transposing read takes 8 bytes per lane from the rows 8 (l/16) + 0 .. 3 of a k-step, two
// adjacent chunks of each: unswizzled those are sixteen rows whose chunks lie on the same 16 of the 64 banks (a row is
// half the banks wide, rows two apart coincide), an eight-way conflict; the swizzle moves each group of eight rows to
// banks of its own, which leaves the two-way conflict that 512 bytes per instruction cannot avoid.
__device__ __forceinline__ constexpr int staged_swizzle(int k) { return ((k >> 3) & 3) << 1; }
__device__ __forceinline__ i32x4 staged_fragment(uint16_t (*src)[64], int ks, int c, int lq, int g)
{
    // (rows 32 ks + 8 g + 0 .. 7 share the swizzle 2 g)
    const int chunk = (2 * c + ((lq >> 1) & 1)) ^ (2 * g);
    CYC_LDS char *p = (CYC_LDS char *)&src[ks * 32 + 8 * g + (lq >> 2)][0] + 16 * chunk + 8 * (lq & 1);
    const i32x2 lo = __builtin_bit_cast(i32x2, __builtin_amdgcn_ds_read_tr16_b64_v4bf16((CYC_LDS bf16x4 *)p));
    const i32x2 hi = __builtin_bit_cast(i32x2, __builtin_amdgcn_ds_read_tr16_b64_v4bf16((CYC_LDS bf16x4 *)(p + 4 * 64 * 2)));
    return (i32x4){lo[0], lo[1], hi[0], hi[1]};
}

template <int KM>
struct TileProductT {
    static constexpr int NKS = KM / 32;
    i32x4 a[NKS];
    int nks;

    // start the copies of both operands; nothing is waited for
    // rows_in_lds: the tile's own rows of Lh will be at hand in LDS as their mirror image (see apply): none are loaded
    __device__ __forceinline__ void request(uint16_t (*Bs)[64], const uint16_t *__restrict__ Lh, int64_t n, int64_t row0, int nrows,
                                            int64_t k0, int64_t k1, int64_t j0, int tid, bool rows_in_lds = false)
    {
        const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), lq = lane & 15, g = lane >> 4, K = (int)(k1 - k0);
        nks = K / 32;
        // the streamed operand: 8 rows of 128 bytes per copy, memory to LDS directly, all copies in flight at once
        const uint32_t lds_base = (uint32_t)(uintptr_t)(CYC_LDS char *)&Bs[0][0];
        for (int k = 8 * w; k < K; k += 8 * (NT / 64)) {
            // lane l fills slot l%8 of row k + l/8: with the chunk that belongs there (staged_swizzle)
            const uint32_t voff = (uint32_t)(lane >> 3) * (uint32_t)(n * 2) + (uint32_t)((lane & 7) ^ staged_swizzle(k)) * 16;
            const char *base = (const char *)(Lh + (k0 + k) * n + j0);
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                         :
                         : "s"(lds_base + k * 128), "v"(voff), "s"(base)
                         : "memory", "m0");
        }
        // the stationary operand: row 16 w + lq of the tile, k = 32 ks + 8 g .. +7
        if (rows_in_lds) return;                                           // uniform
        const int r = 16 * w + lq;
        const uint16_t *rowp = Lh + (row0 + (r < nrows ? r : nrows - 1)) * n + k0 + 8 * g;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
            if (ks < nks) a[ks] = *(const i32x4 *)(rowp + 32 * ks);        // uniform; a load of 16 rows is 64 line requests: none to spare
    }

    // S -= product; call with the tile S in place in LDS and no barrier needed before: waits for the copies itself
    // As: nullptr, or Lh[k0:k1, row0:row0+64] in LDS, the mirror image of the tile's own rows (request with rows_in_lds):
    // the stationary fragment of rows 16 w .. is then read like a streamed fragment of column block w
    __device__ __forceinline__ void apply(float (*S)[LDT], uint16_t (*Bs)[64], int tid, uint16_t (*As)[64] = nullptr)
    {
        const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), lq = lane & 15, g = lane >> 4;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        f32x4 acc[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] = (f32x4){0, 0, 0, 0};
        if (As) {
            // every fragment from LDS: a loop that reads the fragments of the next k-step before it multiplies the
            // current ones (unrolled with a condition per step, as below, each step would wait for its own reads)
            i32x4 f[2][5];                                                       // [parity of the k-step]: stationary, streamed x 4
            auto read_step = [&](int ks, i32x4(&dst)[5]) __attribute__((always_inline)) {
                dst[0] = staged_fragment(As, ks, w, lq, g);
#pragma unroll
                for (int j = 0; j < 4; ++j) dst[1 + j] = staged_fragment(Bs, ks, j, lq, g);
            };
            auto multiply = [&](const i32x4(&src)[5]) __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, src[0]), __builtin_bit_cast(bf16x8, src[1 + j]), acc[j], 0, 0, 0);
            };
            read_step(0, f[0]);                                                  // (nks is even and at least 2)
            if (nks == 2) {                                                      // (a panel whose earlier terms were taken out ahead)
                read_step(1, f[1]);
                multiply(f[0]);
                multiply(f[1]);
            } else {
                for (int ks = 0; ks < nks; ks += 2) {
                    read_step(ks + 1, f[1]);
                    multiply(f[0]);
                    if (ks + 2 < nks) read_step(ks + 2, f[0]);
                    multiply(f[1]);
                }
            }
        }
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
            if (!As && ks < nks) {                                               // uniform over the workgroup
                i32x4 b[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) b[j] = staged_fragment(Bs, ks, j, lq, g);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[ks]), __builtin_bit_cast(bf16x8, b[j]), acc[j], 0, 0, 0);
            }
        }
        // accumulator register r of lane l is row 4 (l/16) + r, column l%16 of its 16 x 16 tile
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) S[16 * w + 4 * g + r][16 * j + lq] -= acc[j][r];
        __syncthreads();
    }
};

typedef TileProductT<KMAX> TileProduct;

constexpr float W_NORM_LIMIT = 8.0f;      // the product with a tile's inverse stands in for the recurrence below it (see chol_panel_kernel)

// The factorisation proper of a diagonal tile whose S (with everything left of it taken out) is in T: the column
// recurrence (factor_tile64 for a full tile), then L, and Lh in both triangles, written out by all.  See diag_tile.
// unsafe: two bytes in LDS, 0 with a barrier since; scratch: LDS (factor_tile64).  W: where the
// tile's inverse goes, or nullptr.  beside(G, w): called in the full-tile case by every wave w < G in the phases G = 1 .. 3.
template <class Beside>
__device__ __forceinline__ void diag_rest(float (*T)[LDT], char *unsafe, float *scratch, float *L, uint16_t *Lh, int64_t n, int64_t j0, int cols, int r,
                                          float *W, bool hint, Beside beside, float *copy = nullptr)
{
    InverseColumns inverse;
    static_assert(FACTOR_SCRATCH * sizeof(float) <= KMAX * 64 * sizeof(uint16_t), "the staged operand's place serves as scratch");
    if (cols == NBMAX) {
        // (the rows of L of a group go out as soon as the group is finished, by the wave that kept them; Lh, which is mirrored, at
        // the end)
        const bool aligned = n % 8 == 0 && ((uintptr_t)L & 15) == 0 && ((uintptr_t)Lh & 15) == 0;
        hint = factor_tile64<4>(T, unsafe, scratch, W, inverse, r, hint, [&](auto phase, int w) __attribute__((always_inline)) {
            constexpr int G = decltype(phase)::value;
            if (w == G - 1 && aligned) {
                f32x4 v[4];
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    const int row = 16 * (G - 1) + 4 * p + (r >> 4 & 3);
                    v[p] = *(const f32x4 *)&T[row][4 * (r & 15)];
#pragma unroll
                    for (int q = 0; q < 4; ++q) v[p][q] = 4 * (r & 15) + q <= row ? v[p][q] : 0.0f;
                }
#pragma unroll
                for (int p = 0; p < 4; ++p) *(f32x4 *)(L + (j0 + 16 * (G - 1) + 4 * p + (r >> 4 & 3)) * n + j0 + 4 * (r & 15)) = v[p];
            }
            beside(phase, w);
        });
    } else if (cols > 32) {
        factor_tile64<4>(T, unsafe, scratch, (float *)nullptr, inverse, r, false, [](auto, int) {});
    } else if (cols > 16) {
        factor_tile64<2>(T, unsafe, scratch, (float *)nullptr, inverse, r, false, [](auto, int) {});
    } else {
        factor_tile64<1>(T, unsafe, scratch, (float *)nullptr, inverse, r, false, [](auto, int) {});
    }
    if (copy) {
        // a second copy of the tile as it stands in LDS, rows of 64 floats (see chol_panel_kernel, Dcopy)
#pragma unroll
        for (int i = 0; i < NBMAX * 16 / NT; ++i) {
            const int row = NT / 16 * i + (r >> 4);
            *(f32x4 *)(copy + row * NBMAX + 4 * (r & 15)) = *(const f32x4 *)&T[row][4 * (r & 15)];
        }
    }
    const bool stored = store_tile<true, NT, 3, 48>(T, L + j0 * n + j0, Lh + j0 * n + j0, n, cols, cols, r);
    if (!stored) store_rows<true>(T, L + j0 * n + j0, Lh + j0 * n + j0, n, cols, cols, r);
    if (cols == NBMAX && W) finish_inverse<LDT>(T, scratch, W, inverse, r, hint);
}

// L_jj = CHOL(S_jj) for the tile at (j0, j0) with `cols` rows and columns.  S is read from Sm (row stride n: A itself
// for the first panel, L afterwards); L gets the factor below and on the diagonal and zero above it, Lh its bf16
// rounding in both triangles.  One workgroup of NT threads.  T (first 64 KB of LDS: a read reaches its word with the 16-bit offset field from one
// base register; further up every read needs an address register of its own) and Bs are the workgroup's LDS.
__device__ __forceinline__ void diag_tile(float (*T)[LDT], uint16_t (*Bs)[64], char *unsafe, const float *Sm, float *L, uint16_t *Lh, int64_t n,
                                          int64_t j0, int cols, int64_t k0, int r, float *W)
{
    if (r < 2) unsafe[r] = 0;              // (a barrier follows below)
    // (both operands of the tile's own update are the rows j0 .. of Lh: the staged one, Lh[k0:j0, j0:j0+64], is their
    // mirror image, and the stationary fragments are read from it as well)
    TileProduct product;
    if (k0 < j0) product.request(Bs, Lh, n, j0, cols, k0, j0, j0, r, true);     // k0 < j0 only for full tiles, see launch_chol
    load_tile<true>(T, Sm + j0 * n + j0, n, cols, cols, r);     // the whole square; what lies above the diagonal is not used
    if (k0 < j0) product.apply(T, Bs, r, Bs);
    else __syncthreads();
    diag_rest(T, unsafe, (float *)&Bs[0][0], L, Lh, n, j0, cols, r, W, false, [](auto, int) {});
}

__global__ __launch_bounds__(NT, 2) void chol_diag_kernel(const float *Sm, float *L, uint16_t *Lh, int64_t n, int64_t j0, int cols,
                                                       int64_t k0, float *W)
{
    __shared__ __attribute__((aligned(16))) struct {
        float T[NBMAX][LDT];          // S on entry, L as columns finish
        uint16_t Bs[KMAX][64];        // streamed operand of the tile's own update
        char unsafe[2];               // see factor_tile64
    } lds;
    diag_tile(lds.T, lds.Bs, lds.unsafe, Sm, L, Lh, n, j0, cols, k0, threadIdx.x, W);
}

// L_ij = TRSM(S_ij, L_jj) for all rows below the diagonal tile: rows j1 + 64 * blockIdx.x .., sixteen to a wave.
// next_Sm != nullptr: the workgroup of the first 64 rows goes on to factor the next diagonal tile, (j1, j1), whose S is
// read from next_Sm: it produces the only part of that tile's update that is still missing, and a launch of its own
// for the tile would first wait for memory again.  That workgroup requests the tile's S and the operands of its
// update over the group's earlier panels with everything else, first thing, and multiplies them out beside its rows'
// recurrence, sixteen rows of the tile to a wave.  Then the k range of this panel is added, straight from the solved
// rows in LDS, and the tile is factored; that workgroup's rows come as a product with the inverse of L_jj where that is well
// conditioned (Win, or nullptr: see InverseColumns; Wout: the next tile's), all others', which nothing waits for, by the recurrence.
// While the tile is factored, waves that are done with it write this workgroup's own rows out.
// On the path per launch at n = 8192, in cycles: 5k until the tiles are in LDS, 2.7k the rows, 1.8k the panel's k range into the next
// tile, 16.5k that tile, 2.7k Lh and the last rows of L and of the inverse (31k with the tile's recurrence in one wave, one lane
// to a row, helped by a second: 14.5k, and 5k more for a third that computed the inverse four columns behind; that made 18.6k a tile
// for the rows of all other workgroups, which are 6k now).  8192: 2388 -> 2083 us, and 2115 with the hint and limits of factor_tile64; 2048: 563 -> 506; 200: 61.5 -> 51.8.
__global__ __launch_bounds__(NT, 2) void chol_panel_kernel(const float *Sm, float *L, uint16_t *Lh, int64_t n, int64_t j0, int cols,
                                                        int64_t k0, const float *next_Sm, const float *__restrict__ Win,
                                                           float *Wout, const float *Dcopy,
                                                        float *next_copy, int64_t k0_first, int ahead)
{
    // one block, D and X first (see diag_tile)
    __shared__ __attribute__((aligned(16))) struct {
        float D[NBMAX][LDT];          // L_jj
        float X[64][LDT];             // this workgroup's rows: S on entry, L as columns finish
        uint16_t Bs[KMAX][64];        // streamed operand of the tile's own update
        uint16_t Bs2[KMAX][64];       // streamed operand of the next diagonal tile's update
        float rinv[64];               // the reciprocals of the diagonal of L_jj
        char unsafe[2];               // the next diagonal tile: see factor_tile64
    } lds;
    auto &D = lds.D;
    auto &X = lds.X;
    auto &Bs = lds.Bs;
    auto &Bs2 = lds.Bs2;
    const int tid = threadIdx.x, lane = tid & 63;
    // ahead != 0: the last two workgroups of the launch work for the NEXT launch's first workgroup, the one that everything
    // waits for.  Its two tiles, rows j1 + 64 .. of the column blocks j1 and j1 + 64 (its own rows and the diagonal tile that
    // rides along with it), lose the terms of the group's panels left of this one here, in place in S, while this launch
    // runs; that workgroup then starts at k = j0 (its k0_first) instead of at the group's first column, with a quarter of
    // the operands to fetch and two k-steps of each product instead of up to fourteen.  (Per entry the terms are then
    // subtracted in two chains, not one.)  Nothing else in this launch reads or writes those two tiles.
    const int row_blocks = (int)gridDim.x - (ahead ? 2 : 0);
    if ((int)blockIdx.x >= row_blocks) {
        const int64_t row0 = j0 + cols + NBMAX, col0 = j0 + cols + ((int)blockIdx.x - row_blocks) * NBMAX;
        float *tile = L + row0 * n + col0;                                 // (S of a later group's panels lives in L)
        TileProduct product;
        TileLoad of_S;
        product.request(Bs, Lh, n, row0, NBMAX, k0, j0, col0, tid);
        of_S.request(tile, n, NBMAX, NBMAX, tid);
        of_S.place(X, tile, n, NBMAX, NBMAX, tid);
        product.apply(X, Bs, tid);
#pragma unroll
        for (int i = 0; i < NBMAX * 16 / NT; ++i) {
            const int r = NT / 16 * i + (tid >> 4);
            *(f32x4 *)(tile + (int64_t)r * n + 4 * (tid & 15)) = *(const f32x4 *)&X[r][4 * (tid & 15)];
        }
        return;
    }
    if (blockIdx.x == 0) k0 = k0_first;                                    // uniform (see above)
    if (tid < 2) lds.unsafe[tid] = 0;
    // (requested here with everything else, looked at only where the rows are formed, so that nothing waits for them on their own)
    const bool may_invert = blockIdx.x == 0 && cols == NBMAX && Win != nullptr;        // uniform over the workgroup
    f32x4 winv[10], sum_L = {0, 0, 0, 0}, sum_W = sum_L;   // this lane's 40 values of W: pieces (cb, q), q <= cb
    if (may_invert) {
        sum_L = *(const f32x4 *)(Win + W_FLOATS);
        sum_W = *(const f32x4 *)(Win + W_FLOATS + 4);
        int p = 0;
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
#pragma unroll
            for (int q4 = 0; q4 <= cb; ++q4) winv[p++] = *(const f32x4 *)(Win + (cb * 4 + q4) * 256 + lane * 4);
    }
    const int64_t j1 = j0 + cols;
    const int64_t first = j1 + (int64_t)blockIdx.x * 64;
    const int nrows = (int)(n - first < 64 ? n - first : 64);
    // L is zero above the diagonal, and the products of the matrix-multiply kernel have written S there (a group's window
    // starts at the group's first row): every workgroup clears the mirror image of its tile's place, the rows of the
    // panel against its own columns.  Over all panels and workgroups that is everything above the diagonal tiles (which
    // clear their own upper halves), and nothing writes there after the group's product, which precedes its panels.
    // (At the end of the workgroup's work: ahead of its loads these stores would sit in the same queue before them.)
    auto clear_mirror_place = [&](int t, int nth) __attribute__((always_inline)) {
        if (cols == NBMAX && nrows == 64 && n % 4 == 0 && (uintptr_t)L % 16 == 0) {
#pragma unroll 4
            for (int i = t >> 4; i < NBMAX; i += nth / 16) *(f32x4 *)(L + (j0 + i) * n + first + 4 * (t & 15)) = (f32x4){0, 0, 0, 0};
        } else {
            for (int i = t >> 6; i < cols; i += nth / 64)
                if ((t & 63) < nrows) L[(j0 + i) * n + first + (t & 63)] = 0.0f;
        }
    };
    // ---- the next diagonal tile, first part: its S and the operands of the part of its update that does not involve
    // this panel are requested with everything else (their own LDS buffer, Bs2, so that they need not wait for Bs)
    const bool fused = next_Sm != nullptr && blockIdx.x == 0;          // uniform over the workgroup
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), lq = lane & 15, g = lane >> 4;
    const int nks_e = fused ? (int)(j0 - k0) / 32 : 0;                 // k-steps of that tile's update that do not involve this panel
    f32x4 sv[4], accn[4];                                              // its S (this thread's pieces); its update, rows 16 w ..: [column tile]
    // rows `first_row` .. +count-1 of the streamed operand Lh[., j1 : j1+64] into Bs2 from row `to` on, 8 rows per copy,
    // the copies dealt out to `waves` waves of which this is number `me`
    auto copy_rows = [&](int64_t first_row, int to, int count, int me, int waves) __attribute__((always_inline)) {
        const uint32_t lds_base = (uint32_t)(uintptr_t)(CYC_LDS char *)&Bs2[0][0];
        for (int k = 8 * me; k < count; k += 8 * waves) {
            const uint32_t voff = (uint32_t)(lane >> 3) * (uint32_t)(n * 2) + (uint32_t)((lane & 7) ^ staged_swizzle(to + k)) * 16;
            const char *base = (const char *)(Lh + (first_row + k) * n + j1);
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                         :
                         : "s"(lds_base + (to + k) * 128), "v"(voff), "s"(base)
                         : "memory", "m0");
        }
    };
    if (fused) {
#pragma unroll
        for (int i = 0; i < 4; ++i) sv[i] = *(const f32x4 *)(next_Sm + (j1 + 16 * i + (tid >> 4)) * n + j1 + 4 * (tid & 15));
        if (nks_e > 0) {
            // (only the streamed operand, Lh[k0:j0, j1:j1+64]: the stationary one, the rows j1 .. j1+63 of Lh over the same k,
            // is its mirror image, and the transposing read that makes a streamed fragment of column block c makes the
            // stationary fragment of row block c out of the same words)
            copy_rows(k0, 0, 32 * nks_e, w, NT / 64);
        }
    }
    TileProduct product;
    // (the workgroup that goes on to the next diagonal tile finds its own rows of Lh over k0 .. j0 in Bs2, mirrored: what
    // is left to fetch are whole rows, and nothing on the path waits for a load of 64 separate cache lines)
    const bool rows_in_lds = fused && nks_e > 0;
    if (k0 < j0) product.request(Bs, Lh, n, first, nrows, k0, j0, j0, tid, rows_in_lds);
    TileLoad of_D, of_X;
    // (Dcopy: L_jj is read from there, rows of 64 floats, because a product launched since it was factored has written over
    // its place in L, which the last workgroup restores)
    const float *Dsrc = Dcopy ? Dcopy : L + j0 * n + j0;
    const int64_t ldD = Dcopy ? NBMAX : n;
    of_D.request(Dsrc, ldD, cols, cols, tid);
    of_X.request(Sm + first * n + j0, n, nrows, cols, tid);
    of_D.place<true>(D, Dsrc, ldD, cols, cols, tid);
    of_X.place(X, Sm + first * n + j0, n, nrows, cols, tid);
    // (nks_e > 0 implies k0 < j0: apply waits for every copy of this wave, Bs2's included, before its barrier)
    if (k0 < j0) product.apply(X, Bs, tid, rows_in_lds ? Bs2 : nullptr);
    else __syncthreads();
    if (Dcopy && (int)blockIdx.x == row_blocks - 1) (void)store_tile<true>(D, L + j0 * n + j0, Lh + j0 * n + j0, n, cols, cols, tid);
#pragma unroll
    for (int j = 0; j < 4; ++j) accn[j] = (f32x4){0, 0, 0, 0};
    {
        // Sixteen rows to a wave (rows past the last one repeat it)
        wave_f32x4 S[4], t[4], x[4];
        float *const row = &X[16 * w + lq][0];
#pragma unroll
        for (int G = 0; G < 4; ++G) t[G] = S[G] = *(const wave_f32x4 *)(row + 16 * G + 4 * g);
        // the k-steps of the next diagonal tile's update over the group's earlier panels (both operands out of Bs2, see above)
        i32x4 f[2][5];                                                          // [parity of the k-step]: stationary, streamed x 4
        auto read_step = [&](int ks, i32x4(&dst)[5]) __attribute__((always_inline)) {
            dst[0] = staged_fragment(Bs2, ks, w, lq, g);
#pragma unroll
            for (int j = 0; j < 4; ++j) dst[1 + j] = staged_fragment(Bs2, ks, j, lq, g);
        };
        auto multiply = [&](const i32x4(&src)[5]) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                accn[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, src[0]), __builtin_bit_cast(bf16x8, src[1 + j]), accn[j], 0, 0, 0);
        };
        // (an upper bound of || |W| |L| ||_1, which is what the product's error grows with)
        // (the sign of the sums of |L| is a hint for the next diagonal tile, see factor_tile64)
        auto largest = [](const f32x4 &v) __attribute__((always_inline)) {
            return __builtin_fmaxf(__builtin_fmaxf(__builtin_fabsf(v[0]), __builtin_fabsf(v[1])), __builtin_fmaxf(__builtin_fabsf(v[2]), __builtin_fabsf(v[3])));
        };
        const float norm_L = largest(sum_L);
        const float norm_W = largest(sum_W);
        if (may_invert && __builtin_amdgcn_readfirstlane(norm_L * norm_W <= W_NORM_LIMIT) != 0) {
            // X <- S W^T.  A operand lane l: row 16w + l%16 of S, k = 4 ks + l/16; B operand: W[16 cb + l%16][4 ks + l/16], zero
            // for ks >= 4 (cb + 1); accumulator register r of lane l: row 16w + 4 (l/16) + r, column 16 cb + l%16.  Each wave
            // reads only its own rows of X before it overwrites them.
            float sa[16];
#pragma unroll
            for (int ks = 0; ks < 16; ++ks) sa[ks] = X[16 * w + lq][4 * ks + g];
            f32x4 xo[4];
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) xo[cb] = (f32x4){0, 0, 0, 0};
            // Between the MFMAs of this product (32 cycles of the matrix pipe each) run the k-steps of the next diagonal tile's
            // update, their fragments read a step ahead.  (The usual numbers of them, none and two, have a copy of the loop each
            // in which they are constants: as conditions at run time they cut every step of the product into pieces that wait for
            // their own reads.)
            auto product_loop = [&](auto steps_c) __attribute__((always_inline)) {
                constexpr int NE = decltype(steps_c)::value;                    // that many k-steps, or -1: nks_e of them (at most 14)
                auto has = [&](int ks) __attribute__((always_inline)) { return NE >= 0 ? ks < NE : ks < nks_e; };
                if (has(0)) read_step(0, f[0]);
#pragma unroll
                for (int ks = 0; ks < 16; ++ks) {
                    if (has(ks + 1)) read_step(ks + 1, f[(ks + 1) & 1]);
#pragma unroll
                    for (int cb = ks / 4; cb < 4; ++cb)
                        xo[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(sa[ks], winv[cb * (cb + 1) / 2 + ks / 4][ks % 4], xo[cb], 0, 0, 0);
                    if (has(ks)) multiply(f[ks & 1]);
                }
            };
            if (nks_e == 0) product_loop(std::integral_constant<int, 0>{});
            else if (nks_e == 2) product_loop(std::integral_constant<int, 2>{});
            else product_loop(std::integral_constant<int, -1>{});
#pragma unroll
            for (int cb = 0; cb < 4; ++cb)
#pragma unroll
                for (int r = 0; r < 4; ++r) X[16 * w + 4 * g + r][16 * cb + lq] = xo[cb][r];
        } else {
            // The divisions of a column share their divisor: quotients from its reciprocal, unless something is outside the
            // range in which these are IEEE's.  (Columns past the last one are zeros against the identity.)
            Pivot p;
            p.from_root(lane < cols ? D[lane][lane] : 1.0f);
            lds.rinv[lane] = p.r;                                               // (the same numbers by every wave: no barrier)
            auto solve = [&](auto by_pivots) __attribute__((always_inline)) {
                constexpr bool PIVOTS = decltype(by_pivots)::value;
                if (cols > 32) {
                    solve_rows16<PIVOTS, NBLK>(D, lds.rinv, t, row, lane, [](auto, float) {});
                } else if (cols > 16) {
                    wave_f32x4 u[2] = {t[0], t[1]};
                    solve_rows16<PIVOTS, NBLK / 2>(D, lds.rinv, u, row, lane, [](auto, float) {});
                } else {
                    wave_f32x4 u[1] = {t[0]};
                    solve_rows16<PIVOTS, NBLK / 4>(D, lds.rinv, u, row, lane, [](auto, float) {});
                }
            };
            solve(std::true_type{});
#pragma unroll
            for (int G = 0; G < 4; ++G) x[G] = 16 * G < cols ? *(const wave_f32x4 *)(row + 16 * G + 4 * g) : (wave_f32x4){1, 1, 1, 1};
            const unsigned worst = max(max(worst_code(x[0]), worst_code(x[1])), max(max(worst_code(x[2]), worst_code(x[3])), p.code()));
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(worst > SAFE_SPAN) != 0, 0)) {
                const bool safe = p.code() <= SAFE_SPAN && all_safe(x[0]) && all_safe(x[1]) && all_safe(x[2]) && all_safe(x[3]);
                if (__builtin_amdgcn_ballot_w64(!safe) != 0) {
#pragma unroll
                    for (int G = 0; G < 4; ++G) t[G] = S[G];
                    solve(std::false_type{});
                }
            }
            if (nks_e > 0) {                                                    // (an even number)
                read_step(0, f[0]);
                for (int ks = 0; ks < nks_e; ks += 2) {
                    read_step(ks + 1, f[1]);
                    multiply(f[0]);
                    if (ks + 2 < nks_e) read_step(ks + 2, f[0]);
                    multiply(f[1]);
                }
            }
        }
    }
    __syncthreads();
    // In the workgroup that goes on to the next diagonal tile some waves are done before others while that tile is factored:
    // they write this workgroup's rows out then (diag_rest below), off the path.  (There the tile is full and every
    // pointer aligned: the host fuses under those conditions only.)
    const bool deferred = fused && cols == NBMAX;
    if (!deferred) {
        if (!store_tile<false>(X, L + first * n + j0, Lh + first * n + j0, n, nrows, cols, tid))
            store_rows<false>(X, L + first * n + j0, Lh + first * n + j0, n, nrows, cols, tid);
        if (nrows == 64 && cols == NBMAX && n % 8 == 0 && (uintptr_t)Lh % 16 == 0) {
            store_mirror<NT>(X, Lh + j0 * n + first, n, tid);
        } else {
            // sixteen columns to a wave, a row to a lane: consecutive lanes, consecutive addresses
            float v[16];
#pragma unroll
            for (int c = 0; c < 16; ++c) v[c] = X[lane][16 * w + c];
            if (lane < nrows) {
#pragma unroll
                for (int c = 0; c < 16; ++c)
                    if (16 * w + c < cols) Lh[(j0 + 16 * w + c) * n + first + lane] = round_bf16(v[c]);
            }
        }
    }
    if (!fused) clear_mirror_place(tid, NT);
    if (fused) {
        // ---- the next diagonal tile, third part: the k range of this panel.  Its operands are the rows this
        // workgroup has just solved, still in X: both are the same fragments of X rounded to bfloat16 (the streamed
        // operand is the mirror image of the stationary one), so nothing has to come back from memory.
        auto fragment = [&](int q, int u) __attribute__((always_inline)) {     // row 16 q + lq, k = 32 u + 8 g .. +7 of the panel
            const float *p = &X[16 * q + lq][32 * u + 8 * g];
            const f32x4 lo = *(const f32x4 *)p, hi = *(const f32x4 *)(p + 4);
            i32x4 f;
            f[0] = (int)pack_bf16(lo[0], lo[1]);
            f[1] = (int)pack_bf16(lo[2], lo[3]);
            f[2] = (int)pack_bf16(hi[0], hi[1]);
            f[3] = (int)pack_bf16(hi[2], hi[3]);
            return f;
        };
#pragma unroll
        for (int i = 0; i < 4; ++i) *(f32x4 *)&D[16 * i + (tid >> 4)][4 * (tid & 15)] = sv[i];      // S into the tile (D is free)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            i32x4 bq[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) bq[j] = fragment(j, u);
            const i32x4 aq = fragment(w, u);
#pragma unroll
            for (int j = 0; j < 4; ++j)
                accn[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, aq), __builtin_bit_cast(bf16x8, bq[j]), accn[j], 0, 0, 0);
        }
        __syncthreads();
        // accumulator register r of lane l is row 4 (l/16) + r, column l%16 of its 16 x 16 tile
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) D[16 * w + 4 * g + r][16 * j + lq] -= accn[j][r];
        __syncthreads();
        // (zero where there is no inverse; one tile in eight is tried afresh)
        const bool hint = __builtin_amdgcn_readfirstlane((int)__builtin_signbit(sum_L[0])) != 0 && (j1 / NBMAX & 7) != 0;
        diag_rest(D, lds.unsafe, (float *)&Bs[0][0], L, Lh, n, j1, NBMAX, tid, Wout, hint, [&](auto phase, int wave) __attribute__((always_inline)) {
            // this workgroup's own rows, deferred above, shared by the first two waves
            constexpr int G = decltype(phase)::value;
            const int t = tid & 63;
            if (G == 1) clear_mirror_place(t, 64);
            if (G == 2 && wave == 0) store_tile<false, 64, 1>(X, L + first * n + j0, Lh + first * n + j0, n, nrows, cols, t);
            if (G == 2 && wave == 1) store_mirror<64>(X, Lh + j0 * n + first, n, t);
            if (G == 3 && wave == 1) store_tile<false, 64, 2>(X, L + first * n + j0, Lh + first * n + j0, n, nrows, cols, t);
        }, next_copy);
    }
}

}  // namespace

// one tile of 64 x 64 floats (see launch_chol: the first diagonal tile of a group rides along with the group before), and the
// inverse of one diagonal tile twice, for the launch that reads and the launch that writes
constexpr int64_t INVERSE = W_ALL * (int64_t)sizeof(float);
int64_t chol_workspace_bytes(int64_t n, int64_t nb)
{
    return nb == NBMAX && n >= 2 * NBMAX ? NBMAX * NBMAX * (int64_t)sizeof(float) + 2 * INVERSE : 0;
}

hipError_t launch_chol(const void *A_, void *L_, void *Lh_, int64_t n, int64_t nb, void *workspace, hipStream_t s)
{
    const float *A = (const float *)A_;
    float *L = (float *)L_;
    uint16_t *Lh = (uint16_t *)Lh_;
    if (nb < 1 || nb > NBMAX || n < 1 || n > (1 << 22)) return hipErrorInvalidValue;
    float *const tile_copy = chol_workspace_bytes(n, nb) > 0 ? (float *)workspace : nullptr;
    auto W_of = [&](int64_t j, int c) { return tile_copy && c == NBMAX ? (float *)((char *)(tile_copy + NBMAX * NBMAX) + j / NBMAX % 2 * INVERSE) : (float *)nullptr; };
    // One product per panel would have only nb columns and all earlier tiles as its k range: a few workgroups
    // walking a long k loop.  So the panels are taken in groups of GROUP: at the first panel of a group one product
    // covers the columns of the whole group against all tiles left of the group; the later panels of the group
    // then only add the terms of the group's own earlier panels (k range at most (GROUP - 1) * nb).  The terms of a
    // sum are the paper's; they are merely added in two chains instead of one.
    constexpr int GROUP = 8;          // measured at n = 8192: 4: 4.74 ms, 8: 4.22, 12: 4.26, 16: 4.33; with the side stream below 4: 4.11, 8: 3.99
    auto product = [&](int64_t r0, int64_t c0, int64_t ncols, int64_t k0, int64_t k1, const float *src, hipStream_t on) {
        Problem p;                        // L[r0:, c0:c0+ncols] = src[r0:, c0:c0+ncols] - Lh[r0:, k0:k1] * Lh[k0:k1, c0:c0+ncols]
        p.A = Lh + r0 * n + k0;           // finished factor, rows r0.., columns k0..k1
        p.lda = n;
        p.B = Lh + k0 * n + c0;           // its transpose, by mirror storage
        p.ldb = n;
        p.C = L + r0 * n + c0;
        p.Cin = src + r0 * n + c0;
        p.ldc = n;
        p.batch = 1;
        p.M = n - r0;
        p.K = k1 - k0;
        p.N = ncols;
        p.strideA = p.strideB = p.strideC = 0;
        p.i8 = false;
        // (a product beside the tile kernels, on the side stream, keeps to blocks of 128 and as few compute units: spread over all
        // of them in small blocks it was done sooner and held up the chain, 2461 against 2384 us at n = 8192)
        const int tile = on != s ? choose_mfma_tile(p) : 0;
        return tile ? launch_mfma(p, tile, 16, on) : launch_product(p, on);
    };
    bool diag_done = false;           // the diagonal tile of this panel was factored by the rows kernel of the panel before
    int64_t prepared_from = -1;       // >= 0: the launch before took the k range [k0, prepared_from) out of this launch's first workgroup's tiles
    bool copied = false;              // ... across a group boundary: L_jj is to be read from the copy in the workspace
    // the side stream is worth its events only when there are at least three groups
    SideStreamLock side_lock;
    SideStream *side = n > 2 * GROUP * nb ? side_lock.acquire() : nullptr;
    int64_t ahead = -1;               // first column of the group whose product over the groups before the last is on the side stream
    bool unjoined = false;            // work is on the side stream that the caller's stream does not wait for yet
    // a refused launch ends the call: what is already on the side stream is first joined back into the caller's stream
    auto fail = [&](hipError_t e) {
        if (unjoined) (void)hipStreamWaitEvent(s, side->join[0], 0);
        return e;
    };
    for (int64_t j0 = 0; j0 < n; j0 += nb) {
        const int cols = (int)(j0 + nb <= n ? nb : n - j0);
        const int64_t j1 = j0 + cols;
        const int64_t g0 = j0 / (GROUP * nb) * (GROUP * nb);      // first column of this panel's group
        const float *Sm = A;                                      // where S of this panel is read from
        if (j0 == g0 && g0 > 0) {
            const int64_t gcols = g0 + GROUP * nb <= n ? GROUP * nb : n - g0;
            if (ahead == g0) {
                // the part over the groups before the last was multiplied out on the side stream while the last group
                // was being factored; what is left is the k range of that group
                if (unjoined) {
                    if (hipError_t e = hipStreamWaitEvent(s, side->join[0], 0); e != hipSuccess) return fail(e);
                    unjoined = false;
                }
                // (when the group's first diagonal tile rode along with the last panel, this product writes over its place
                // in L: a copy of the tile is kept in the workspace, see below)
                if (hipError_t e = product(g0, g0, gcols, g0 - GROUP * nb, g0, L, s); e != hipSuccess) return fail(e);
            } else {
                if (hipError_t e = product(g0, g0, gcols, 0, g0, A, s); e != hipSuccess) return fail(e);
            }
            // The product for the NEXT group over everything left of this group does not depend on this group: it goes
            // to the side stream now and runs on the compute units that the tile kernels of this group (at most one
            // workgroup per 64 rows) leave idle.  Per entry the terms are then subtracted in two chains, not one.
            const int64_t g1 = g0 + GROUP * nb;
            if (side && g1 < n) {
                const int64_t ncols = g1 + GROUP * nb <= n ? GROUP * nb : n - g1;
                if (hipError_t e = hipEventRecord(side->fork, s); e != hipSuccess) return fail(e);
                if (hipError_t e = hipStreamWaitEvent(side->stream, side->fork, 0); e != hipSuccess) return fail(e);
                const hipError_t pe = product(g1, g1, ncols, 0, g0, A, side->stream);
                // whatever reached the side stream is covered by the join event, also when the product was refused
                if (hipError_t e = hipEventRecord(side->join[0], side->stream); e != hipSuccess) return fail(e);
                unjoined = true;
                if (pe != hipSuccess) return fail(pe);
                ahead = g1;
            }
        }
        if (g0 > 0) Sm = L;
        // the terms of the group's own earlier panels: multiplied out by the tile kernels themselves where they can
        // (full 64-column tiles with 16-byte aligned rows of Lh), else by a product of their own
        int64_t k0 = j0;                                          // k range [k0, j0) left to the tile kernels
        if (j0 > g0) {
            if (nb == NBMAX && cols == NBMAX && n % 8 == 0 && (uintptr_t)Lh % 16 == 0 && j0 - g0 <= KMAX) {
                k0 = g0;
            } else {
                if (hipError_t e = product(j0, j0, cols, g0, j0, Sm, s); e != hipSuccess) return fail(e);
                Sm = L;
            }
        }
        if (!diag_done) {
            hipError_t e = launch_kernel(chol_diag_kernel, dim3(1), dim3(NT), s, Sm, L, Lh, n, j0, cols, k0, W_of(j0, cols));
            if (e != hipSuccess) return fail(e);
        }
        diag_done = false;
        if (j1 < n) {
            // the next diagonal tile rides along when it is a full tile of the same group whose whole update the tile
            // kernels do themselves: its k range [g0, j1) then starts where this panel's starts
            // (the first diagonal tile of the next group, too, once that group's product over everything left of this
            // group is in, or when nothing lies left of this group: the tile's remaining k range is this group, which is
            // what the rows kernel has at hand)
            const bool next_group = j1 == g0 + GROUP * nb && (ahead == j1 || g0 == 0) && tile_copy != nullptr && j1 + NBMAX < n;
            const bool fuse = k0 == g0 && nb == NBMAX && cols == NBMAX && j1 + NBMAX <= n && (j1 < g0 + GROUP * nb || next_group) &&
                              n % 8 == 0 && (uintptr_t)Lh % 16 == 0 && (uintptr_t)A % 16 == 0 && (uintptr_t)L % 16 == 0 &&
                              j0 - g0 <= KMAX;
            if (fuse && next_group && unjoined) {
                if (hipError_t e = hipStreamWaitEvent(s, side->join[0], 0); e != hipSuccess) return fail(e);
                unjoined = false;
            }
            // (see `ahead` in the kernel: the next launch is a fused one of this group, not its last, S is in L, and there is
            // something left of this panel to take out)
            const bool prepare = fuse && g0 > 0 && j0 > g0 && j1 + NBMAX < g0 + GROUP * nb && j1 + 2 * NBMAX <= n;
            if (prepared_from >= 0 && !(fuse && k0 == g0 && prepared_from == j0 - NBMAX)) return fail(hipErrorUnknown);
            const int64_t k0_first = prepared_from >= 0 ? prepared_from : k0;
            hipError_t e = launch_kernel(chol_panel_kernel, dim3((unsigned)((n - j1 + 63) / 64 + (prepare ? 2 : 0))), dim3(NT), s, Sm, L, Lh, n, j0, cols, k0,
                               fuse ? (g0 > 0 ? (const float *)L : A) : (const float *)nullptr, (const float *)W_of(j0, cols),
                               fuse ? W_of(j1, NBMAX) : (float *)nullptr,
                               copied ? (const float *)tile_copy : (const float *)nullptr, fuse && next_group ? tile_copy : (float *)nullptr,
                               k0_first, prepare ? 1 : 0);
            if (e != hipSuccess) return fail(e);
            prepared_from = prepare ? j0 : -1;
            diag_done = fuse;
            copied = fuse && next_group;
        }
    }
    return hipSuccess;
}

}  // namespace cyc
