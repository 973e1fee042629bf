// cyc_uneven.hip -- the weight-stationary recurrence on the matrix cores for operands whose rows start at any byte:
// odd extents, windows at odd columns, unaligned pointers (what cyc_mfma.hip, whose copies go straight from global
// memory to LDS in aligned 16-byte pieces, does not take).  Its small blocks also serve aligned operands (choose_small_block
// below, and the rules for few rows and few columns in cyc_api.hip).
//
// Same mapping and same byte geometry as cyc_mfma.hip: a k-tile is 128 bytes of a row of A (64 bf16 or 128 int8),
// cut into eight 16-byte chunks; the partial sums are the MFMA accumulators.  What differs is the way into LDS: a chunk
// is fetched into registers with one 16-byte load at whatever address it has, a k-tile ahead, and written to its
// (aligned, swizzled) place in LDS with one 16-byte write.
//
// What bounds it: the address unit.  A wave-wide load of 64 chunks at 2-byte addresses occupies it for about 34 cycles
// (4-byte addresses 26, the aligned copies of cyc_mfma.hip 16), and a k-tile of a 96 x 128 block, 384 cycles of
// MFMAs, takes 28 of them; fetching two k-tiles ahead instead of one, or placing the writes elsewhere among the MFMAs, changed
// nothing (112 - 116 us at 3001 x 2999 x 3003 bf16).  That size took 1352 us on the vector ALU and takes 94 (576 TFLOP/s);
// int8 69; 74 x 787 x 27 took 104 us and takes 9, which is a launch.
//
// No load leaves the operands.  Rows past M re-read row M-1 and chunks wholly past N the last chunk that has a
// column of the matrix; neither is ever stored.  A chunk of B that straddles N reads on into the next row, which
// exists for every row but the last.  The k-tile that contains row K-1 of B and the ends of the rows of A is therefore
// fetched separately: a chunk that would cross the end of its row is loaded so that it ends there and shifted into
// place, zeros filling up.
#include "cyc_internal.h"

#include <algorithm>

namespace cyc {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef i32x4 i32x4_any __attribute__((aligned(1)));      // at any address

#define CYC_LDS __attribute__((address_space(3)))

template <bool I8> struct Mac;
template <> struct Mac<false> {
    typedef float elem;
    typedef f32x4 type;
    static __device__ __forceinline__ type mfma(i32x4 a, i32x4 b, type c)
    { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0); }
};
template <> struct Mac<true> {
    typedef int elem;
    typedef i32x4 type;
    static __device__ __forceinline__ type mfma(i32x4 a, i32x4 b, type c) { return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0); }
};

// A workgroup is WK teams of WM x WN waves.  Every team computes the whole BM x BN block over the k-tiles team, team +
// WK, ...; a wave owns TM x TN MFMA tiles.  With more than one team the teams' sums are added at the end, in
// ascending team order.
template <bool I8_, int TM_, int TN_, int WM_, int WN_, int WK_>
struct Shape {
    static constexpr bool I8 = I8_;
    static constexpr int TM = TM_, TN = TN_, WM = WM_, WN = WN_, WK = WK_;
    static constexpr int ES = I8 ? 1 : 2, E = 16 / ES;          // bytes per element, elements per chunk
    static constexpr int BM = 16 * TM * WM, BN = 16 * TN * WN, BKE = 128 / ES;
    static constexpr int TW = WM * WN, NT = 64 * TW * WK;       // waves per team, threads per workgroup
    static constexpr int RB = BN * ES, CPR = RB / 16;           // bytes and chunks per row of the B tile
    static constexpr int A_BYTES = BM * 128, B_BYTES = BKE * RB, STAGE = A_BYTES + B_BYTES;
    static constexpr int NST = TW > 1 ? 2 : 1;                  // LDS stages; a wave by itself needs no second one
    static constexpr int AI = A_BYTES / 1024 / TW, BI = B_BYTES / 1024 / TW;   // chunks per lane and k-tile
    static_assert(A_BYTES % (1024 * TW) == 0 && B_BYTES % (1024 * TW) == 0 && 64 % CPR == 0, "chunks must divide evenly over the team");
    static_assert(WK == 1 || TW == 1, "teams of one wave join through their own stage");
    static_assert(WK == 1 || STAGE >= TM * TN * 1024, "a stage must hold a wave's sums");
};

__device__ __forceinline__ int swizzle_a(int r) { return (r >> 1) & 7; }
// Half a wave reads, per transpose read, rows k..k+3 and k+8..k+11 of 32 bytes (bf16) or rows k..k+7 and k+16..k+23 of 16
// bytes (int8); the XOR puts those that share a place modulo 256 bytes into different slots.
template <class S> __device__ __forceinline__ int swizzle_b(int k)
{
    if (!S::I8) return S::CPR >= 16 ? ((k & 3) << 1) | (((k >> 3) & 1) << 3) : S::CPR == 8 ? (((k >> 1) & 1) << 1) | (((k >> 3) & 1) << 2) : ((k >> 3) & 1) << 1;
    return S::CPR >= 8 ? ((k >> 1) & 3) | (((k >> 4) & 1) << 2) : S::CPR == 4 ? ((k >> 2) & 1) | (((k >> 4) & 1) << 1) : (k >> 4) & 1;
}

// v shifted down by `bytes` (0 .. 15) bytes, zeros from above
__device__ __forceinline__ i32x4 shift_down(i32x4 v, int bytes)
{
    uint64_t lo = (uint32_t)v[0] | (uint64_t)(uint32_t)v[1] << 32, hi = (uint32_t)v[2] | (uint64_t)(uint32_t)v[3] << 32;
    if (bytes >= 8) { lo = hi; hi = 0; bytes -= 8; }
    if (bytes) { lo = lo >> (8 * bytes) | hi << (64 - 8 * bytes); hi >>= 8 * bytes; }
    return (i32x4){(int)(uint32_t)lo, (int)(lo >> 32), (int)(uint32_t)hi, (int)(hi >> 32)};
}

template <class S>
__global__ __launch_bounds__(S::NT, S::WK == 1 ? 2 : 1) void ws_uneven_kernel(const char *__restrict__ A, const char *__restrict__ B, char *__restrict__ Cout,
                                                          int M, int K, int N, int64_t sA, int64_t sB, int64_t sC, int tiles_m,
                                                          int tiles_n, int64_t lda, int64_t ldb, int64_t ldc, const char *Cin)
{
    constexpr int ES = S::ES, E = S::E, TM = S::TM, TN = S::TN, AI = S::AI, BI = S::BI, RB = S::RB;
    typedef typename Mac<S::I8>::elem elem;
    typedef typename Mac<S::I8>::type acc_t;
    __shared__ __attribute__((aligned(1024))) char lds_raw[S::WK * S::NST * S::STAGE];

    const int l = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int team = wave / S::TW, w = wave % S::TW, wm = w / S::WN, wn = w % S::WN;
    CYC_LDS char *lds = (CYC_LDS char *)lds_raw + team * S::NST * S::STAGE;

    // which block of C: workgroups are dealt round robin to the 8 XCDs; each XCD gets a contiguous run of blocks (the
    // first nblk % 8 one more), four block-rows deep, so that its L2 keeps the rows of A while columns of B pass
    const int nblk = tiles_m * tiles_n, xcd = blockIdx.x & 7;
    const int bid = xcd * (nblk >> 3) + (xcd < (nblk & 7) ? xcd : (nblk & 7)) + (blockIdx.x >> 3);
    const int per_group = 4 * tiles_n, group = bid / per_group, in_group = bid % per_group;
    const int rows_here = tiles_m - group * 4 < 4 ? tiles_m - group * 4 : 4;
    const int m0 = (group * 4 + in_group % rows_here) * S::BM, n0 = in_group / rows_here * S::BN;
    A += (int64_t)blockIdx.y * sA * ES + (int64_t)m0 * lda * ES;
    B += (int64_t)blockIdx.y * sB * ES + (int64_t)n0 * ES;
    Cout += (int64_t)blockIdx.y * sC * 4;

    // this lane's chunks of a k-tile: offsets from the tile's first byte
    const int last = (K - 1) / S::BKE;                       // the k-tile with the ends of the rows of A and the last row of B
    const int64_t step_b = (int64_t)S::BKE * ldb * ES;
    uint32_t off_a[AI], off_b[BI];
#pragma unroll
    for (int x = 0; x < AI; ++x) {
        int r = (w * AI + x) * 8 + (l >> 3);
        const int c = (l & 7) ^ swizzle_a(r);
        r = m0 + r < M ? r : M - 1 - m0;
        off_a[x] = (uint32_t)((int64_t)r * lda * ES) + c * 16;
    }
#pragma unroll
    for (int x = 0; x < BI; ++x) {
        const int kr = (w * BI + x) * (64 / S::CPR) + l / S::CPR;
        int c = (l % S::CPR) ^ swizzle_b<S>(kr);
        c = c * E < N - n0 ? c : (N - 1 - n0) / E;
        off_b[x] = (uint32_t)((int64_t)kr * ldb * ES) + c * 16;
    }
    // k-tile number i as the loop takes them: the one with the ends first, by fetch_ends(); then 0, 1, ... by fetch()
    auto fetch = [&](i32x4(&ra)[AI], i32x4(&rb)[BI], int i) __attribute__((always_inline)) {
        if (i > last) return;
        const char *a = A + (int64_t)(i - 1) * 128, *b = B + (i - 1) * step_b;
        // (the empty statements keep the offsets in 32 bits, as the loads take them beside a scalar base)
#pragma unroll
        for (int x = 0; x < AI; ++x) {
            uint32_t off = off_a[x];
            asm volatile("" : "+v"(off));
            ra[x] = *(const i32x4_any *)(a + off);
        }
#pragma unroll
        for (int x = 0; x < BI; ++x) {
            uint32_t off = off_b[x];
            asm volatile("" : "+v"(off));
            rb[x] = *(const i32x4_any *)(b + off);
        }
    };
    auto fetch_ends = [&](i32x4(&ra)[AI], i32x4(&rb)[BI]) __attribute__((always_inline)) {
        const char *a = A + (int64_t)last * 128, *b = B + last * step_b;
        const int left = K - last * S::BKE;                  // k in this tile: 1 .. BKE
#pragma unroll
        for (int x = 0; x < AI; ++x) {
            const int c = (l & 7) ^ swizzle_a((w * AI + x) * 8 + (l >> 3));
            const int over = c * E + E - left;               // elements of this chunk past the end of the row (K >= E: its start is in the row)
            ra[x] = (i32x4){0, 0, 0, 0};
            if (over < E) {
                const int back = over > 0 ? over * ES : 0;
                ra[x] = shift_down(*(const i32x4_any *)(a + off_a[x] - (int64_t)back), back);
            }
        }
#pragma unroll
        for (int x = 0; x < BI; ++x) {
            const int kr = (w * BI + x) * (64 / S::CPR) + l / S::CPR;
            int c = (l % S::CPR) ^ swizzle_b<S>(kr);
            c = c * E < N - n0 ? c : (N - 1 - n0) / E;
            const int over = c * E + E - (N - n0);           // columns of this chunk past N, below E
            rb[x] = (i32x4){0, 0, 0, 0};
            if (kr < left) {
                const int back = over > 0 ? over * ES : 0;
                rb[x] = shift_down(*(const i32x4_any *)(b + off_b[x] - (int64_t)back), back);
            }
        }
    };
    auto put = [&](const i32x4(&ra)[AI], const i32x4(&rb)[BI], int stage) __attribute__((always_inline)) {
        CYC_LDS char *to = lds + stage * S::STAGE + l * 16;
#pragma unroll
        for (int x = 0; x < AI; ++x) *(CYC_LDS i32x4 *)(to + (w * AI + x) * 1024) = ra[x];
#pragma unroll
        for (int x = 0; x < BI; ++x) *(CYC_LDS i32x4 *)(to + S::A_BYTES + (w * BI + x) * 1024) = rb[x];
    };

    // this lane's fragments in LDS (see cyc_mfma.hip): A row l%16, chunk 4 ks + l/16; B through the transpose read
    int frag_a[2], frag_b[TN];
    {
        const int r = wm * TM * 16 + (l & 15);
        for (int ks = 0; ks < 2; ++ks) frag_a[ks] = r * 128 + (((ks * 4 + (l >> 4)) ^ swizzle_a(r)) << 4);
        const int lq = l & 15, kg = l >> 4, krow = S::I8 ? 16 * kg + (lq >> 1) : 8 * kg + (lq >> 2);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int byte = (wn * TN * 16 + j * 16 + (S::I8 ? 8 * (lq & 1) : 4 * (lq & 3))) * ES;
            frag_b[j] = S::A_BYTES + krow * RB + (((byte >> 4) ^ swizzle_b<S>(krow)) << 4) + (byte & 15);
        }
    }
    // with teams, a sum of its own for either half of the k-tiles: shorter chains, which round less and wait less for one another
    // (relative error at K = 8192 bf16 1.9e-7 with one)
    constexpr int CHAINS = S::WK > 1 ? 2 : 1;
    acc_t acc[CHAINS][TM][TN];
#pragma unroll
    for (int h = 0; h < CHAINS; ++h)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[h][i][j] = (acc_t){0, 0, 0, 0};
    i32x4 fa[2][TM], fb[2][TN];
    auto read_fragments = [&](int stage, int ks) __attribute__((always_inline)) {
        CYC_LDS char *from = lds + stage * S::STAGE;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            CYC_LDS char *p = from + frag_b[j] + ks * (S::BKE / 2) * RB;
            i32x2 lo, hi;
            if (S::I8) {
                lo = __builtin_amdgcn_ds_read_tr8_b64_v2i32((CYC_LDS i32x2 *)p);
                hi = __builtin_amdgcn_ds_read_tr8_b64_v2i32((CYC_LDS i32x2 *)(p + 8 * RB));
            } else {
                lo = __builtin_bit_cast(i32x2, __builtin_amdgcn_ds_read_tr16_b64_v4bf16((CYC_LDS bf16x4 *)p));
                hi = __builtin_bit_cast(i32x2, __builtin_amdgcn_ds_read_tr16_b64_v4bf16((CYC_LDS bf16x4 *)(p + 4 * RB)));
            }
            fb[ks][j] = (i32x4){lo[0], lo[1], hi[0], hi[1]};
        }
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[ks][i] = *(CYC_LDS i32x4 *)(from + frag_a[ks] + i * 16 * 128);
    };
    auto multiply = [&](int ks) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[ks % CHAINS][i][j] = Mac<S::I8>::mfma(fa[ks][i], fb[ks][j], acc[ks % CHAINS][i][j]);
    };
    // every wave of the team has written its chunks of the next k-tile and read its fragments of this one.  (A team of one
    // wave needs only the program order that LDS keeps; the statement then holds the compiler to it.)
    auto meet = [&]() __attribute__((always_inline)) {
        if (S::TW > 1) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        else asm volatile("" ::: "memory");
    };

    // The registers hold the k-tile after the one in LDS.  Past the last k-tile nothing is fetched, and what is put is never
    // read.
    i32x4 ra[AI], rb[BI];
    if constexpr (S::NST == 2) {
        fetch_ends(ra, rb);
        put(ra, rb, 0);
        fetch(ra, rb, 1);
        meet();
        auto turn = [&](int i, int odd) __attribute__((always_inline)) {
            read_fragments(odd, 0);
            read_fragments(odd, 1);
            multiply(0);
            __builtin_amdgcn_sched_barrier(0);
            put(ra, rb, odd ^ 1);
            fetch(ra, rb, i + 2);
            __builtin_amdgcn_sched_barrier(0);
            multiply(1);
            meet();
        };
        for (int i = 0; i <= last; i += 2) {
            turn(i, 0);
            if (i + 1 > last) break;
            turn(i + 1, 1);
        }
    } else {
        if (team == 0) fetch_ends(ra, rb);
        else fetch(ra, rb, team);
        for (int i = team; i <= last; i += S::WK) {
            put(ra, rb, 0);
            fetch(ra, rb, i + S::WK);
            meet();
            read_fragments(0, 0);
            read_fragments(0, 1);
            multiply(0);
            multiply(1);
            meet();
        }
    }

    // C_ij <- [i,k_end]_C: register r of lane l is row 4 (l/16) + r, column l%16 of its MFMA tile
    elem *C = (elem *)Cout;
    auto emit = [&](int i, int j, acc_t v) __attribute__((always_inline)) {
        const int col = n0 + (wn * TN + j) * 16 + (l & 15);
        if (col >= N) return;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = m0 + (wm * TM + i) * 16 + (l >> 4) * 4 + r;
            if (row < M) C[row * ldc + col] = Cin ? ((const elem *)Cin)[row * ldc + col] - v[r] : v[r];
        }
    };
    if constexpr (S::WK == 1) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) emit(i, j, acc[0][i][j]);
    } else {
        // the hand-over along k: every team leaves its sums in its own stage, then each joins its share of the MFMA tiles
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) *(CYC_LDS acc_t *)(lds + (i * TN + j) * 1024 + l * 16) = acc[0][i][j] + acc[CHAINS - 1][i][j];
        __syncthreads();
        CYC_LDS char *all = (CYC_LDS char *)lds_raw + l * 16;
        for (int t = team; t < TM * TN; t += S::WK) {
            acc_t sum = *(CYC_LDS acc_t *)(all + t * 1024);
#pragma unroll
            for (int g = 1; g < S::WK; ++g) sum += *(CYC_LDS acc_t *)(all + g * S::STAGE + t * 1024);
            emit(t / TN, t % TN, sum);
        }
    }
}

template <class S> hipError_t launch_shape(const Problem &p, hipStream_t s)
{
    const int tiles_m = (int)((p.M + S::BM - 1) / S::BM), tiles_n = (int)((p.N + S::BN - 1) / S::BN);
    return launch_kernel(ws_uneven_kernel<S>, dim3((unsigned)(tiles_m * tiles_n), (unsigned)p.batch), dim3(S::NT), s, (const char *)p.A,
                         (const char *)p.B, (char *)p.C, (int)p.M, (int)p.K, (int)p.N, p.strideA, p.strideB, p.strideC, tiles_m, tiles_n,
                         row_stride_a(p), row_stride_b(p), row_stride_c(p), (const char *)p.Cin);
}

template <bool I8> hipError_t launch_dtype(const Problem &p, int block, hipStream_t s)
{
    switch (block) {
        case 256: return launch_shape<Shape<I8, 4, 4, 4, 2, 1>>(p, s);
        case 96: return launch_shape<Shape<I8, 3, 4, 2, 2, 1>>(p, s);
        case 64: return launch_shape<Shape<I8, 2, 2, 2, 2, 1>>(p, s);
        case 32: return launch_shape<Shape<I8, 2, 2, 1, 1, 8>>(p, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

// Any alignment; K and N at least one 16-byte chunk (8 bf16, 16 int8), so that a chunk that ends where its row ends starts
// inside that row.  N below that is taken where K is a multiple of a chunk and more than a k-tile: a chunk of B then reads on
// into the rows after its own (at least a chunk's worth of rows follow every row that is not in the last k-tile; what it reads
// lands in columns that are not stored), and in the last k-tile back into rows before it.
bool supports_uneven(const Problem &p)
{
    const int64_t es = p.i8 ? 1 : 2, e = 16 / es;
    if (p.M < 1 || p.K < e || p.N < 1 || p.batch < 1 || p.batch > 65535) return false;
    if (p.N < e && (p.K % e != 0 || p.K <= 8 * e)) return false;
    if (p.M > (1 << 30) || p.K > (1 << 30) || p.N > (1 << 30)) return false;
    if (((p.M + 31) / 32) * ((p.N + 31) / 32) > (1 << 30)) return false;
    const int64_t lda = row_stride_a(p), ldb = row_stride_b(p);
    if (lda < p.K || ldb < p.N || row_stride_c(p) < p.N) return false;
    // per-lane byte offsets inside a k-tile are kept in 32 bits
    return lda * es * 256 + 256 < ((int64_t)1 << 32) && ldb * es * 128 + 256 < ((int64_t)1 << 32);
}

// Costs in units of 10 ns: a launch, the blocks per compute unit (256 of them) that are started and stored, and the
// k-tiles of the last workgroup to finish (the blocks of 32 cut them among eight teams).  Fitted over operands that change from
// call to call, 560 products of 1 .. 200000 rows and columns, k of 8 .. 4096, batches of up to 1000, bf16 and int8: within 1 % of
// the best block on average, and nowhere behind ws_generic_kernel.  (A rule by rounds and k-tiles alone took the blocks of 32
// wherever k was short, at a round's cost each: bf16 1000000 x 9 x 9 235 us where ws_generic_kernel took 66 and this
// takes 59, 2000 x (16 x 31 x 100) 69 / 33 / 22.)  Microseconds, blocks of 256 / 96 / 64 / 32: 1696 x 977 x 1820 29.7 / 24.5 / 24.7 / 41.4, 1001^3
// 25 / 17 / 10 / 16, 17 x 4001 x 1001 - / 41 / 21 / 10, 34 x 117 x 6419 a hundred times 173 / 99 / 73 / 394, 100^3 8.0 / 7.0 / 4.4 / 4.2.
int choose_uneven_block(const Problem &p)
{
    const int64_t bke = p.i8 ? 128 : 64, kt = (p.K + bke - 1) / bke;
    auto cost = [&](int64_t bm, int64_t bn, int64_t start, int64_t block, int64_t tile, int64_t round, int64_t k) {
        const int64_t n = ((p.M + bm - 1) / bm) * ((p.N + bn - 1) / bn) * p.batch, rounds = (n + 255) / 256;
        return start + block * n / 256 + tile * k * std::max<int64_t>(100, round * rounds) / 100;   // round: of its k-tiles' time, in percent (several workgroups share a compute unit)
    };
    const int64_t c256 = cost(256, 128, 620, 520, 130, 107, kt), c96 = cost(96, 128, 540, 262, 76, 88, kt);
    const int64_t c64 = cost(64, 64, 390, 80, 46, 78, kt), c32 = cost(32, 32, 285, 66, 140, 95, (kt + 7) / 8);
    if (c256 <= c96 && c256 <= c64 && c256 <= c32) return 256;
    if (c96 <= c64 && c96 <= c32) return 96;
    return c64 <= c32 ? 64 : 32;
}

hipError_t launch_uneven(const Problem &p, int block, hipStream_t s)
{
    if (!supports_uneven(p)) return hipErrorInvalidValue;
    return p.i8 ? launch_dtype<true>(p, block, s) : launch_dtype<false>(p, block, s);
}

// Products with aligned rows and few blocks of 128 x 128 leave most of the chip idle: blocks of 64 x 64, or of 32 x 32 with
// eight teams along k, are then the faster ones although they stage through registers.  Costs in units of 10 ns per launch,
// fitted to (bf16, microseconds, 128 / 64 / 32 wide blocks; i8 has twice the k per k-tile and fits the same):
//   64 x 64 x 64 5.5 / 3.9 / 4.0        128 x 1024 x 128 8.8 / 7.5 / 4.5    512^3 6.4 / 5.8 / 4.7      384 x 2048 x 384 14.4 / 11.7 / 6.3
//   768^3 9.1 / 7.1 / 9.6               1024^3 9.5 / 8.5 / 12.4             1536^3 16.3 / 21.4 / 35    200 x 2048 x 4096 17.8 / 12.3 / 18.1
//   16 x (64 x 2048 x 64) 17 / 11 / 6   2 x (33 x 4096 x 4096) 34 / 28 / 20
int choose_small_block(const Problem &p)
{
    if (p.M < 16 || p.N < 16 || !supports_uneven(p)) return 0;
    auto blocks = [&](int64_t b) { return ((p.M + b - 1) / b) * ((p.N + b - 1) / b) * p.batch; };
    const int64_t bke = p.i8 ? 128 : 64, kt = (p.K + bke - 1) / bke, n128 = blocks(128);
    if (n128 > 256) return 0;
    const int64_t r64 = (blocks(64) + 255) / 256, r32 = (blocks(32) + 255) / 256;
    int64_t c128 = 340 + 45 * kt, c64 = 330 + 25 * kt * r64, c32 = 330 + r32 * (30 + 65 * ((kt + 7) / 8));
    // Whole blocks of 128 and whole k-tiles have a kernel of their own, a microsecond quicker, and then every block counts as well
    // (140 such products, bf16 and int8): 64 x (128^3) bf16 5.5 / 5.9 / -, int8 100 x (128^3) 5.6 / 6.7 / 19, 30 x (256 x 384 x 128) 7.5 / 8.2 / 13,
    // 512 x 256 x 128 5.6 / 5.7 / 5.0, 128 x 2048 x 768 18.7 / 16.2 / 8.8
    if (p.M % 128 == 0 && p.N % 128 == 0 && p.K % bke == 0) {
        c128 = 350 + 47 * kt + 3 * n128 / 2;
        c64 = 390 + 38 * kt * r64 + 2 * n128;
        c32 = 250 + r32 * (200 + 13 * kt) + 4 * std::min<int64_t>(n128, 16);
    }
    if (std::min(c64, c32) >= c128) return 0;
    return c32 <= c64 ? 32 : 64;
}

hipError_t launch_product(const Problem &p, hipStream_t s)
{
    const int tile = choose_mfma_tile(p);
    if (tile == 128)
        if (const int block = choose_small_block(p)) return launch_uneven(p, block, s);
    return tile ? launch_mfma(p, tile, 16, s) : launch_any_alignment(p, s);
}

}  // namespace cyc
