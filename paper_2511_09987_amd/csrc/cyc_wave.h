// cyc_wave.h -- device helpers shared by the kernels that run the scalar recurrence of a tile, in one wave or in four
// (the tile kernels of the triangular solve and of the Cholesky factorisation).
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

namespace cyc {

// f(integral_constant<int, 0>), ..., f(integral_constant<int, N - 1>): a loop whose index is a constant in every copy
// from the start (the unrolling pass gives up on bodies as long as those of the tile kernels)
template <class F, int... I>
__device__ __forceinline__ void unrolled(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void unrolled(F &&f)
{
    unrolled(f, std::make_integer_sequence<int, N>{});
}

// IEEE fp32 division num / den (correctly rounded, all special cases) in four phases: the instruction sequence the
// compiler itself expands a division into, cut up so that independent work can be placed between the phases of this
// long dependent chain: scale and reciprocal estimate; a Newton step on the reciprocal; quotient and one correction;
// the last correction and the hardware's fix-up of scaling and special cases.
struct Division {
    float num, den, d0, n0, r, q;
    bool flag;
    __device__ __forceinline__ void phase0(float numerator, float denominator)
    {
        num = numerator;
        den = denominator;
        bool unused;
        d0 = __builtin_amdgcn_div_scalef(num, den, false, &unused);
        n0 = __builtin_amdgcn_div_scalef(num, den, true, &flag);
        r = __builtin_amdgcn_rcpf(d0);
    }
    __device__ __forceinline__ void phase1()
    {
        const float e = __builtin_fmaf(-d0, r, 1.0f);
        r = __builtin_fmaf(e, r, r);
    }
    __device__ __forceinline__ void phase2()
    {
        q = n0 * r;
        const float e = __builtin_fmaf(-d0, q, n0);
        q = __builtin_fmaf(e, r, q);
    }
    __device__ __forceinline__ float phase3()
    {
        const float e = __builtin_fmaf(-d0, q, n0);
        return __builtin_amdgcn_div_fixupf(__builtin_amdgcn_div_fmasf(e, r, q, flag), den, num);
    }
};

// 2 |x| as a bit pattern less that of 2^-50: unsafe above SAFE_SPAN, and for a zero, which is safe (NaN and infinity are not)
constexpr unsigned SAFE_LOW = (127u - 50u) << 24, SAFE_SPAN = 100u << 24;
__device__ __forceinline__ unsigned range_code(float x) { return (__builtin_bit_cast(unsigned, x) << 1) - SAFE_LOW; }
__device__ __forceinline__ bool in_safe_range(unsigned code, unsigned lower) { return code + lower <= SAFE_SPAN + lower || code == 0u - SAFE_LOW; }
// What counts is that a quotient times its divisor is at least 2^-100: with divisors of at least 2^-24 (code: see Pivot) results
// down to 2^-76 are safe, too.  (lower, above: 0 or this)
__device__ __forceinline__ unsigned lower_limit(unsigned code) { return code >= 26u << 24 ? 26u << 24 : 0u; }

// Correctly rounded square root and quotients by it in fewer dependent instructions than the compiler's expansions (7 from
// the pivot to a quotient, 27 there), for a pivot that a whole column is divided by.  Markstein's method: the hardware's
// estimates, off by a unit in the last place at most, corrected by exact remainders, d = g + (s - g g) y / 2, and with a
// correctly rounded reciprocal r, q = q0 - (d q0 - t) r for q0 = t r.  The remainders are exact and the results those of IEEE
// as long as nothing over- or underflows: where every |x| that comes out, pivots included, lies in [2^-50, 2^50] or is zero, or see lower_limit
// (in_safe_range; zeros keep their sign where the pivot is positive); callers take the compiler's way elsewhere.
// Evidence, on the device (cyc_diag_pivots): the root on every float in [2^-100, 2^100); for every divisor's
// significand D, 24 bits, the reciprocal and the quotients of the numerators for which these lie within 15 / (2 D) units of a
// midpoint (all of them for odd D): the error before the last rounding, at most 1.5 units * 2^-23, reaches 6 / (2 D).  The
// reciprocal of a root is a unit off for 24 squares in [1, 4): there every numerator.
// One exception that a look at the results does not show: a numerator k 2^-149 over the divisor next below 2 k gives 0 here,
// and the smallest denormal number, 2^-149, by division.
// (One unit is added to the estimate of 1 / sqrt(s): without it the reciprocal of a significand of 24 ones comes out as a tie.)
struct Pivot {
    float d, r;                                               // sqrt(s), 1 / d
    __device__ __forceinline__ void from_square(float s)
    {
        const float y = __builtin_amdgcn_rsqf(s), g = __builtin_amdgcn_sqrtf(s);
        d = __builtin_fmaf(__builtin_fmaf(-g, g, s), 0.5f * y, g);
        refine(__builtin_bit_cast(float, __builtin_bit_cast(int, y) + 1));
    }
    __device__ __forceinline__ void from_root(float root)
    {
        d = root;
        refine(__builtin_amdgcn_rcpf(d));
    }
    __device__ __forceinline__ float quotient(float t) const
    {
        const float q = t * r;
        return __builtin_fmaf(-__builtin_fmaf(d, q, -t), r, q);
    }
    // of a divisor: below SAFE_SPAN when it is one for quotient()
    __device__ __forceinline__ unsigned code() const { return d > 0.0f ? range_code(d) : ~0u; }

private:
    __device__ __forceinline__ void refine(float estimate) { r = __builtin_fmaf(__builtin_fmaf(-d, estimate, 1.0f), estimate, estimate); }
};
// The column recurrence of a 64-wide tile as a fixed list of steps, for the kernels that run it in one wave with
// the lane's row in registers.  The 64 columns go in 16 blocks of four.  The four chains of block b first take the
// columns left of the block (b "bulk" steps of four k each: 16 independent multiply-adds), then the 4 x 4 corner
// finishes the four columns one after the other, each with a division: a chain of dependent instructions.  In a lone
// wave a dependent instruction issues every ~8 cycles, an independent one every ~5, so the corner of block b is
// interleaved with bulk steps of block b + 1: its steps over k4 < b do not need the columns the corner is producing,
// and up to EARLY of them are taken out of turn, one beside each corner column.  Every entry still takes its terms
// in ascending k.  StepList is the resulting execution order of all 120 bulk steps.
constexpr int NBLK = 64 / 4, EARLY = 4, NSTEP = NBLK * (NBLK - 1) / 2;
constexpr int early_of(int b) { return b < 1 ? 0 : (b - 1 < EARLY ? b - 1 : EARLY); }
struct StepList {
    signed char b[NSTEP + 2], k[NSTEP + 2];
};
constexpr StepList make_steps()
{
    StepList s{};
    int n = 0;
    for (int b = 0; b < NBLK; ++b) {
        for (int k4 = early_of(b); k4 < b; ++k4) {           // in turn, before the corner of block b
            s.b[n] = (signed char)b;
            s.k[n++] = (signed char)k4;
        }
        if (b + 1 < NBLK)
            for (int k4 = 0; k4 < early_of(b + 1); ++k4) {   // out of turn, beside the corner of block b
                s.b[n] = (signed char)(b + 1);
                s.k[n++] = (signed char)k4;
            }
    }
    s.b[n] = s.b[n + 1] = -1;                                // (requests past the end do nothing)
    return s;
}
constexpr StepList STEPS = make_steps();

// ---- Sixteen rows per wave.  Both recurrences over a 64-wide tile, one in which the pivots are known (rows of
// X L^T = S, a right-hand side of L y = r being such a row) and the factorisation itself, in the accumulator layout of
// v_mfma_f32_16x16x4_f32 with the columns on its row axis: register r of lane l = 16 g + i holds column 16 G + 4 g + r of row i,
// G = 0 .. 3 counting the groups of sixteen columns.  A block of four columns is then solved in the sixteen lanes that
// hold it, its four values spread to operand order by three lane swaps, and taken out of all columns right of it by one MFMA
// per group, which adds its four products in ascending k with one rounding each: the terms, the order and the bits of the
// scalar chain t = fma(-x_k, L_ck, t).  What is left is bound by
// instruction issue, about 6 cycles an instruction in a wave alone on its SIMD: 6k cycles for 64 rows and columns.  A row per lane
// in one wave, 2016 multiply-adds and eleven instructions a division, took 18.6k.
typedef float wave_f32x4 __attribute__((ext_vector_type(4), may_alias));

// The four values that the lanes 16 GK .. 16 GK + 15 hold, one to a group of lanes: lane 16 q + i gets value q of lane 16 GK + i.
template <int GK>
__device__ __forceinline__ float spread16(const wave_f32x4 &x)
{
    auto bits = [](float v) __attribute__((always_inline)) { return __builtin_bit_cast(unsigned, v); };
    const auto u = __builtin_amdgcn_permlane32_swap(bits(x[0]), bits(x[2]), false, false);
    const auto v = __builtin_amdgcn_permlane32_swap(bits(x[1]), bits(x[3]), false, false);
    const auto w = __builtin_amdgcn_permlane16_swap(u[GK / 2], v[GK / 2], false, false);
    const unsigned r = w[GK % 2];
    return __builtin_bit_cast(float, r);
}

// row[c] <- the solution of X L^T = S for the wave's sixteen rows, whose S is in t (used up); row: where the lane's row i lies in
// LDS, 64 columns and four of padding.  D: L in LDS, fp32, row-major; only what lies on and below the diagonal matters.  rinv: the
// reciprocals of its diagonal (PIVOTS; see Pivot: the caller looks at what came out, and solves again without PIVOTS where that
// is outside the safe range).  each(block, out) is called once per block of four columns with its number, a constant, and minus its
// values in operand order: lane 16 q + i has column 4 block + q of row i.  BLOCKS: so many blocks only.
template <bool PIVOTS, int BLOCKS, int LDD, class Each>
__device__ __forceinline__ void solve_rows16(const float (*D)[LDD], const float *rinv, wave_f32x4 (&t)[BLOCKS / 4], float *row, int lane, Each each)
{
    const int i = lane & 15, g = lane >> 4;
    // (as many values of a corner's row as it has: what a read brings and nobody uses is given to the next read's destination, which
    // then waits for the first)
    typedef float f32x2 __attribute__((ext_vector_type(2), may_alias));
    typedef float f32x3 __attribute__((ext_vector_type(3), may_alias));
    float c0[2];
    f32x2 c1[2];
    f32x3 c2[2];
    wave_f32x4 c3[2], ri[2];
    float a[2][4];                                                              // rows 16 h + i of L, columns 4 b + g
    auto request = [&](auto index) __attribute__((always_inline)) {             // what block b needs
        constexpr int b = decltype(index)::value, p = b & 1;
        c0[p] = D[4 * b][4 * b];
        c1[p] = *(const f32x2 *)&D[4 * b + 1][4 * b];
        c2[p] = *(const f32x3 *)&D[4 * b + 2][4 * b];
        c3[p] = *(const wave_f32x4 *)&D[4 * b + 3][4 * b];
        if (PIVOTS) ri[p] = *(const wave_f32x4 *)(rinv + 4 * b);
#pragma unroll
        for (int h = (b + 1) / 4; h < BLOCKS / 4; ++h) a[p][h] = D[16 * h + i][4 * b + g];
    };
    request(std::integral_constant<int, 0>{});
    unrolled<BLOCKS>([&](auto index) __attribute__((always_inline)) {
        constexpr int b = decltype(index)::value, G = b / 4, gk = b % 4, first = (b + 1) / 4;
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (b + 1 < BLOCKS) request(std::integral_constant<int, b + 1>{});
        __builtin_amdgcn_sched_barrier(0);
        wave_f32x4 c = t[G], v;                                                 // (a copy: the other lanes hold other columns)
        constexpr int p = b & 1;
        const float corner[4][4] = {{c0[p]}, {c1[p][0], c1[p][1]}, {c2[p][0], c2[p][1], c2[p][2]}, {c3[p][0], c3[p][1], c3[p][2], c3[p][3]}};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float d = corner[j][j];
            if (PIVOTS) {
                const float r = ri[p][j], q = c[j] * r;
                v[j] = __builtin_fmaf(-__builtin_fmaf(d, q, -c[j]), r, q);
            } else {
                v[j] = c[j] / d;
            }
#pragma unroll
            for (int e = j + 1; e < 4; ++e) c[e] = __builtin_fmaf(-v[j], corner[e][j], c[e]);
        }
        *(wave_f32x4 *)(row + (g == gk ? 16 * G + 4 * gk : 64)) = v;            // (the other lanes': into the padding)
        const float out = -spread16<gk>(v);
        each(index, out);
#pragma unroll
        for (int h = first; h < BLOCKS / 4; ++h) t[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[p][h], out, t[h], 0, 0, 0);
    });
}
// the worst of four results, and whether all of them are safe (zeros included)
__device__ __forceinline__ unsigned worst_code(const wave_f32x4 &x) { return max(max(range_code(x[0]), range_code(x[1])), max(range_code(x[2]), range_code(x[3]))); }
__device__ __forceinline__ bool all_safe(const wave_f32x4 &x, unsigned lower = 0)
{
    return in_safe_range(range_code(x[0]), lower) && in_safe_range(range_code(x[1]), lower) && in_safe_range(range_code(x[2]), lower) &&
           in_safe_range(range_code(x[3]), lower);
}

// The largest of sixteen column sums of which each lane 16 g + i holds the part of column i in its own rows; infinity for NaN.
__device__ __forceinline__ float largest_column(float part)
{
    const unsigned u = __builtin_bit_cast(unsigned, part);
    const auto h = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const unsigned h0 = h[0], h1 = h[1];
    const unsigned m = __builtin_bit_cast(unsigned, __builtin_bit_cast(float, h0) + __builtin_bit_cast(float, h1));
    const auto f = __builtin_amdgcn_permlane32_swap(m, m, false, false);
    const unsigned f0 = f[0], f1 = f[1];
    float v = __builtin_bit_cast(float, f0) + __builtin_bit_cast(float, f1);
    v = v == v ? v : __builtin_inff();
    auto dpp = [](float x, auto ctrl) __attribute__((always_inline)) {
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value, 0xf, 0xf, true));
    };
    v = __builtin_fmaxf(v, dpp(v, std::integral_constant<int, 0xB1>{}));       // quad_perm 1,0,3,2
    v = __builtin_fmaxf(v, dpp(v, std::integral_constant<int, 0x4E>{}));       // quad_perm 2,3,0,1
    v = __builtin_fmaxf(v, dpp(v, std::integral_constant<int, 0x141>{}));      // row_half_mirror
    return __builtin_fmaxf(v, dpp(v, std::integral_constant<int, 0x140>{}));   // row_mirror
}

// W = L^-1 of a tile beside its factorisation (factor_tile64): wave w takes the columns 16 w .. 16 w + 15, sixteen right-hand
// sides of L y = e_j by the recurrence of solve_rows16, and the rows of group G of them as soon as that group of columns of L is
// finished.  Reciprocals for the quotients: W is an approximation.  It goes to memory in the order in which the product of the rows
// below wants its operand: entry (r, j) in piece 4 (r / 16) + j / 16 of 1 KiB, at [(r % 16) + 16 (j % 4)][(j / 4) % 4].  Behind the
// pieces, per wave, the largest column sum of |L| and of |W| over its columns (infinity for NaN).
constexpr int W_FLOATS = 64 * 64, W_ALL = W_FLOATS + 8;
struct InverseColumns {
    wave_f32x4 t[4];                                           // rows 16 H + 4 g + r of column 16 w + i, the running right-hand side
    float sum_L, sum_W;                                        // of column 16 w + i, this lane's rows
    __device__ __forceinline__ void start(int w, int lane)
    {
        const int i = lane & 15, g = lane >> 4;
#pragma unroll
        for (int H = 0; H < 4; ++H)
#pragma unroll
            for (int r = 0; r < 4; ++r) t[H][r] = H == w && 4 * g + r == i ? 1.0f : 0.0f;
        sum_L = sum_W = 0.0f;
    }
    // scratch: 16 x 20 floats of LDS of the wave's own
    template <int G, int LDD>
    __device__ __forceinline__ void group(const float (*T)[LDD], float *scratch, float *__restrict__ W, int w, int lane)
    {
        const int i = lane & 15, g = lane >> 4;
        wave_f32x4 x = {0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float l = T[16 * G + 4 * g + r][16 * w + i];
            sum_L += 16 * G + 4 * g + r >= 16 * w + i ? __builtin_fabsf(l) : 0.0f;
        }
        unrolled<4>([&](auto index) __attribute__((always_inline)) {
            constexpr int gk = decltype(index)::value, first = gk == 3 ? G + 1 : G;
            wave_f32x4 c = t[G], v;
            float l[4][4], a[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int e = 0; e <= j; ++e) l[j][e] = T[16 * G + 4 * gk + j][16 * G + 4 * gk + e];
#pragma unroll
            for (int H = first; H < 4; ++H) a[H] = T[16 * H + i][16 * G + 4 * gk + g];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                Pivot p;
                p.from_root(l[j][j]);
                v[j] = c[j] * p.r;
#pragma unroll
                for (int e = j + 1; e < 4; ++e) c[e] = __builtin_fmaf(-v[j], l[e][j], c[e]);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) x[j] = g == gk ? v[j] : x[j];
            if constexpr (first < 4) {
                const float out = -spread16<gk>(v);
#pragma unroll
                for (int H = first; H < 4; ++H) t[H] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[H], out, t[H], 0, 0, 0);
            }
        });
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            sum_W += __builtin_fabsf(x[r]);
            scratch[(4 * g + r) * 20 + i] = x[r];
        }
        wave_f32x4 piece;
#pragma unroll
        for (int q = 0; q < 4; ++q) piece[q] = scratch[i * 20 + 4 * q + g];
        *(wave_f32x4 *)(W + (4 * G + w) * 256 + 4 * lane) = piece;
    }
    // hint: see factor_tile64; it goes along as the sign of the sums of |L|
    __device__ __forceinline__ void finish(float *__restrict__ W, int w, int lane, bool hint)
    {
        const float largest_L = largest_column(sum_L), largest_W = largest_column(sum_W);
        if (lane == 0) {
            W[W_FLOATS + w] = hint ? -largest_L : largest_L;
            W[W_FLOATS + 4 + w] = largest_W;
        }
    }
};

// CHOL of a 64 x 64 tile in LDS by four waves: T holds S on entry (on and below the diagonal) and L on return, mirrored into
// its upper half.  Wave w keeps the rows 16 w .. 16 w + 15.  The columns go in four groups of sixteen; in the phase of group G
// every wave that has rows in or below it factors the 16 x 16 block on the diagonal for itself, beside its own rows of the group,
// so that pivots and coefficients come from the wave's own lanes and nothing is handed over inside a phase; between phases
// the finished columns cross LDS.  Then the terms of group G are taken out of group G + 1, those of the groups before
// it having gone beside phase G.
// A wave that is done mirrors the columns of its group into the upper half and goes on with its columns of the inverse
// (InverseColumns; W == nullptr: none is computed); what the last group of rows of that needs is left for finish_inverse().
// beside(G, w): called in the phases G = 1 .. 3 by every wave w < G; the first G groups of columns and of rows are finished then
// (called again where the tile is started over).  scratch: LDS, FACTOR_SCRATCH floats.
// GROUPS: of a tile padded with the identity from column 16 GROUPS on, only so many groups of columns (and of rows).
// Roots and quotients come from estimates and exact remainders (Pivot).  At the end of every phase the wave looks at what came out,
// and the tile is started over with the compiler's root and division, which takes 10 us, where something may not be IEEE's:
// a result that is not zero and outside [2^-50, 2^50] or, as long as every pivot is at least 2^-24, outside [2^-76, 2^50] (what
// counts is that the product of a quotient and its divisor is at least 2^-100).  hint: the tile before it was like that, begin with root and
// division; returned: whether this one was, or began so.  A covariance whose entries fall to nothing within a tile is then
// factored once per tile: n = 4096, entries 0.5^|i - j|, 1725 us with a second pass per tile, 1041 now; exp(-((i - j) / 3)^2 / 2), 2057 and 1634
// (with root and division always, a row to a lane in one wave: 1151 and 1617, and 1151 in place of 1021 where all lies in the range).
// A barrier must have made S visible; ends with one.  unsafe: two bytes in LDS, 0 on entry.
constexpr int FACTOR_SCRATCH = 4 * 320 + 64 * 64;
template <int GROUPS, int LDD, class Beside>
__device__ __forceinline__ bool factor_tile64(float (*T)[LDD], char *unsafe, float *scratch, float *W, InverseColumns &inverse, int tid, bool hint, Beside beside)
{
    float *const saved = scratch + 4 * 320;                    // S, to start from again
    static_assert(LDD >= 68, "four columns of padding take the stores that go nowhere");
    const int lane = tid & 63, i = lane & 15, g = lane >> 4, w = __builtin_amdgcn_readfirstlane(tid >> 6), own_row = 16 * w + i;
    float *const row = &T[own_row][0];
    auto lane_value = [](float v, int l) __attribute__((always_inline)) {
        return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
    };
    auto mirror = [&](auto group) __attribute__((always_inline)) {             // T[16 G + c][r] <- L[r][16 G + c], r = lane > 16 G + c
        constexpr int G = decltype(group)::value;
        wave_f32x4 m[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) m[q] = *(const wave_f32x4 *)&T[lane][16 * G + 4 * q];
#pragma unroll
        for (int c = 0; c < 16; ++c) *(16 * G + c < lane ? &T[16 * G + c][lane] : &T[lane][64]) = m[c / 4][c % 4];
    };
    auto factor = [&](auto by_pivots) __attribute__((always_inline)) {
        constexpr bool PIVOTS = decltype(by_pivots)::value;
        wave_f32x4 s[GROUPS], sd[GROUPS];                      // S of the own rows and of the blocks on the diagonal, group by group
        float mine[NBLK];                                      // the own rows of L, spread: lane 16 q + i of block b is column 4 b + q
#pragma unroll
        for (int G = 0; G < GROUPS; ++G) {
            s[G] = *(const wave_f32x4 *)(row + 16 * G + 4 * g);
            sd[G] = *(const wave_f32x4 *)&T[16 * G + i][16 * G + 4 * g];
            // (kept for the second try; in registers they made the kernel spill into accumulation registers)
            if (PIVOTS) *(wave_f32x4 *)(saved + 64 * own_row + 16 * G + 4 * g) = s[G];
        }
        __syncthreads();
        if (W) inverse.start(w, lane);
        unrolled<GROUPS>([&](auto group) __attribute__((always_inline)) {
            constexpr int G = decltype(group)::value, NEXT = G < GROUPS - 1 ? G + 1 : G;
            if (w >= G && w < GROUPS) {                                      // uniform over the wave
                float ahead[NBLK];                             // minus rows of group G + 1, the columns before group G
                if constexpr (G > 0) {
                    float a[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) a[q] = -T[16 * G + i][16 * (G - 1) + 4 * q + g];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        sd[G] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[q], -a[q], sd[G], 0, 0, 0);
                        s[G] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[q], mine[4 * (G - 1) + q], s[G], 0, 0, 0);
                    }
                }
                if constexpr (G < GROUPS - 1) {
#pragma unroll
                    for (int k = 0; k < 4 * G; ++k) ahead[k] = -T[16 * (G + 1) + i][4 * k + g];
                }
                wave_f32x4 d = sd[G], t = s[G];
                unrolled<4>([&](auto index) __attribute__((always_inline)) {
                    constexpr int gk = decltype(index)::value;
                    wave_f32x4 cd = d, ct = t, xd, xt;         // (copies: the other lanes hold other columns)
                    // (the next pivot needs nothing but its own row: formed from that in every lane, one lane's is read)
                    float own = cd[0];
                    unrolled<4>([&](auto column) __attribute__((always_inline)) {
                        constexpr int j = decltype(column)::value, n = 4 * gk + j;
                        __builtin_amdgcn_sched_barrier(0);
                        const float square = lane_value(own, 20 * gk + j);     // row 4 gk + j, in the lanes that hold this column
                        float pivot, qd, qt;
                        if (PIVOTS) {
                            Pivot p;
                            p.from_square(square);
                            pivot = p.d;
                            qd = p.quotient(cd[j]);
                            if (j < 3) own = __builtin_fmaf(-qd, qd, cd[j + 1]);
                            qt = p.quotient(ct[j]);
                        } else {
                            pivot = __builtin_sqrtf(square);
                            qd = cd[j] / pivot;
                            if (j < 3) own = __builtin_fmaf(-qd, qd, cd[j + 1]);
                            qt = ct[j] / pivot;
                        }
#pragma unroll
                        for (int e = j + 1; e < 4; ++e) {
                            const float l = lane_value(qd, 20 * gk + e);
                            cd[e] = __builtin_fmaf(-qd, l, cd[e]);
                            ct[e] = __builtin_fmaf(-qt, l, ct[e]);
                        }
                        xd[j] = qd;
                        xt[j] = own_row == 16 * G + n ? pivot : qt;
                        if constexpr (G < GROUPS - 1 && n / 2 < 4 * G) {                // one of the terms of the groups before out of group G + 1
                            constexpr int k = n / 2;
                            if constexpr (n % 2 == 0) sd[NEXT] = __builtin_amdgcn_mfma_f32_16x16x4f32(ahead[k], -ahead[k], sd[NEXT], 0, 0, 0);
                            else s[NEXT] = __builtin_amdgcn_mfma_f32_16x16x4f32(ahead[k], mine[k], s[NEXT], 0, 0, 0);
                        }
                    });
                    *(wave_f32x4 *)(row + (g == gk ? 16 * G + 4 * gk : 64)) = xt;    // (the other lanes': into the padding)
                    const float spread_d = -spread16<gk>(xd);
                    mine[4 * G + gk] = spread16<gk>(xt);
                    if constexpr (gk < 3) {
                        d = __builtin_amdgcn_mfma_f32_16x16x4f32(spread_d, -spread_d, d, 0, 0, 0);
                        t = __builtin_amdgcn_mfma_f32_16x16x4f32(spread_d, mine[4 * G + gk], t, 0, 0, 0);
                    }
                });
                if (PIVOTS) {
                    // Is everything safe?  (Each wave looks at its own rows; what lies above the diagonal is nobody's.)
                    wave_f32x4 seen = *(const wave_f32x4 *)(row + 16 * G + 4 * g);
#pragma unroll
                    for (int r = 0; r < 4; ++r) seen[r] = own_row >= 16 * G + 4 * g + r ? seen[r] : 1.0f;
                    if (__builtin_expect(__builtin_amdgcn_ballot_w64(worst_code(seen) > SAFE_SPAN) != 0, 0)) {
                        if (!all_safe(seen)) {
                            // (zeros come out above every limit less one)
                            unsigned low = ~0u, high = 0;
#pragma unroll
                            for (int r = 0; r < 4; ++r) {
                                const unsigned twice = __builtin_bit_cast(unsigned, seen[r]) << 1;
                                low = min(low, twice - 1);
                                high = max(high, twice);
                            }
                            unsafe[0] = 1;
                            if (low < ((127u - 76u) << 24) - 1 || high > (127u + 50u) << 24) unsafe[1] = 1;
                        }
                    }
                }
            } else {
                constexpr int before = G > 0 ? G - 1 : 0;
                if (w == before) mirror(std::integral_constant<int, before>{});
                if (W) inverse.template group<before>(T, scratch + 320 * w, W, w, lane);
                if (w < G) beside(group, w);
            }
            __syncthreads();
        });
    };
    bool again = hint;
    if (!again) {
        factor(std::true_type{});
        if (__builtin_expect(*(volatile char *)unsafe != 0, 0)) {
            again = ((volatile char *)unsafe)[1] != 0 || __builtin_amdgcn_ballot_w64(lane < 16 * GROUPS && T[lane][lane] < 0x1p-24f) != 0;
            __syncthreads();                                   // (every wave has looked at the pivots)
            if (again) {
#pragma unroll
                for (int G = 0; G < GROUPS; ++G) *(wave_f32x4 *)(row + 16 * G + 4 * g) = *(const wave_f32x4 *)(saved + 64 * own_row + 16 * G + 4 * g);
                __syncthreads();
            }
        }
    }
    if (__builtin_expect(again, 0)) factor(std::false_type{});
    if (w == 0) mirror(std::integral_constant<int, GROUPS - 1>{});
    __syncthreads();
    return again;
}
template <int LDD>
__device__ __forceinline__ void finish_inverse(const float (*T)[LDD], float *scratch, float *W, InverseColumns &inverse, int tid, bool hint)
{
    const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    inverse.group<3>(T, scratch + 320 * w, W, w, lane);
    inverse.finish(W, w, lane, hint);
}

}  // namespace cyc
