// tsqr_panel.h -- one panel of a Householder factorization on the FP64 matrix
// cores: the building block of the leaves and of the reduction tree.
//
// R := R-factor of [R; C], R an NC x NC triangle in LDS (packed by rows), C a
// block of 16 RB rows in the registers of one wavefront, four columns (a panel)
// at a time.  With X = C(:, 4P..4P+3), the four reflectors of the panel
//     v_j = [e_j; s_j x_j],   x_j = X(:, j) after the panel's reflectors before j
// need only inner products of X with the trailing columns, never the columns
// themselves:
//   1. G = X^T [X, C_trailing], one matrix product over the rows of C;
//   2. per reflector j, with sigma^2 = G(j, j) and d = G(j, :),
//        beta = -sgn sqrt(alpha^2 + sigma^2),  w = R(j, :) + s d,
//        R(j, :) -= tau w,   f = tau s w,
//      and the products that are left follow x_i := x_i - f_i x_j and
//      c := c - f x_j:   G(i, :) -= f_i G(j, :) + f (G(j, i) - f_i sigma^2);
//   3. C_trailing -= X F, one matrix product, with F from f by back
//      substitution (x_j in terms of the columns of X).
// Steps 1 and 3 are the arithmetic (2 m n^2 flops over a whole matrix); step 2
// works on 4 x NC numbers, one column per lane, with no cross-lane reduction
// and no exchange through LDS, so a panel has one dependent chain of four
// reflectors instead of four chains with a reduction over the rows in each.
//
// Step 2 computes sigma_i^2 from inner products of columns that still contain
// their components along x_j, j < i, so it loses accuracy by the factor
//     growth = sum_j (f_i ||x_j||)^2 / (alpha_i^2 + sigma_i^2).
// Where growth exceeds kMaxGrowth, or where a sigma_i^2 came out as no normal
// number, the result is not used: the panel's own four columns are factored one
// after the other (panel_columns), each from a fresh sum of squares, and steps 1
// and 3 are done with the vectors found (panel_trailing).  That is the plain
// Householder step, so nothing is assumed about C; the bound only decides how
// much work a panel takes (uniform or moderately conditioned columns never
// reach it).  Starting again from fresh inner products behind every column whose
// growth was over the limit, with all other columns carried along, took up to five
// passes a panel (200001 x 37, eight decades, FP64: 286 us, 227 now; 4000 x 12,
// six decades: 72 us, 39 now).
//
// Register layout.  The matrix instruction is the 4x4x4 FP64 product with four
// independent blocks, D_b = A_b B_b + C_b.  Writing lane l as 16 d2 + 4 d1 + d0,
// block b lies in the lanes with d1 = b, and
//     A_b(i, k) from lane (d2 = k, d0 = i),  B_b(k, j) from lane (d2 = k, d0 = j),
//     D_b(i, j) to lane (d2 = i, d0 = j).
// c[rb][s] holds rows 16 rb + 4 d1 + d2 of columns 4 s + d0.  So a register
// of C is a B operand (and a register of X an A operand) of step 1 as it stands
// and the C/D operand of step 3: the trailing columns never move.  Only X moves,
// d2 <-> d0, through LDS, to be the A operand of step 3.  The four blocks of G
// are partial sums; they are added within the 16-lane rows by DPP and the result
// is transposed to one column per lane with the row swaps of gfx950.
#pragma once

#include <hip/hip_runtime.h>

#include "tsqr_internal.h"

namespace tsqr {
namespace dev {

using float4v = float __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double mfma4(double a, double b, double c)
{
    return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ float4v mfma4(float a, float b, float4v c)
{
    return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 0, 0, 0);
}

// Placed between matrix instructions and a branch.  Reading a matrix result
// needs up to 9 wait states that the compiler has to insert.  It does so
// within a basic block, but a register copy that its allocator placed at the
// start of the block behind a branch was found reading the result of the last
// instruction before that branch with one wait state between, and took the old
// value.
__device__ __forceinline__ void mfma_settle()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 7\n\ts_nop 1");
    __builtin_amdgcn_sched_barrier(0);
}

// The registers of a chunk of 16 RPL rows and 4 NS columns, and where they lie:
// register (r, s) holds row 16 r + p, column 4 s + q of the lane (q, p).
template <typename T, int RPL, int NS>
struct Chunk;

template <int RPL, int NS>
struct Chunk<double, RPL, NS> {
    double v[RPL][NS];
    __device__ __forceinline__ double get(int r, int s) const { return v[r][s]; }
    __device__ __forceinline__ void put(int r, int s, double x) { v[r][s] = x; }
    static __device__ __forceinline__ int q(int lane) { return lane & 3; }
    static __device__ __forceinline__ int p(int lane) { return (lane & 12) + (lane >> 4); }
};

template <int RPL, int NS>
struct Chunk<float, RPL, NS> {
    static constexpr int RV = (RPL + 3) / 4;     // four rows make up one accumulator
    float4v v[RV][NS];
    __device__ __forceinline__ float get(int r, int s) const { return v[r / 4][s][r % 4]; }
    __device__ __forceinline__ void put(int r, int s, float x) { v[r / 4][s][r % 4] = x; }
    static __device__ __forceinline__ int q(int lane) { return lane & 3; }
    static __device__ __forceinline__ int p(int lane) { return lane >> 2; }
};

// Slot s of a chunk as a chunk of its own
template <typename T, int RB, int NS>
__device__ __forceinline__ Chunk<T, RB, 1> slot_of(const Chunk<T, RB, NS>& c, int s)
{
    Chunk<T, RB, 1> x;
#pragma unroll
    for (int r = 0; r < RB; ++r) x.put(r, 0, c.get(r, s));
    return x;
}

// LDS work area of one wavefront.  FP64: F (4 rows, stride kFStride so that the
// four rows read together lie in different banks), then X with d2 and d0
// exchanged.  FP32: F, the four coefficients of a column together.
constexpr int kFStride = 68;
// FP64: position of (d2 = k, d1, d0 = i) of a row block of X at kXOff(k) + 4 d1 + i,
// with the four k apart so that neither the writes (i varies slowest over the
// lanes) nor the reads (k slowest) of half a wavefront meet in a bank
constexpr int kXBlock = 84;
__device__ __forceinline__ int x_offset(int k) { return 18 * (k & 1) + 48 * (k >> 1); }
template <typename T, int RPL>
struct PanelLds {
    static constexpr int kElems = sizeof(T) == 8 ? 4 * kFStride + RPL * kXBlock : 4 * kWave;
};

// Row blocks of 16 of a triangle as the bottom operand of a merge
template <typename T, int NC>
struct MergeRows {
    static constexpr int RB = sizeof(T) == 8 ? (4 * Slots<NC>::NS + 15) / 16 : 4;
};

// The limit trades accuracy against panels done one column at a time where
// columns are nearly dependent.  FP64, singular values over six decades: 4000 x 30
// at limit 10 faster than one column at a time throughout, at 4 slower by 15%;
// error of R against an 80-bit reference at 4000 x 20 1.15 and 0.83 times that of
// one column at a time.  Columns of moderate condition never reach either.
constexpr int kMaxGrowth = 10;

// old with the banks (quads of a 16-lane row) in BANKS replaced by x moved by CTRL
template <int CTRL, int BANKS>
__device__ __forceinline__ double dpp_into(double old, double x)
{
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(old), __double2loint(x), CTRL, 0xF, BANKS, false);
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(old), __double2hiint(x), CTRL, 0xF, BANKS, false);
    return __hiloint2double(hi, lo);
}
template <int CTRL, int BANKS>
__device__ __forceinline__ float dpp_into(float old, float x)
{
    return __int_as_float(
        __builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(x), CTRL, 0xF, BANKS, false));
}

// Sums over the four quads of each 16-lane row of a, b, c, d: the sum of a in
// quad 0, of b in quad 1, of c in quad 2, of d in quad 3.
__device__ __forceinline__ double quad_sums(double a, double b, double c, double d)
{
    // ac: quads 0, 1 hold a0 + a2, a1 + a3; quads 2, 3 hold c0 + c2, c1 + c3
    const double ac = dpp_into<0xE4, 0xC>(a, c) + dpp_into<0x128, 0xC>(dpp_mov<0x128>(a), c);
    const double bd = dpp_into<0xE4, 0xC>(b, d) + dpp_into<0x128, 0xC>(dpp_mov<0x128>(b), d);
    // even quads add their right neighbour in ac, odd quads their left one in bd
    return dpp_into<0xE4, 0xA>(ac, bd) + dpp_into<0x124, 0xA>(dpp_mov<0x12C>(ac), bd);
}
// In FP32 an addition takes its operand through DPP, so adding first and
// merging afterwards is shorter.  All four rows of the accumulators step by
// step: a DPP operand may be read only three instructions after it is written,
// and the other rows fill that gap (one row after the other, a panel's sums
// held 38 wait instructions; 4117 x 28: 69.0 us, now 64.8).  Chunks of more
// than 8 rows per lane run two wavefronts to a SIMD, which hides the waits, and
// have no registers for it: they go row by row (Rows; 2^22 x 50 with 12 rows
// per lane: 638 us step by step, 625 row by row).
template <bool Rows>
__device__ __forceinline__ float4v quad_sums(float4v a, float4v b, float4v c, float4v d)
{
    float4v ac, bd, x;
    if constexpr (Rows) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float e = dpp_into<0xE4, 0xC>(a[i] + dpp_mov<0x128>((float)a[i]), c[i] + dpp_mov<0x128>((float)c[i]));
            const float o = dpp_into<0xE4, 0xC>(b[i] + dpp_mov<0x128>((float)b[i]), d[i] + dpp_mov<0x128>((float)d[i]));
            ac[i] = dpp_into<0xE4, 0xA>(e + dpp_mov<0x12C>(e), o + dpp_mov<0x124>(o));
        }
        return ac;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) ac[i] = a[i] + dpp_mov<0x128>((float)a[i]);
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = c[i] + dpp_mov<0x128>((float)c[i]);
#pragma unroll
    for (int i = 0; i < 4; ++i) ac[i] = dpp_into<0xE4, 0xC>((float)ac[i], (float)x[i]);
#pragma unroll
    for (int i = 0; i < 4; ++i) bd[i] = b[i] + dpp_mov<0x128>((float)b[i]);
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = d[i] + dpp_mov<0x128>((float)d[i]);
#pragma unroll
    for (int i = 0; i < 4; ++i) bd[i] = dpp_into<0xE4, 0xC>((float)bd[i], (float)x[i]);
#pragma unroll
    for (int i = 0; i < 4; ++i) ac[i] = ac[i] + dpp_mov<0x12C>((float)ac[i]);
#pragma unroll
    for (int i = 0; i < 4; ++i) bd[i] = bd[i] + dpp_mov<0x124>((float)bd[i]);
#pragma unroll
    for (int i = 0; i < 4; ++i) ac[i] = dpp_into<0xE4, 0xA>((float)ac[i], (float)bd[i]);
    return ac;
}

// The sum over the four quads of each 16-lane row, in all four.
template <typename T>
__device__ __forceinline__ T quad_sum(T a)
{
    a = a + dpp_mov<0x128>(a);
    return a + dpp_mov<0x124>(a);
}

// a.rows 1, 3 <-> b.rows 0, 2 (16-lane rows)
__device__ __forceinline__ void swap_rows16(double& a, double& b)
{
    const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
    a = __hiloint2double((int)hi[0], (int)lo[0]);
    b = __hiloint2double((int)hi[1], (int)lo[1]);
}
__device__ __forceinline__ void swap_rows16(float& a, float& b)
{
    const auto x = __builtin_amdgcn_permlane16_swap(__float_as_int(a), __float_as_int(b), false, false);
    a = __int_as_float((int)x[0]);
    b = __int_as_float((int)x[1]);
}
// a.rows 2, 3 <-> b.rows 0, 1
__device__ __forceinline__ void swap_rows32(double& a, double& b)
{
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
    a = __hiloint2double((int)hi[0], (int)lo[0]);
    b = __hiloint2double((int)hi[1], (int)lo[1]);
}
__device__ __forceinline__ void swap_rows32(float& a, float& b)
{
    const auto x = __builtin_amdgcn_permlane32_swap(__float_as_int(a), __float_as_int(b), false, false);
    a = __int_as_float((int)x[0]);
    b = __int_as_float((int)x[1]);
}

// 4 x 4 transpose of the quads' registers and lanes: out[k] of lane i is in[i]
// of lane k (lanes numbered within a quad).
__device__ __forceinline__ float4v quad_transpose(float4v x, int lane)
{
    const bool odd = lane & 1, high = lane & 2;
    // quad_perm [1,0,3,2] = 0xB1, [2,3,0,1] = 0x4E; the moves run in every lane, ahead of the selects
    const float x0 = x[0], x1 = x[1], x2 = x[2], x3 = x[3];
    const float m0 = dpp_mov<0xB1>(x0), m1 = dpp_mov<0xB1>(x1), m2 = dpp_mov<0xB1>(x2), m3 = dpp_mov<0xB1>(x3);
    const float a0 = odd ? m1 : x0, a1 = odd ? x1 : m0, a2 = odd ? m3 : x2, a3 = odd ? x3 : m2;
    const float b0 = dpp_mov<0x4E>(a0), b1 = dpp_mov<0x4E>(a1), b2 = dpp_mov<0x4E>(a2), b3 = dpp_mov<0x4E>(a3);
    return float4v{high ? b2 : a0, high ? b3 : a1, high ? a2 : b0, high ? a3 : b1};
}

// Step 1 of a panel: g[i] = X(:, i) . C(:, lane), one column per lane, for the
// columns of slots [S0, S1) of C (other lanes get values that nothing uses), X
// slot A of x.  Only the first RA row blocks take part.
template <int S0, int S1>
struct Groups {
    static constexpr int T0 = S0 / 4, T1 = (S1 + 3) / 4;         // live groups of 16 columns
    // slots outside [S0, S1) are not needed: any live one stands in
    static constexpr int live(int s) { return s < S0 ? S0 : (s >= S1 ? S1 - 1 : s); }
};

template <int A, int S0, int S1, int RA, int RB, int NX, int NS>
__device__ __forceinline__ void panel_products(const Chunk<double, RB, NX>& x, const Chunk<double, RB, NS>& c,
                                               double (&g)[4])
{
    using Gr = Groups<S0, S1>;
    constexpr int T0 = Gr::T0, T1 = Gr::T1;
    double G[NS];
#pragma unroll
    for (int rb = 0; rb < RA; ++rb)
        static_for<S0, S1>([&](auto sc) {
            constexpr int s = decltype(sc)::value;
            G[s] = mfma4(x.v[rb][A], c.v[rb][s], rb == 0 ? 0.0 : G[s]);
        });
    // add the four blocks; column 16 t + 4 b + j of row i of G to lane (d2 = i, d1 = b, d0 = j) of g[t]
    static_for<T0, T1>([&](auto tc) {
        constexpr int t = decltype(tc)::value, a = 4 * t;
        if constexpr (Gr::live(a) == Gr::live(a + 3))
            g[t] = quad_sum(G[Gr::live(a)]);
        else
            g[t] = quad_sums(G[Gr::live(a)], G[Gr::live(a + 1)], G[Gr::live(a + 2)], G[Gr::live(a + 3)]);
    });
    static_for<0, T0>([&](auto tc) { g[decltype(tc)::value] = g[T0]; });
    static_for<T1, 4>([&](auto tc) { g[decltype(tc)::value] = g[T1 - 1]; });
    // transpose t and d2
    swap_rows16(g[0], g[1]);
    swap_rows16(g[2], g[3]);
    swap_rows32(g[0], g[2]);
    swap_rows32(g[1], g[3]);
}

template <int A, int S0, int S1, int RA, int RB, int NX, int NS>
__device__ __forceinline__ void panel_products(const Chunk<float, RB, NX>& x, const Chunk<float, RB, NS>& c,
                                               float (&g)[4])
{
    using Gr = Groups<S0, S1>;
    constexpr int T0 = Gr::T0, T1 = Gr::T1;
    float4v G[NS];
    static_for<S0, S1>([&](auto sc) { G[decltype(sc)::value] = float4v{0.0f, 0.0f, 0.0f, 0.0f}; });
#pragma unroll
    for (int r = 0; r < RA; ++r)
        static_for<S0, S1>([&](auto sc) {
            constexpr int s = decltype(sc)::value;
            G[s] = mfma4((float)x.v[r / 4][A][r % 4], (float)c.v[r / 4][s][r % 4], G[s]);
        });
    // add the sixteen blocks: within the 16-lane rows, then over the rows, slot s
    // ending in quad s
    float4v t4[4];
    static_for<T0, T1>([&](auto tc) {
        constexpr int t = decltype(tc)::value, a = 4 * t;
        if constexpr (Gr::live(a) == Gr::live(a + 3)) {
#pragma unroll
            for (int i = 0; i < 4; ++i) t4[t][i] = quad_sum((float)G[Gr::live(a)][i]);
        } else {
            t4[t] = quad_sums<(RB > 8)>(G[Gr::live(a)], G[Gr::live(a + 1)], G[Gr::live(a + 2)], G[Gr::live(a + 3)]);
        }
    });
    static_for<0, T0>([&](auto tc) { t4[decltype(tc)::value] = t4[T0]; });
    static_for<T1, 4>([&](auto tc) { t4[decltype(tc)::value] = t4[T1 - 1]; });
    float u[4], v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float x = t4[0][i], y = t4[1][i];
        swap_rows16(x, y);
        u[i] = x + y;
    }
    if constexpr (T1 <= 2) {
        // no columns in the upper half of the lanes
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = u[i];
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float x = t4[2][i], y = t4[3][i];
            swap_rows16(x, y);
            v[i] = x + y;
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        swap_rows32(u[i], v[i]);
        g[i] = u[i] + v[i];
    }
}

// x_i . x_j of a panel's columns: entry (i, j) is read from one lane
template <int RA, int RB>
__device__ __forceinline__ void panel_gram(const Chunk<double, RB, 1>& x, double (&v)[4])
{
    double G = 0.0;
#pragma unroll
    for (int rb = 0; rb < RA; ++rb) G = mfma4(x.v[rb][0], x.v[rb][0], G);
    v[0] = quad_sum(G);
}
__device__ __forceinline__ double gram_entry(const double (&v)[4], int i, int j) { return lane_value(v[0], 16 * i + j); }

template <int RA, int RB>
__device__ __forceinline__ void panel_gram(const Chunk<float, RB, 1>& x, float (&v)[4])
{
    float4v G = float4v{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int r = 0; r < RA; ++r) G = mfma4((float)x.v[r / 4][0][r % 4], (float)x.v[r / 4][0][r % 4], G);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        float a = quad_sum((float)G[i]), b = a;
        swap_rows16(a, b);               // the other row of each pair of rows
        a = a + b;
        b = a;
        swap_rows32(a, b);
        v[i] = a + b;
    }
    v[3] = 0.0f;
}
__device__ __forceinline__ float gram_entry(const float (&v)[4], int i, int j) { return lane_value(v[i], j); }

// The reflectors of a panel (step 2), one column of [R; C] per lane, the panel's
// own NJ columns in the lanes from J0 on: g[j] are the inner products of X(:, j)
// with the lane's column, r[j] the panel's row j of R.
// Columns below lo are done already.  On return r holds the new rows, nf the
// coefficients -F in terms of the columns of X (zero for columns outside
// [lo, hi)), tau and s the reflectors' scalars, and the result is hi: NJ, or
// the column in front of which the panel was cut.
//
// With y = 1/sqrt(alpha^2 + sigma^2), z = |alpha| y and q = 1/(1 + z):
//     tau = 1 + z,  s = sgn y q,  tau s = sgn y,  R(j, :) - tau w = -(z R(j, :) + sgn y d).
// The diagonal entry takes the norm itself, S y with one Newton correction whose
// residual is that of alpha^2 + sigma^2, without the rounding of S: the roundings
// there are most of the error of an R whose diagonal is its largest part.  Mean
// relative error of R against an 80-bit reference, uniform entries, over that of one
// column at a time: FP64 20000 x 50 1.10, 100000 x 40 1.16, FP32 30000 x 8 1.11
// with S rounded and every correction added to G(i, i); 1.01, 0.96 and 1.02 so,
// for 1% of the time.
// y and q from the hardware estimates (about 2^-24 on gfx950 in FP64, 1 ulp in
// FP32) by one third-order step each, which leaves 2^-72 (FP32: second-order).
template <typename T>
__device__ __forceinline__ T refined_rcp(T u)
{
    const T q = hw_rcp(u);
    const T e = fmadd(-u, q, T(1));
    return fmadd(q, sizeof(T) == 8 ? fmadd(e, e, e) : e, q);
}

// The scalars of one reflector: z, q, sgn y (see above) and beta.  An S below
// the smallest normal number (rounding can leave it negative) still gives
// finite z, q and y; S = 0, a zero column below a zero alpha, gives z = 0.
template <typename T>
struct PanelScalars {
    T z, q, sy, beta;
};
template <typename T>
__device__ __forceinline__ PanelScalars<T> panel_scalars(T alpha, T sigma2, T S)
{
#pragma clang fp contract(off)
    PanelScalars<T> h;
    const T St = max_raw(S, Limits<T>::tiny);
    const T y0 = hw_rsq(St);
    const T t = St * y0;
    const T e = fmadd(-t, y0, T(1));
    const T c = e * (sizeof(T) == 8 ? fmadd(e, T(0.375), T(0.5)) : T(0.5));
    const T y = fmadd(y0, c, y0);
    h.z = absv(alpha) * y;
    h.q = refined_rcp(T(1) + h.z);
    h.sy = with_sign(y, sign_of(alpha));
    const T nrm = St * y;
    h.beta = with_sign(fmadd(T(0.5) * y, fmadd(alpha, alpha, fmadd(-nrm, nrm, sigma2)), nrm), sign_of(alpha) ^ 0x80000000u);
    return h;
}

// Reflector j of a panel on the lane's column: its row of R, the coefficient
// nf = -tau s w, and the products that are left, G(i, :) in g[i] + e[i].  n[j][i] is
// -f of column J0 + i, grow the sum over the reflectors of (f sigma)^2.  The first
// part of a correction may cancel G(i, i) and goes to it at once, with one
// rounding; the second is small and is summed apart, so that G(i, i), which is
// large beside both where columns are nearly orthogonal, is rounded once for
// all of them.
template <typename T, int J0, int NJ, int j, bool Mask>
__device__ __forceinline__ void panel_apply(const PanelScalars<T>& h, T sigma2, T (&g)[4], T (&r)[4], T (&nf)[4],
                                            T (&n)[4][4], T (&e)[4], T& grow, int lane)
{
#pragma clang fp contract(off)
    const T w = fmadd(h.sy * h.q, g[j], r[j]);
    r[j] = lane == J0 + j ? h.beta : fmadd(-h.z, r[j], -h.sy * g[j]);
    nf[j] = -h.sy * w;
    if constexpr (Mask) nf[j] = lane > J0 + j ? nf[j] : T(0);
    if constexpr (j + 1 < NJ) {
        const T p = nf[j] * sigma2;
        const T hv = g[j] + p;            // x_j . (the lane's column after reflector j)
        grow = fmadd(nf[j], p, grow);
#pragma unroll
        for (int i = j + 1; i < NJ; ++i) {
            n[j][i] = lane_value(nf[j], J0 + i);
            const T hi = lane_value(hv, J0 + i);
            g[i] = fmadd(n[j][i], g[j], g[i]);
            e[i] = j == 0 ? nf[j] * hi : fmadd(nf[j], hi, e[i]);
        }
    }
}

// F: c - sum_j f_j x_j with x_j = X(:, j) - sum_{i<j} f_ij x_i
template <typename T, int NJ>
__device__ __forceinline__ void panel_coefficients(T (&nf)[4], const T (&n)[4][4])
{
#pragma unroll
    for (int j = NJ - 2; j >= 0; --j)
#pragma unroll
        for (int i = j + 1; i < NJ; ++i) nf[j] = fmadd(n[j][i], nf[i], nf[j]);
}

// All reflectors of a panel at once.  Returns false, with g and r spoilt, where
// the panel has to be done one column at a time: growth over the limit, or a
// sum of squares below the smallest normal number.  A zero column below a zero
// alpha (every column past n is one) does no harm here: its row of R is zero,
// and with tau = 0 its reflector is the identity.  With WQ, nf is valid (zero
// where a reflector does not act) in the lanes of the panel's own columns too.
template <typename T, int J0, int NJ, bool WQ>
__device__ __forceinline__ bool panel_reflectors(T (&g)[4], T (&r)[4], T (&nf)[4], T (&tau)[4], T (&s)[4], int lane)
{
    T n[4][4], e[4], alpha[4], sigma2[4];
    T grow = T(0);
    int least = 0;                        // the least sigma^2 (by its high word: integers stay on the scalar unit)
    uint64_t over = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) nf[j] = tau[j] = s[j] = T(0);
    static_for<0, NJ>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        if constexpr (j > 0) g[j] = g[j] + e[j];
        alpha[j] = lane_value(r[j], J0 + j);
        sigma2[j] = lane_value(g[j], J0 + j);
        const T S = fmadd(alpha[j], alpha[j], sigma2[j]);
        least = j == 0 || high_word(sigma2[j]) < least ? high_word(sigma2[j]) : least;
        if constexpr (j > 0)
            over |= __builtin_amdgcn_ballot_w64(!(grow <= T(kMaxGrowth) * S)) & ((uint64_t)1 << (J0 + j));
        const PanelScalars<T> h = panel_scalars(alpha[j], sigma2[j], S);
        s[j] = h.sy * h.q;
        tau[j] = T(1) + h.z;
        panel_apply<T, J0, NJ, j, WQ>(h, sigma2[j], g, r, nf, n, e, grow, lane);
    });
    panel_coefficients<T, NJ>(nf, n);
    bool good = over == 0;
    if (least < Limits<T>::tiny_high) [[unlikely]] {
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            if (__builtin_amdgcn_ballot_w64(sigma2[j] < Limits<T>::tiny) != 0) {
                if (__builtin_amdgcn_ballot_w64(sigma2[j] != T(0) || alpha[j] != T(0)) != 0) good = false;
                r[j] = lane == J0 + j ? alpha[j] : r[j];
                s[j] = tau[j] = T(0);
            }
    }
    return good;
}

// The sum over the lanes of a column (those that agree in lane & 3), in all of them
template <typename T>
__device__ __forceinline__ T column_sum(T x)
{
    T a = quad_sum(x), b = a;
    swap_rows16(a, b);                   // the other row of each pair of rows
    a = a + b;
    b = a;
    swap_rows32(a, b);
    return a + b;
}

// The panel x one column at a time, its first RA row blocks, nj columns: they become the vectors x_j, the panel's own part of R (row0: its
// first row in LDS, of `row` entries) becomes that of the result, and the
// scalars z, sgn y and s of reflector j go to work[4 j ..] (the place of F, which
// is written later).  The result tells whether the growth stayed below the limit and
// every sum of squares was a normal number, so that all columns at once would
// have done.  Before step j the columns have been turned by j lanes within
// their quads, so that one loop body, which finds the pivot column in lane 0 of each
// quad, serves all four; x_j is fetched twice by DPP rather than kept, which
// would take the registers that kernels at the limit do not have.
template <typename T, int RA, int RB>
__device__ __forceinline__ bool panel_columns(Chunk<T, RB, 1>& c, T* row0, int row, int nj, T* work, int lane)
{
#pragma clang fp contract(off)
    const int q = c.q(lane);
    T grow = T(0);
    bool calm = true;
    T* Rj = row0;                        // entry (J0 + j, J0 + k) is Rj[k]
#pragma nounroll
    for (int j = 0; j < 4; ++j) {
        if (j < nj) {
            const int k = (q + j) & 3;   // the lane's column at this step
            T d = T(0);
#pragma unroll
            for (int r = 0; r < RA; ++r) d = fmadd(dpp_mov<0x00>(c.get(r, 0)), c.get(r, 0), d);
            d = column_sum(d);
            const T rk = k < row ? Rj[k] : T(0);
            const T alpha = lane_value(rk, 0), sigma2 = lane_value(d, 0);
            const T S = fmadd(alpha, alpha, sigma2);
            PanelScalars<T> h = panel_scalars(alpha, sigma2, S);
            const bool normal = __builtin_amdgcn_ballot_w64(sigma2 >= Limits<T>::tiny) != 0;
            if (!normal) {               // an identity reflector
                h.z = T(-1);
                h.sy = T(0);
                h.beta = alpha;
            }
            calm = calm && (__builtin_amdgcn_ballot_w64(!(grow <= T(kMaxGrowth) * S)) & 1) == 0 &&
                   (normal || __builtin_amdgcn_ballot_w64(sigma2 != T(0) || alpha != T(0)) == 0);
            const T s = h.sy * h.q;
            const T f = h.sy * fmadd(s, d, rk);
#pragma unroll
            for (int r = 0; r < RA; ++r) {
                T own = c.get(r, 0);
                asm volatile("" : "+v"(own));
                const T x = dpp_mov<0x00>(own);
                c.put(r, 0, k > j ? fmadd(-f, x, own) : own);    // (0 times a NaN is one)
            }
            grow = k > j ? fmadd(f, f * sigma2, grow) : grow;
            if (lane < 4 && k >= j && k < row) Rj[k] = k == j ? h.beta : fmadd(-h.z, rk, -h.sy * d);
            if (lane == 0) {
                work[4 * j] = h.z;
                work[4 * j + 1] = h.sy;
                work[4 * j + 2] = s;
            }
            lds_order();
            Rj += row - 1 - j;
        }
        // quad_perm [1,2,3,0]
        grow = dpp_mov<0x39>(grow);
#pragma unroll
        for (int r = 0; r < RA; ++r) c.put(r, 0, dpp_mov<0x39>(c.get(r, 0)));
    }
    return calm;
}

// The columns after such a panel: their rows of R and the coefficients nf, from
// the inner products g with its vectors and those among them (v).
template <typename T, int J0, int NJ>
__device__ __forceinline__ void panel_trailing(const T* work, const T (&v)[4], T (&g)[4], T (&r)[4], T (&nf)[4],
                                               T (&tau)[4], T (&s)[4], int lane)
{
#pragma clang fp contract(off)
#pragma unroll
    for (int j = 0; j < 4; ++j) nf[j] = tau[j] = s[j] = T(0);
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const T z = work[4 * j], sy = work[4 * j + 1];
        s[j] = work[4 * j + 2];
        tau[j] = T(1) + z;
        nf[j] = -sy * fmadd(s[j], g[j], r[j]);
        r[j] = lane < J0 + 4 ? r[j] : fmadd(-z, r[j], -sy * g[j]);
#pragma unroll
        for (int i = j + 1; i < NJ; ++i) g[i] = fmadd(nf[j], gram_entry(v, j, i), g[i]);
    }
}

// The lane's own column's entry of an array over the panel's columns
template <typename T>
__device__ __forceinline__ T of_column(const T (&s)[4], int lane)
{
    const int q = lane & 3;
    return q == 0 ? s[0] : q == 1 ? s[1] : q == 2 ? s[2] : s[3];
}

// Step 3 of a panel: the columns of slot s (and, for WQ, the panel's own
// reflectors) from F in LDS and X in the layout of an A operand.
template <typename T, int RA>
struct PanelUpdate;

template <int RA>
struct PanelUpdate<double, RA> {
    double xt[RA];
    const double* fr;
    template <typename C>
    static __device__ __forceinline__ void stage(const C& c, int P, double* work, int lane)
    {
        double* x = work + 4 * kFStride + x_offset(lane & 3) + (lane & 12) + (lane >> 4);
#pragma unroll
        for (int rb = 0; rb < RA; ++rb) x[rb * kXBlock] = c.v[rb][P];
    }
    static __device__ __forceinline__ void put_f(double* work, int lane, const double (&nf)[4])
    {
#pragma unroll
        for (int j = 0; j < 4; ++j) work[j * kFStride + lane] = nf[j];
    }
    // X, staged before, in the layout of an A operand
    template <typename C>
    __device__ __forceinline__ void fetch(const C&, int, const double* work, int lane)
    {
        fr = work + (lane >> 4) * kFStride + (lane & 3);
        const double* x = work + 4 * kFStride + x_offset(lane >> 4) + (lane & 15);
#pragma unroll
        for (int rb = 0; rb < RA; ++rb) xt[rb] = x[rb * kXBlock];
    }
    template <typename C>
    __device__ __forceinline__ void apply(C& c, int s) const
    {
        const double f = fr[4 * s];
#pragma unroll
        for (int rb = 0; rb < RA; ++rb) c.v[rb][s] = mfma4(xt[rb], f, c.v[rb][s]);
    }
    // the columns of slot s, moved to slot s - 1
    template <typename C>
    __device__ __forceinline__ void apply_shift(C& c, int s) const
    {
        const double f = fr[4 * s];
#pragma unroll
        for (int rb = 0; rb < RA; ++rb) c.v[rb][s - 1] = mfma4(xt[rb], f, c.v[rb][s]);
    }
    // row block rb of the vectors v_j = s_j x_j, x_j = X(:, j) + sum_{i<j} nf_i(J0 + j) X(:, i)
    template <typename Keep>
    __device__ __forceinline__ void reflectors(int P, int lane, const double (&s)[4], Keep&& keep) const
    {
        const int d0 = lane & 3, d2 = lane >> 4;
        const double sd = of_column(s, lane);
        const double f = d2 < d0 ? fr[4 * P] * sd : (d2 == d0 ? sd : 0.0);
        double v[RA];
#pragma unroll
        for (int rb = 0; rb < RA; ++rb) v[rb] = mfma4(xt[rb], f, 0.0);
        mfma_settle();
#pragma unroll
        for (int rb = 0; rb < RA; ++rb) keep(rb, v[rb]);
    }
};

template <int RA>
struct PanelUpdate<float, RA> {
    static constexpr int RV = (RA + 3) / 4;
    float4v xt[RV];
    const float4v* fr;
    template <typename C>
    static __device__ __forceinline__ void stage(const C&, int, float*, int)
    {
    }
    static __device__ __forceinline__ void put_f(float* work, int lane, const float (&nf)[4])
    {
        reinterpret_cast<float4v*>(work)[lane] = float4v{nf[0], nf[1], nf[2], nf[3]};
    }
    template <typename C>
    __device__ __forceinline__ void fetch(const C& c, int P, const float* work, int lane)
    {
        fr = reinterpret_cast<const float4v*>(work) + (lane & 3);
#pragma unroll
        for (int r = 0; r < RV; ++r) xt[r] = quad_transpose(c.v[r][P], lane);
    }
    template <typename C>
    __device__ __forceinline__ void apply(C& c, int s) const
    {
        const float4v f = fr[4 * s];
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int r = 0; r < RV; ++r) c.v[r][s] = mfma4((float)xt[r][k], (float)f[k], c.v[r][s]);
    }
    template <typename C>
    __device__ __forceinline__ void apply_shift(C& c, int s) const
    {
        const float4v f = fr[4 * s];
#pragma unroll
        for (int r = 0; r < RV; ++r) c.v[r][s - 1] = mfma4((float)xt[r][0], (float)f[0], c.v[r][s]);
#pragma unroll
        for (int k = 1; k < 4; ++k)
#pragma unroll
            for (int r = 0; r < RV; ++r) c.v[r][s - 1] = mfma4((float)xt[r][k], (float)f[k], c.v[r][s - 1]);
    }
    template <typename Keep>
    __device__ __forceinline__ void reflectors(int P, int lane, const float (&s)[4], Keep&& keep) const
    {
        const int j = lane & 3;
        const float sd = of_column(s, lane);
        const float4v nf = fr[4 * P];
        float4v x[RV];
#pragma unroll
        for (int r = 0; r < RV; ++r) x[r] = float4v{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float f = k < j ? (float)nf[k] * sd : (k == j ? sd : 0.0f);
#pragma unroll
            for (int r = 0; r < RV; ++r) x[r] = mfma4((float)xt[r][k], f, x[r]);
        }
        mfma_settle();
#pragma unroll
        for (int r = 0; r < RA; ++r) keep(r, (float)x[r / 4][r % 4]);
    }
};

// One panel, see the top of the file.  Only the first RA row blocks are
// nonzero in the panel's columns.  Bit P of hard, kept from chunk to chunk, is set
// where the panel was last done one column at a time and its growth called for
// it: the columns of a matrix that are close to each other are so in every chunk,
// and the attempt to do them all at once is left out.  keep(rb, v, tau)
// receives the chunk part of the panel's reflectors where WQ is set: v = s_j x_j
// in the layout of c.
template <typename T, int NC, int RB, int RA, int P, bool WQ, typename Keep>
__device__ __forceinline__ void panel_step(Chunk<T, RB, Slots<NC>::NS>& c, T* Rs, T* work, unsigned& hard, Keep&& keep)
{
    constexpr int NS = Slots<NC>::NS;
    constexpr int J0 = 4 * P;
    constexpr int NJ = NC - J0 < 4 ? NC - J0 : 4;
    using Update = PanelUpdate<T, RA>;
    const int lane = lane_id();
    T* Rl = Rs + lane;
    // rows J0.. of R, one column per lane (lanes left of the diagonal and past
    // NC read other entries of the padded triangle; nothing uses them)
    T r[4], g[4], nf[4], tau[4], s[4];
    auto rows = [&] {
#pragma unroll
        for (int j = 0; j < NJ; ++j) r[j] = Rl[Tri<NC>::off(J0 + j) - (J0 + j)];
    };
    // (the lane passes through an opaque copy so that the compiler does not keep
    // the masks of every panel alive over the whole chunk)
    int col = lane;
    asm volatile("" : "+v"(col));
    Update up;
    bool columns = hard >> P & 1;
    if (!columns) [[likely]] {
        rows();
        Update::stage(c, P, work, lane);
        lds_order();
        panel_products<P, P, NS, RA>(c, c, g);
        columns = !panel_reflectors<T, J0, NJ, WQ>(g, r, nf, tau, s, col);
        up.fetch(c, P, work, lane);
    }
    if (columns) [[unlikely]] {
        // on a copy of the slot: in FP64 at one wavefront per SIMD the chunk
        // lies in registers that only the matrix instructions reach, and a panel
        // that could change it here would be moved out of them in either case
        // (2^22 x 50: 935 us against 870)
        Chunk<T, RB, 1> x = slot_of(c, P);
        const bool calm = panel_columns<T, RA>(x, Rs + Tri<NC>::off(J0), NC - J0, NJ, work, col);
        hard = calm ? hard & ~(1u << P) : hard | 1u << P;
        rows();
        Update::stage(x, 0, work, lane);
        lds_order();
        T v[4];
        panel_gram<RA>(x, v);
        if constexpr (P + 1 < NS) panel_products<0, P + 1, NS, RA>(x, c, g);
        panel_trailing<T, J0, NJ>(work, v, g, r, nf, tau, s, col);
        up.fetch(x, 0, work, lane);
        if constexpr (WQ) {
            const T sd = of_column(s, lane);
#pragma unroll
            for (int rb = 0; rb < RA; ++rb) keep(rb, sd * x.get(rb, 0), tau);
        }
    }
    // last row first: a lane left of a row's diagonal writes into the end of
    // the row before, which the next store writes again.
    if ((unsigned)(col - J0) < (unsigned)(NC - J0)) {
#pragma unroll
        for (int j = NJ - 1; j >= 0; --j) {
            Rl[Tri<NC>::off(J0 + j) - (J0 + j)] = r[j];
            asm volatile("" ::: "memory");
        }
    }
    Update::put_f(work, lane, nf);
    lds_order();
    static_for<P + 1, NS>([&](auto sc) { up.apply(c, decltype(sc)::value); });
    mfma_settle();
    if constexpr (WQ) {
        if (!columns) [[likely]]
            up.reflectors(P, lane, s, [&](int rb, T v) { keep(rb, v, tau); });
    }
    lds_order();
}

// ---- the operator on two triangles ---------------------------------------------
//
// R := qr([R; R2]), R packed in LDS, R2 in registers: the operator of section 2 in
// the structured form of Table 3 (a panel touches only the row blocks of R2 that
// reach its columns).  A merge runs its code once or a few times, so the fetch of
// instructions that are in no cache yet counts: fully unrolled (40 KB), a merge
// that a kernel ran for the first time took about twice its warm 14 us.  The
// panels of a row block K (four of them) therefore share one loop body: the
// current panel is always slot 0 and the lanes 0..3, every update moves its slot
// down by one (the matrix instruction writes where it likes), and the slots that
// run out at the end, at most three, are updated for nothing.

// Slot s of row block rb holds column block s + first(rb) when the merge begins.
// FP64 keeps the nonzero part only; the FP32 accumulator holds the four row blocks
// together.
template <typename T>
__device__ __forceinline__ constexpr int merge_first(int rb)
{
    return sizeof(T) == 8 ? 4 * rb : 0;
}

// The panels 4 K .. of row block K that hold a column before n.  Panels whose bit is set in close are done one
// column at a time without an attempt at all four.  With WQ the
// reflectors' R2 parts go to Vn (packed by rows) and their tau to tau_out.
template <typename T, int NC, int K, bool WQ>
__device__ __forceinline__ void merge_row_block(Chunk<T, MergeRows<T, NC>::RB, Slots<NC>::NS>& c, T* Rs, T* work,
                                                int n, unsigned close, T* Vn, T* tau_out)
{
    constexpr int NS = Slots<NC>::NS;
    constexpr int S = NS - 4 * K;                  // live slots at the start
    constexpr int RA = K + 1;
    using Update = PanelUpdate<T, RA>;
    const int lane = lane_id();
    const int q = c.q(lane), p = c.p(lane);
    T* Rl = Rs + lane;
    const int end = S < 4 ? NS : 4 * K + 4, last = panels_of(n) < end ? panels_of(n) : end;
    int P = 4 * K;
    if (4 * P >= kMinColumns<NC> && P >= last) return;
    // (once at least: registers that a loop may leave as they are get copied)
#pragma nounroll
    do {
        const int J0 = 4 * P;
        // offset of entry (J0 + j, J0 + lane) of the packed triangle, without the lane
        int at[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) at[j] = __builtin_amdgcn_readfirstlane(Tri<NC>::off(J0 + j) - j);
        T r[4], g[4], nf[4], tau[4], s[4];
        auto rows = [&] {
#pragma unroll
            for (int j = 0; j < 4; ++j) r[j] = Rl[at[j]];
            if constexpr (NC % 4 != 0) {
                // the columns past NC of the last slot stay zero
#pragma unroll
                for (int j = 0; j < 4; ++j) r[j] = lane < NC - J0 && J0 + j < NC ? r[j] : T(0);
            }
        };
        [[maybe_unused]] auto keep = [&](int rb, T v) {
            const int i = 16 * rb + p, k = J0 + q;
            if (i <= k && k < NC) Vn[Tri<NC>::off(i) + k - i] = v;
        };
        Update up;
        bool columns = close >> P & 1;
        if (!columns) [[likely]] {
            rows();
            Update::stage(c, 0, work, lane);
            lds_order();
            panel_products<0, 0, S, RA>(c, c, g);
            columns = !panel_reflectors<T, 0, 4, WQ>(g, r, nf, tau, s, lane);
            up.fetch(c, 0, work, lane);
        }
        if (columns) [[unlikely]] {
            Chunk<T, MergeRows<T, NC>::RB, 1> x = slot_of(c, 0);
            panel_columns<T, RA>(x, Rs + at[0], NC - J0, NC - J0 < 4 ? NC - J0 : 4, work, lane);
            rows();
            Update::stage(x, 0, work, lane);
            lds_order();
            T v[4];
            panel_gram<RA>(x, v);
            if constexpr (S > 1) panel_products<0, 1, S, RA>(x, c, g);
            panel_trailing<T, 0, 4>(work, v, g, r, nf, tau, s, lane);
            up.fetch(x, 0, work, lane);
            if constexpr (WQ) {
                const T sd = of_column(s, lane);
#pragma unroll
                for (int rb = 0; rb < RA; ++rb) keep(rb, sd * x.get(rb, 0));
            }
        }
        // last row first, as in panel_step
        if (lane < NC - J0) {
#pragma unroll
            for (int j = 3; j >= 0; --j) {
                if (NC % 4 == 0 || j < NC % 4 || J0 + j < NC) Rl[at[j]] = r[j];
                asm volatile("" ::: "memory");
            }
        }
        Update::put_f(work, lane, nf);
        lds_order();
        if constexpr (WQ) {
            if (!columns) [[likely]]
                up.reflectors(0, lane, s, keep);
            if (lane < 4 && J0 + lane < NC) tau_out[J0 + lane] = of_column(tau, lane);
        }
        static_for<1, S>([&](auto sc) { up.apply_shift(c, decltype(sc)::value); });
        mfma_settle();
        lds_order();
    } while (++P < last);
}

template <typename T, int NC, bool WQ>
__device__ __forceinline__ void merge_panels(Chunk<T, MergeRows<T, NC>::RB, Slots<NC>::NS>& c, T* Rs, T* work,
                                             int n, unsigned close, T* Vn, T* tau_out)
{
    static_for<0, (Slots<NC>::NS + 3) / 4>(
        [&](auto kc) { merge_row_block<T, NC, decltype(kc)::value, WQ>(c, Rs, work, n, close, Vn, tau_out); });
}

// The triangle tri (packed by rows, LDS or global) as the bottom operand of
// merge_panels.
template <typename T, int NC>
__device__ __forceinline__ void triangle_chunk(const T* tri, Chunk<T, MergeRows<T, NC>::RB, Slots<NC>::NS>& c)
{
    constexpr int NS = Slots<NC>::NS;
    const int lane = lane_id();
    const int q = c.q(lane), p = c.p(lane);
#pragma unroll
    for (int rb = 0; rb < MergeRows<T, NC>::RB; ++rb) {
        const int i = 16 * rb + p;
        const int base = Tri<NC>::off(i) - i + q;       // entry (i, 4 s + q) is at base + 4 s
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int b = s + merge_first<T>(rb), k = 4 * b + q;
            const bool in = i <= k && k < NC;
            const T t = (b >= NS || 4 * b + 3 < 16 * rb) ? T(0) : tri[in ? base + 4 * b : 0];
            c.put(rb, s, in && b < NS ? t : T(0));
        }
    }
}

}  // namespace dev
}  // namespace tsqr
