// tsqr_mixed.h -- FP64 correction of an FP32 R factor (mixed precision).
//
// Given A (m x n, stored in FP32) and R~, the R factor of A computed by the
// FP32 TSQR path (section 2 of the paper in FP32), one FP64 pass gives R to
// FP64 accuracy when kappa(A) * u32 << 1:
//     Y = A R~^-1   (FP64; kappa(Y) = 1 + O(kappa(A) u32)),
//     G = Y^T Y,    R_c = chol(G) (upper, G = R_c^T R_c),    R = R_c R~.
// This is the second pass of CholeskyQR2 (Fukaya, Nakatsukasa, Yanagisawa and
// Yamamoto, 2014) with the FP32 Householder factorization as the first pass.
// The Cholesky factorization fails (a pivot that is not positive and finite)
// when R~ is too inaccurate, and R~ is not trusted either when the bound
// ||R_c||_F ||R_c^-1||_F on kappa(A R~^-1) exceeds 1e4; the instance is then
// flagged, and a batched FP64 TSQR launch over the FP32 storage, whose
// workgroups exit at once for unflagged instances, refactors it (decided on
// the device, no host sync).  R~ may also come from the FP32 TSQR of a row
// sample (the sampled plan): the correction is the same.
//
// Two kernels:
//   mixed_gram_kernel   one workgroup of two wavefronts per (row block,
//                       instance), on the FP64 matrix cores: the operand table
//                       of the blocked substitution (below) from R~, then
//                       Y = A R~^-1 and the rows' contribution to G = Y^T Y,
//                       16 rows of each wavefront at a time; the partial G goes
//                       to a workspace slot.
//   mixed_finish_kernel one wavefront per instance: sums the slots in a fixed
//                       order (bit-reproducible), Cholesky with one column per
//                       lane, a bound on kappa(A R~^-1), R = R_c R~,
//                       sign-normalized by construction (both factors have
//                       positive diagonals).
//
// The matrix-core instruction is the 4x4x4 FP64 product with four independent
// blocks, D_b = A_b B_b + C_b (b = 0..3).  Writing lane l as 16 d2 + 4 d1 + d0,
// it takes block d1 of each operand from the lanes with that d1, and
//     A_b(i, k) from lane (d2 = k, d0 = i),  B_b(k, j) from lane (d2 = k, d0 = j),
//     D_b(i, j) to lane (d2 = i, d0 = j)
// (measured on gfx950).  So a result D can be used again as a B operand as it
// stands, and moving it to the contraction position (d2 <-> d0) makes it
// usable as either operand.  The four blocks are four groups of 4 rows of A,
// so one instruction covers 16 rows; every operand below is a 4 x 4 block.
//
// Substitution in transposed form, over the 4-column blocks J of Y = A R~^-1:
//     Z_J^T = A_J^T - sum_{I<J} (R~_IJ)^T Y_I^T,    Y_J^T = (R~_JJ^-1)^T Z_J^T
// (column block J of Y R~ = A, solved with the inverse of the 4 x 4 diagonal
// block: blocked forward substitution, as in a blocked TRSM).  Y_I^T is a D
// result and enters the later updates as their B operand directly; the A
// operands are the constant blocks -(R~_IJ)^T and (R~_JJ^-1)^T.  The updates
// run right-looking (each Y_I^T goes into every later Z_J^T at once), so the
// dependent chain is two instructions per block.  Then every Y_J^T moves its
// rows to the contraction position (a store to LDS at the partner lane's
// index), and
//     G_IJ += (Y_I)^T Y_J      for I <= J,
// one instruction per block pair, accumulated in registers over the row block.
// A wavefront takes whole tiles: it keeps all of G and most of the operands in
// its 512 registers (one wavefront per SIMD at n > 32) and adds the products of
// the tile before between the steps of a tile's substitution, which fills the
// two-instruction chain.  Bound by instruction issue: at n = 50 a tile is 182
// matrix instructions of 16 cycles and about 200 others of 5, of which the
// operand reads from LDS were 91.  256 x 65536 x 50 takes 1.85 ms (the whole
// call with a 4096-row sample 2370 us); with half of G per wavefront, every
// operand read from LDS and two wavefronts per SIMD it was 2.0 ms (2510 us).
// The loads must not be consumed before their tile: with the select of rows
// past the end at the load, each tile waited for the next one's (2840 us).
#pragma once

#include "tsqr_device.h"
#include "tsqr_internal.h"

namespace tsqr {

namespace dev {

// block pairs I <= J in column order
__host__ __device__ constexpr int pair_index(int I, int J) { return J * (J + 1) / 2 + I; }

// block pair p -> (I, J), the inverse of pair_index
__host__ __device__ constexpr int pair_col(int p)
{
    int J = 0;
    while (pair_index(0, J + 1) <= p) ++J;
    return J;
}
__host__ __device__ constexpr int pair_row(int p) { return p - pair_index(0, pair_col(p)); }

// Entry (i, k) of the A operand for block pair p = (I, J), with R~ (FP32,
// column-major, ld n) extended by the identity past column n:
//     I < J:  -R~(4I + k, 4J + i)
//     I = J:  X(k, i),  X = R~_JJ^-1 (4 x 4 upper triangular, by back
//             substitution; a zero pivot gives infinities, and the Cholesky
//             factorization then flags the instance)
__device__ inline double substitution_operand(const float* Rt, int n, int p, int i, int k)
{
    auto rt = [&](int r, int c) -> double {
        if (r > c) return 0.0;
        return (c < n) ? (double)Rt[r + (int64_t)c * n] : (r == c ? 1.0 : 0.0);
    };
    const int J = pair_col(p), I = p - pair_index(0, J);
    if (I < J) return -rt(4 * I + k, 4 * J + i);
    // column i of X = U^-1, U = R~_JJ: X(i, i) = 1/U(i, i) and, upward,
    // X(r, i) = -(sum_{q=r+1..i} U(r, q) X(q, i)) / U(r, r)
    const int c0 = 4 * J;
    double x[4] = {0.0, 0.0, 0.0, 0.0};
    x[i] = 1.0 / rt(c0 + i, c0 + i);
    for (int r = i - 1; r >= 0; --r) {
        double t = 0.0;
        for (int q = r + 1; q <= i; ++q) t += rt(c0 + r, c0 + q) * x[q];
        x[r] = -t / rt(c0 + r, c0 + r);
    }
    return x[k];
}

constexpr int kGramWaves = 2;

// Operands of the substitution that a wavefront of the Gram kernel keeps in
// registers; it reads the others from the LDS table in every tile.  Of its 512
// registers, two go to each entry of G and to each such operand, 6 NB to the
// tiles in flight; with less than about 112 left for the rest, the compiler
// moves operands between the two halves of the register file instead.
template <int NC>
constexpr int kGramHeld = MfmaGram<NC>::NP < 200 - 3 * MfmaGram<NC>::NB - MfmaGram<NC>::NP
                              ? MfmaGram<NC>::NP
                              : 200 - 3 * MfmaGram<NC>::NB - MfmaGram<NC>::NP;

template <int NC>
__global__ void __launch_bounds__(kGramWaves * kWave, MfmaGram<NC>::NP <= 36 ? 2 : 1) mixed_gram_kernel(MixedArgs a)
{
    constexpr int NB = MfmaGram<NC>::NB;
    constexpr int NP = MfmaGram<NC>::NP;
    constexpr int W = MfmaGram<NC>::W;
    constexpr int HELD = kGramHeld<NC>;
    // the operand table, entry (i, k) of pair p at 16 p + 4 i + k
    __shared__ double opl[NP * 16];
    // each wavefront's Y^T blocks, stored at the contraction position (lane
    // (d2, d1, d0) writes where lane (d0, d1, d2) reads)
    __shared__ double ys[kGramWaves][NB][kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int d0 = lane & 3, d1 = (lane >> 2) & 3, d2 = lane >> 4;
    const int b = blockIdx.y;
    const int n = a.n;
    const float* Rt = a.Rt + (int64_t)b * n * n;
    for (int idx = threadIdx.x; idx < NP * 16; idx += kGramWaves * kWave)
        opl[idx] = substitution_operand(Rt, n, idx >> 4, (idx >> 2) & 3, idx & 3);
#pragma unroll
    for (int I = 0; I < NB; ++I) ys[wave][I][lane] = 0.0;
    __syncthreads();
    int lofs = 4 * d0 + d2;
    double op[HELD];
#pragma unroll
    for (int p = 0; p < HELD; ++p) op[p] = opl[p * 16 + lofs];
    auto opnd = [&](auto pc) -> double {
        constexpr int p = decltype(pc)::value;
        if constexpr (p < HELD) return op[p];
        else return opl[p * 16 + lofs];
    };
    double g[NP];
#pragma unroll
    for (int q = 0; q < NP; ++q) g[q] = 0.0;

    const float* A = a.A + (int64_t)b * a.stride_a;
    const int64_t r0 = (int64_t)blockIdx.x * a.rows_per_block;
    const int64_t r1 = (r0 + a.rows_per_block < a.m) ? r0 + a.rows_per_block : a.m;
    // Lane (d2, d1, d0) holds row 4 d1 + d0 of a 16-row tile in column 4J + d2
    // of block J: the D layout of Z_J^T.  Columns past n read column n - 1
    // instead (no select in the loop): they only reach padding columns of Y
    // and padding entries of G, since R~ is the identity there and its
    // off-diagonal blocks are zero in padding rows, and the finish kernel never
    // reads those entries.  Block J is read from the uniform column 4 jc(J),
    // jc(J) = min(J, jl) with jl = (n - 1)/4, at the per-lane offset of
    // (column - 4 jc(J)) in [0, 3]: d2 for J < jl, eb from jl on.  The lanes of
    // rows past the row block read the tile's first row and count it as zero
    // when the tile is used: a select at the load would wait for it there.
    const int trow = 4 * d1 + d0;
    const int tdst = 16 * d0 + 4 * d1 + d2;     // the d2 <-> d0 partner
    const int jl = (n - 1) >> 2;
    const int eb = ((4 * jl + d2 < n) ? 4 * jl + d2 : n - 1) - 4 * jl;
    const int64_t cola = (int64_t)d2 * a.lda, colb = (int64_t)eb * a.lda;
    auto load_tile = [&](float (&dst)[NB], int64_t base) {
        const int64_t row = base + trow < r1 ? trow : 0;
        const int64_t offa = row + cola, offb = row + colb;
#pragma unroll
        for (int J = 0; J < NB; ++J) {
            const int jc = J < jl ? J : jl;
            const float* __restrict__ colp = A + base + (int64_t)(4 * jc) * a.lda;
            dst[J] = colp[J < jl ? offa : offb];
        }
    };
    // Tile t of the wavefront is at r0 + 16 (wave + kGramWaves t).  An
    // iteration substitutes one tile and, between the steps of that dependent
    // chain, adds the products of the tile before (zero in the first one).
    // Tiles are loaded two iterations ahead (two register buffers, the loop
    // unrolled by two; past the last tile, that tile again with all its rows
    // counted as zero, so that no branch stands between a load and its use).
    constexpr int64_t STEP = kGramWaves * 16;
    const int64_t first = r0 + 16 * wave;
    const int64_t last = first + (r1 - first - 1) / STEP * STEP;       // with a tile at all: first < r1
    auto iteration = [&](float (&cur)[NB], int64_t base) {
        if constexpr (HELD < NP) asm volatile("" : "+v"(lofs));     // operands past HELD are read where they are used
        double z[NB], t[NB];
#pragma unroll
        for (int I = 0; I < NB; ++I) t[I] = ys[wave][I][lane];
#pragma unroll
        for (int J = 0; J < NB; ++J) z[J] = (double)(base + trow < r1 ? cur[J] : 0.0f);
        load_tile(cur, base + 2 * STEP < last ? base + 2 * STEP : last);
        __builtin_amdgcn_sched_barrier(0);      // the loads stay at the start of the iteration
        static_for<0, NB>([&](auto ic) {
            constexpr int I = decltype(ic)::value;
            z[I] = mfma4(opnd(std::integral_constant<int, pair_index(I, I)>{}), z[I], 0.0);          // Y_I^T
            static_for<NP * I / NB, NP * (I + 1) / NB>([&](auto qc) {
                constexpr int q = decltype(qc)::value;
                g[q] = mfma4(t[pair_row(q)], t[pair_col(q)], g[q]);
            });
            static_for<I + 1, NB>([&](auto jc) {
                constexpr int J = decltype(jc)::value;
                z[J] = mfma4(opnd(std::integral_constant<int, pair_index(I, J)>{}), z[I], z[J]);     // Z_J^T -= (R~_IJ)^T Y_I^T
            });
        });
#pragma unroll
        for (int I = 0; I < NB; ++I) ys[wave][I][tdst] = z[I];
        wave_sync();
        __builtin_amdgcn_sched_barrier(0);
    };
    float nx0[NB], nx1[NB];
    if (first < r1) {
        load_tile(nx0, first);
        load_tile(nx1, first + STEP < last ? first + STEP : last);
    }
    for (int64_t base = first; base < r1; base += 2 * STEP) {
        iteration(nx0, base);
        iteration(nx1, base + STEP);
    }
    double t[NB];
#pragma unroll
    for (int I = 0; I < NB; ++I) t[I] = ys[wave][I][lane];
    static_for<0, NP>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        g[q] = mfma4(t[pair_row(q)], t[pair_col(q)], g[q]);
    });
    // the four row groups (instruction blocks, d1) hold partial sums of every
    // block of G: add them within each 16-lane row, then over the wavefronts
    // (through the operand table's LDS), and the lanes of the first wavefront
    // with d1 = 0 write block (I, J) of the upper block triangle, entry (d2, d0)
    __syncthreads();
    static_for<0, NP>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        double v = g[q];
        v = v + dpp_mov<0x124>(v);    // row_ror:4
        v = v + dpp_mov<0x128>(v);    // row_ror:8
        g[q] = v;
        if (wave == 1 && d1 == 0) opl[q * 16 + 4 * d2 + d0] = v;
    });
    __syncthreads();
    if (wave != 0 || d1 != 0) return;
    double* out = a.part + ((int64_t)b * a.blocks + blockIdx.x) * (W * W);
    static_for<0, NP>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        out[(4 * pair_row(q) + d2) * W + 4 * pair_col(q) + d0] = g[q] + opl[q * 16 + 4 * d2 + d0];
    });
}
static_assert(kGramWaves == 2, "the sum over wavefronts is written for two");

// bound on ||Rc||_F ||Rc^-1||_F (>= kappa_2(A R~^-1)) for a trusted correction;
// an FP32 R~ of a matrix with kappa(A) <= 1e8 gives about n (1 + kappa(A) 2^-24)
constexpr double kMaxKappaY = 1e4;

template <int NC>
__global__ void __launch_bounds__(kWave) mixed_finish_kernel(MixedArgs a)
{
    constexpr int W = MfmaGram<NC>::W;
    __shared__ double Rc[NC * NC];       // column-major, ld NC
    __shared__ double Rtl[NC * NC];      // R~ column-major, zero below the diagonal
    const int lane = threadIdx.x;
    const int b = blockIdx.x;
    const int n = a.n;
    const float* Rt = a.Rt + (int64_t)b * n * n;
    for (int idx = lane; idx < NC * NC; idx += kWave) {
        const int i = idx % NC, j = idx / NC;
        Rtl[idx] = (i <= j && j < n) ? (double)Rt[i + j * n] : 0.0;
    }
    // column `lane` of G (rows 0..lane), the partial sums added in block order;
    // a slot's NC loads are issued together (entries below the diagonal
    // block triangle are never written and are discarded below)
    double c[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) c[i] = 0.0;
    const double* part = a.part + (int64_t)b * a.blocks * (W * W) + (lane < n ? lane : 0);
    for (int w = 0; w < a.blocks; ++w) {
#pragma unroll
        for (int i = 0; i < NC; ++i) c[i] += part[(int64_t)w * (W * W) + i * W];
    }
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        // padding columns: identity, so the factor stays nonsingular
        const bool in = i <= lane && lane < n;
        c[i] = in ? c[i] : ((i == lane && lane >= n) ? 1.0 : 0.0);
    }
    // Cholesky G = Rc^T Rc, column `lane` of Rc in c (rows 0..lane)
    bool good = true;
    static_for<0, NC>([&](auto kc) {
        constexpr int K = decltype(kc)::value;
        double d = 0.0;
#pragma unroll
        for (int i = 0; i < K; ++i) d = fmadd(bpermute(K << 2, c[i]), c[i], d);
        const double t = c[K] - d;
        const double piv = lane_value(t, K);
        good = good && (piv > 0.0) && (piv < __builtin_inf());
        const double r = __builtin_sqrt(piv);
        c[K] = (lane > K) ? t / r : ((lane == K) ? r : 0.0);
    });
#pragma unroll
    for (int i = 0; i < NC; ++i)
        if (lane < NC) Rc[i + lane * NC] = c[i];
    wave_sync();
    // Y = A R~^-1 = Q Rc, so kappa_2(Y) = kappa_2(Rc) <= ||Rc||_F ||Rc^-1||_F.
    // Past kMaxKappaY the correction is not trusted (its Gram matrix carries
    // a relative error of order kappa(Y)^2 u in its smallest directions) and
    // the instance takes the FP64 path as well.  Column `lane` of X = Rc^-1 by
    // back substitution against the rows of Rc in LDS; padding columns are
    // left out of both norms.
    {
        double sr = 0.0, sx = 0.0;
#pragma unroll
        for (int i = 0; i < NC; ++i) sr = fmadd(c[i], c[i], sr);
        double x[NC];
#pragma unroll
        for (int i = NC - 1; i >= 0; --i) {
            double t = (i == lane) ? 1.0 : 0.0;
#pragma unroll
            for (int k = i + 1; k < NC; ++k) t = fmadd(-Rc[i + k * NC], x[k], t);
            x[i] = (i <= lane) ? t / Rc[i + i * NC] : 0.0;
            sx = fmadd(x[i], x[i], sx);
        }
        if (lane >= n) sx = sr = 0.0;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            sx += __shfl_xor(sx, off);
            sr += __shfl_xor(sr, off);
        }
        good = good && (sr * sx <= kMaxKappaY * kMaxKappaY);
    }
    // R = Rc R~, column `lane`: R(i, lane) = sum_{k >= i} Rc(i, k) R~(k, lane)
    double* R = a.R + (int64_t)b * a.ldr * n;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        double s = 0.0;
#pragma unroll
        for (int k = i; k < NC; ++k) s = fmadd(Rc[i + k * NC], Rtl[k + (lane < NC ? lane : 0) * NC], s);
        if (i < n && lane < n) R[i + (int64_t)lane * a.ldr] = (i <= lane) ? s : 0.0;
    }
    if (lane == 0) {
        a.flags[b] = good ? 0 : 1;
        if (a.flags_out) a.flags_out[b] = good ? 0 : 1;
    }
}

}  // namespace dev
}  // namespace tsqr
