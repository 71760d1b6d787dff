// tsqr_q.h -- the Q factor of TSQR from its stored reflectors.
//
// The leaf+tree kernel in the Q-factor mode keeps every reflector it applies:
// the chunk parts s*x of each leaf's reflectors (V, m x n) with their tau, and
// for every merge of the tree the R2 parts of the operator's reflectors (an
// upper triangle) with their tau (the V and tau outputs of Table 3).  Q is
// then the product of all those reflectors applied to [D; 0], D the signs of
// R's diagonal (R = D R_raw makes Q = Q_raw D), taken in reverse order of
// application:
//   tree pass  (one launch per level, root first): a merge with reflectors
//              H_0..H_{n-1} on the stack [top; bottom] maps the node's n x n
//              block Q_in to H_0 ... H_{n-1} [Q_in; 0]; its top half is the
//              block of the left child, its bottom half that of the right.
//   leaf pass  (one workgroup per leaf, chunks last to first): the chunk's
//              reflectors map the running n x n block T to H_0 ... H_{n-1}
//              [T; 0]; the bottom part is Q's rows of the chunk, the top part
//              the running block for the previous chunk.
// This is the implicit representation of Q that the paper's section 3 notes a
// reduction cannot return, formed explicitly.
//
// All passes apply four reflectors at a time (apply_panel below) on the matrix
// cores, in the register layout of tsqr_panel.h.  With X the panel's four
// columns of V, T its four rows of the top block and C the bottom block, the
// panel needs W = T + X^T C (one matrix product over the rows), the four
// coefficients y_j = tau_j w_j with the w that are left corrected by the inner
// products v_i . v_j (four numbers per column, one column per lane), T -= y, and
// C -= X y (one matrix product).
#pragma once

#include "tsqr_device.h"
#include "tsqr_internal.h"

namespace tsqr {
namespace dev {

constexpr int kTopStride = kWave;      // row J of a top block at J * kTopStride, one column per lane
// (the blocks in the workspace lie by rows as well: qblk NC x NC, tq NC x kQtCols)

// v_i . v_j of the panel's columns: entry (i, j) is read from one lane
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

// The four reflectors of panel P, X in x (its first RA row blocks), applied to
// the stack [T; C]: T in LDS (rows of kTopStride), C the KS slots of c.  Forward:
// H_0 first (Q^T); otherwise H_3 first (Q).  With Zero, C is zero on entry.
// Lane J of taus holds tau_J.  Lanes past 4 KS compute on a spare column of T.
template <typename T, int NC, int RB, int RA, int P, int KS, bool Forward, bool Zero>
__device__ __forceinline__ void apply_panel(const Chunk<T, RB, 1>& x, Chunk<T, RB, KS>& c, T* top, T* work, T taus)
{
    constexpr int J0 = 4 * P;
    constexpr int NJ = NC - J0 < 4 ? NC - J0 : 4;
    using Update = PanelUpdate<T, RA>;
    const int lane = lane_id();
    T t[4], g[4], v[4], y[4] = {T(0), T(0), T(0), T(0)};
    T* tl = top + J0 * kTopStride + lane;
#pragma unroll
    for (int j = 0; j < NJ; ++j) t[j] = tl[j * kTopStride];
    Update::stage(x, 0, work, lane);
    lds_order();
    panel_gram<RA>(x, v);
    if constexpr (!Zero) panel_products<0, 0, KS, RA>(x, c, g);
    T w[4];
#pragma unroll
    for (int j = 0; j < NJ; ++j) w[j] = Zero ? t[j] : t[j] + g[j];
    static_for<0, NJ>([&](auto jc) {
        constexpr int j = Forward ? decltype(jc)::value : NJ - 1 - decltype(jc)::value;
        y[j] = lane_value(taus, J0 + j) * w[j];
#pragma unroll
        for (int i = Forward ? j + 1 : 0; i < (Forward ? NJ : j); ++i)
            w[i] = fmadd(-gram_entry(v, i < j ? i : j, i < j ? j : i), y[j], w[i]);
    });
#pragma unroll
    for (int j = 0; j < NJ; ++j) tl[j * kTopStride] = t[j] - y[j];
#pragma unroll
    for (int j = 0; j < 4; ++j) y[j] = -y[j];
    Update::put_f(work, lane, y);
    lds_order();
    const Update up(x, 0, work, lane);
    static_for<0, KS>([&](auto sc) { up.apply(c, decltype(sc)::value); });
    mfma_settle();
    lds_order();
}

// Column block P of V (a chunk's rows from row base + p on; every row of the
// chunk is stored) into x; columns past n read a block of zeros.
template <typename T, int RPL>
__device__ __forceinline__ void load_reflectors(Chunk<T, RPL, 1>& x, const T* V, int64_t ldv, int64_t base, int P, int n,
                                                int q, int p)
{
    const int k = 4 * P + q;
    const T* ptr = k < n ? V + base + p + (int64_t)k * ldv : zeros_for(V) + p;
#pragma unroll
    for (int r = 0; r < RPL; ++r) x.put(r, 0, ptr[16 * r]);
}

// The merge's reflectors, panel P: rows of the packed triangle in LDS
template <typename T, int NC, int P, int RB>
__device__ __forceinline__ void node_reflectors(Chunk<T, RB, 1>& x, const T* Vl, int q, int p)
{
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int i = 16 * rb + p, k = 4 * P + q;
        const bool in = rb <= P / 4 && i <= k && k < NC;
        const T t = Vl[in ? Tri<NC>::off(i) + k - i : 0];
        x.put(rb, 0, in ? t : T(0));
    }
}

// Level `level` of the tree, root first: workgroup g takes the merge whose
// left operand is leaf g * 2^(level+1).
template <typename T, int NC>
__global__ void __launch_bounds__(kWave) q_tree_kernel(LeafTreeArgs<T> a, int level)
{
    constexpr int NT = Tri<NC>::kSize;
    constexpr int RB = MergeRows<T, NC>::RB, NS = Slots<NC>::NS;
    using C = Chunk<T, RB, NS>;
    __shared__ T Vl[NT];
    __shared__ T top[NC * kTopStride];
    __shared__ __align__(16) T work[PanelLds<T, RB>::kElems];
    const int lane = threadIdx.x;
    const int q = C::q(lane), p = C::p(lane);
    const int span = 1 << level;
    const int left = blockIdx.x * 2 * span;
    const int right = left + span;
    const int id = left + span - 1;
    T* qL = a.qs.qblk + (int64_t)left * NC * NC;
    T* qR = a.qs.qblk + (int64_t)right * NC * NC;
    const T tau = lane < NC ? a.qs.tau_node[(int64_t)id * NC + lane] : T(0);
    for (int i = lane; i < NT; i += kWave) Vl[i] = a.qs.Vn[(int64_t)id * NT + i];
    for (int j = 0; j < NC; ++j) top[j * kTopStride + lane] = lane < NC ? qL[j * NC + lane] : T(0);
    wave_sync();
    C c;
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int s = 0; s < NS; ++s) c.put(r, s, T(0));
    static_for<0, NS>([&](auto pc) {
        constexpr int P = NS - 1 - decltype(pc)::value;
        Chunk<T, RB, 1> x;
        node_reflectors<T, NC, P>(x, Vl, q, p);
        apply_panel<T, NC, RB, P / 4 + 1, P, NS, false, P == NS - 1>(x, c, top, work, tau);
    });
    wave_sync();
    for (int j = 0; j < NC; ++j)
        if (lane < NC) qL[j * NC + lane] = top[j * kTopStride + lane];
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int row = 16 * r + p, k = 4 * s + q;
            if (row < NC && k < NC) qR[row * NC + k] = c.get(r, s);
        }
}

// Q's rows of one leaf: workgroup g takes leaf g.  Bound by the instruction
// rate: per panel 2 x 16 KS RPL-row matrix products and about 150 other
// instructions; the next panel's reflectors are loaded a panel ahead.
template <typename T, int NC, int RPL>
__global__ void __launch_bounds__(kWave) q_leaf_kernel(LeafTreeArgs<T> a, T* Q, int64_t ldq)
{
    constexpr int CH = 16 * RPL;
    constexpr int NS = Slots<NC>::NS;
    using C = Chunk<T, RPL, NS>;
    __shared__ T top[NC * kTopStride];
    __shared__ __align__(16) T work[PanelLds<T, RPL>::kElems];
    const int lane = threadIdx.x;
    const int q = C::q(lane), p = C::p(lane);
    const int leaf = blockIdx.x;
    const int n = a.n;
    const int64_t r0 = (int64_t)leaf * a.leaf_rows;
    const int64_t r1 = (r0 + a.leaf_rows < a.m) ? r0 + a.leaf_rows : a.m;
    const T* qin = a.qs.qblk + (int64_t)leaf * NC * NC;
    for (int j = 0; j < NC; ++j) top[j * kTopStride + lane] = lane < NC ? qin[j * NC + lane] : T(0);
    wave_sync();
    if (r1 <= r0) return;
    const int64_t nchunks = (r1 - r0 + CH - 1) / CH;
    // panels past n hold no reflectors; the last one that does comes first
    const int plast = (n - 1) / 4;
    const int64_t c0 = r0 / CH;                  // the leaf's first chunk among all
    auto taus = [&](int64_t t) { return lane < NC ? a.qs.tau_leaf[(c0 + t) * NC + lane] : T(0); };
    Chunk<T, RPL, 1> x, nx;
    load_reflectors<T, RPL>(nx, a.qs.V, a.qs.ldv, r0 + (nchunks - 1) * CH, plast, n, q, p);
    T ntau = taus(nchunks - 1);
    for (int64_t t = nchunks - 1; t >= 0; --t) {
        const int64_t cbase = r0 + t * CH;
        const int64_t tn = t > 0 ? t - 1 : 0;    // the chunk after this one
        const T tau = ntau;
        ntau = taus(tn);
        C c;
#pragma unroll
        for (int r = 0; r < RPL; ++r)
#pragma unroll
            for (int s = 0; s < NS; ++s) c.put(r, s, T(0));
        static_for<0, NS>([&](auto pc) {
            constexpr int P = NS - 1 - decltype(pc)::value;
            if (P <= plast) {
                x = nx;
                if constexpr (P > 0)
                    load_reflectors<T, RPL>(nx, a.qs.V, a.qs.ldv, cbase, P - 1, n, q, p);
                else
                    load_reflectors<T, RPL>(nx, a.qs.V, a.qs.ldv, r0 + tn * CH, plast, n, q, p);
                apply_panel<T, NC, RPL, RPL, P, NS, false, false>(x, c, top, work, tau);
            }
        });
#pragma unroll
        for (int r = 0; r < RPL; ++r) {
            const int64_t row = cbase + p + 16 * r;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const int k = 4 * s + q;
                if (row < r1 && k < n) Q[row + (int64_t)k * ldq] = c.get(r, s);
            }
        }
    }
}

// ---- applying Q^T without forming Q ---------------------------------------------
//
// C = Q^T B (n x k) replays the factorization's reflectors on B in the order
// the factorization applied them to A:
//   leaf pass  (one workgroup per leaf, chunks first to last): the running
//              n x k block T (zero at the start) stacked on the chunk's rows of
//              B is mapped by the chunk's reflectors H_0, ..., H_{n-1} in turn;
//              what is left in the chunk's rows belongs to rows of Q_full^T B
//              past the first n and is dropped.
//   tree pass  (one launch per level, leaves first): a merge maps the stack
//              [T_left; T_right] by its reflectors and keeps the top block.
//   finish     C = D T_root, D the signs the root applied to R.
// k is taken in panels (52 columns in FP64, 64 in FP32); KS column slots
// (4 columns each) are compiled for the panel width and for panels of at most
// 32, 16 and 4 columns.  The per-leaf blocks are kQtCols = 64
// columns wide.

template <typename T, int NC, int RPL, int KS>
__global__ void __launch_bounds__(kWave) qt_leaf_kernel(QtArgs<T> x)
{
    constexpr int CH = 16 * RPL;
    constexpr int NS = Slots<NC>::NS;
    using C = Chunk<T, RPL, KS>;
    __shared__ T top[NC * kTopStride];
    __shared__ __align__(16) T work[PanelLds<T, RPL>::kElems];
    const LeafTreeArgs<T>& a = x.a;
    const int lane = threadIdx.x;
    const int q = C::q(lane), p = C::p(lane);
    const int leaf = blockIdx.x;
    const int n = a.n;
    const int64_t r0 = (int64_t)leaf * a.leaf_rows;
    const int64_t r1 = (r0 + a.leaf_rows < a.m) ? r0 + a.leaf_rows : a.m;
    for (int j = 0; j < NC; ++j) top[j * kTopStride + lane] = T(0);
    wave_sync();
    const int64_t nchunks = r1 > r0 ? (r1 - r0 + CH - 1) / CH : 0;
    const int plast = (n - 1) / 4;
    const int64_t c0 = r0 / CH;                  // the leaf's first chunk among all
    auto taus = [&](int64_t t) { return lane < NC ? a.qs.tau_leaf[(c0 + t) * NC + lane] : T(0); };
    // a chunk's rows of B; the next chunk's are loaded a chunk ahead where the
    // registers allow it
    auto load_b = [&](C& c, int64_t t) {
#pragma unroll
        for (int r = 0; r < RPL; ++r) {
            const int64_t row = r0 + t * CH + p + 16 * r;
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const int col = 4 * s + q;
                c.put(r, s, (row < r1 && col < x.k) ? x.B[row + (int64_t)col * x.ldb] : T(0));
            }
        }
    };
    constexpr bool kAhead = KS <= 4;
    Chunk<T, RPL, 1> v, nv;
    C c, nb;
    T ntau = T(0);
    if (nchunks > 0) {
        load_reflectors<T, RPL>(nv, a.qs.V, a.qs.ldv, r0, 0, n, q, p);
        ntau = taus(0);
        if constexpr (kAhead) load_b(nb, 0);
    }
    for (int64_t t = 0; t < nchunks; ++t) {
        const int64_t cbase = r0 + t * CH;
        const int64_t tn = t + 1 < nchunks ? t + 1 : t;     // the chunk after this one
        const T tau = ntau;
        ntau = taus(tn);
        if constexpr (kAhead) {
            c = nb;
            load_b(nb, tn);
        } else {
            load_b(c, t);
        }
        static_for<0, NS>([&](auto pc) {
            constexpr int P = decltype(pc)::value;
            if (P <= plast) {
                v = nv;
                const bool last = P == plast;
                load_reflectors<T, RPL>(nv, a.qs.V, a.qs.ldv, last ? r0 + tn * CH : cbase, last ? 0 : P + 1, n, q, p);
                apply_panel<T, NC, RPL, RPL, P, KS, true, false>(v, c, top, work, tau);
            }
        });
    }
    wave_sync();
    T* out = x.tq + (int64_t)leaf * NC * kQtCols;
    for (int j = 0; j < NC; ++j)
        if (lane < 4 * KS) out[j * kQtCols + lane] = top[j * kTopStride + lane];
}

// Level `level` of the tree, leaves first: workgroup g takes the merge whose
// left operand is leaf g * 2^(level+1).
template <typename T, int NC, int KS>
__global__ void __launch_bounds__(kWave) qt_tree_kernel(QtArgs<T> x, int level)
{
    constexpr int NT = Tri<NC>::kSize;
    constexpr int RB = MergeRows<T, NC>::RB, NS = Slots<NC>::NS;
    using C = Chunk<T, RB, KS>;
    const LeafTreeArgs<T>& a = x.a;
    __shared__ T Vl[NT];
    __shared__ T top[NC * kTopStride];
    __shared__ __align__(16) T work[PanelLds<T, RB>::kElems];
    const int lane = threadIdx.x;
    const int q = C::q(lane), p = C::p(lane);
    const int span = 1 << level;
    const int left = blockIdx.x * 2 * span;
    const int right = left + span;
    const int id = left + span - 1;
    T* tl = x.tq + (int64_t)left * NC * kQtCols;
    const T* tr = x.tq + (int64_t)right * NC * kQtCols;
    const T tau = lane < NC ? a.qs.tau_node[(int64_t)id * NC + lane] : T(0);
    for (int i = lane; i < NT; i += kWave) Vl[i] = a.qs.Vn[(int64_t)id * NT + i];
    for (int j = 0; j < NC; ++j) top[j * kTopStride + lane] = lane < 4 * KS ? tl[j * kQtCols + lane] : T(0);
    C c;
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int row = 16 * r + p;
            c.put(r, s, row < NC ? tr[row * kQtCols + 4 * s + q] : T(0));
        }
    wave_sync();
    static_for<0, NS>([&](auto pc) {
        constexpr int P = decltype(pc)::value;
        Chunk<T, RB, 1> v;
        node_reflectors<T, NC, P>(v, Vl, q, p);
        apply_panel<T, NC, RB, P / 4 + 1, P, KS, true, false>(v, c, top, work, tau);
    });
    wave_sync();
    for (int j = 0; j < NC; ++j)
        if (lane < 4 * KS) tl[j * kQtCols + lane] = top[j * kTopStride + lane];
}

// C(i, j) = D(i) T_root(i, j) for the k0-th panel of columns, D from the root's
// sign block (the diagonal of the first leaf's Q block).
template <typename T, int NC>
__global__ void __launch_bounds__(kWave) qt_finish_kernel(QtArgs<T> x)
{
    const int n = x.a.n;
    for (int idx = blockIdx.x * kWave + threadIdx.x; idx < n * x.k; idx += gridDim.x * kWave) {
        const int i = idx % n, j = idx / n;
        x.C[i + (int64_t)j * x.ldc] = x.a.qs.qblk[i + i * NC] * x.tq[i * kQtCols + j];
    }
}

}  // namespace dev
}  // namespace tsqr
