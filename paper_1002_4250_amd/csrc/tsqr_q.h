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

// Rows of kCols columns (leading dimension ld, lanes past them zero) from global
// memory to a top block: all loads first, so they are in flight together
template <typename T, int NC, int kCols, int kLd>
__device__ __forceinline__ void load_top(const T* __restrict__ src, T* top)
{
    const int lane = lane_id();
    T t[NC];
#pragma unroll
    for (int j = 0; j < NC; ++j) t[j] = src[j * kLd + (lane < kCols ? lane : 0)];
#pragma unroll
    for (int j = 0; j < NC; ++j) top[j * kTopStride + lane] = lane < kCols ? t[j] : T(0);
}
template <typename T, int NC, int kCols, int kLd>
__device__ __forceinline__ void store_top(const T* top, T* __restrict__ dst)
{
    const int lane = lane_id();
#pragma unroll
    for (int j = 0; j < NC; ++j) {
        const T t = top[j * kTopStride + lane];
        if (lane < kCols) dst[j * kLd + lane] = t;
    }
}

// the rows of the last panel past NC
template <typename T, int NC>
__device__ __forceinline__ void zero_spare_rows(T* top)
{
    for (int j = NC; j < 4 * Slots<NC>::NS; ++j) top[j * kTopStride + lane_id()] = T(0);
}

// The four reflectors from column J0 on, X in x (its first RA row blocks), applied to
// the stack [T; C]: T in LDS (rows of kTopStride), C the KS slots of c.  Forward:
// H_0 first (Q^T); otherwise H_3 first (Q).  Lane J of taus holds tau_J (zero past
// the last reflector).  Lanes past 4 KS compute on a spare column of T.  One loop
// body serves every panel: the passes over the tree run it a dozen times per
// launch, and unrolled their time was mostly the fetch of instructions (34 us per
// level at n = 50, FP64).
template <typename T, int RB, int RA, int KS, bool Forward>
__device__ __forceinline__ void apply_panel(int J0, const Chunk<T, RB, 1>& x, Chunk<T, RB, KS>& c, T* top, T* work,
                                            T taus)
{
    constexpr int NJ = 4;
    using Update = PanelUpdate<T, RA>;
    const int lane = lane_id();
    T t[4], g[4], v[4], y[4] = {T(0), T(0), T(0), T(0)};
    T* tl = top + J0 * kTopStride + lane;
#pragma unroll
    for (int j = 0; j < NJ; ++j) t[j] = tl[j * kTopStride];
    Update::stage(x, 0, work, lane);
    lds_order();
    panel_gram<RA>(x, v);
    panel_products<0, 0, KS, RA>(x, c, g);
    T w[4];
#pragma unroll
    for (int j = 0; j < NJ; ++j) w[j] = t[j] + g[j];
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
    Update up;
    up.fetch(x, 0, work, lane);
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
template <typename T, int NC, int RB>
__device__ __forceinline__ void node_reflectors(Chunk<T, RB, 1>& x, const T* Vl, int P, int q, int p)
{
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int i = 16 * rb + p, k = 4 * P + q;
        const bool in = i <= k && k < NC;
        const T t = Vl[in ? Tri<NC>::off(i) + k - i : 0];
        x.put(rb, 0, in ? t : T(0));
    }
}

// All reflectors of a merge of n columns applied to [T; C].  The panels of the first
// two row blocks leave the other rows alone.
template <typename T, int NC, int KS, bool Forward>
__device__ __forceinline__ void apply_node(Chunk<T, MergeRows<T, NC>::RB, KS>& c, const T* Vl, T* top, T* work, T tau,
                                           int n, int q, int p)
{
    constexpr int RB = MergeRows<T, NC>::RB, NS = Slots<NC>::NS;
    constexpr int RL = RB < 2 ? RB : 2, PL = NS < 8 ? NS : 8;
    const int np = panels_of(n);
    // (at least one panel: registers that a loop may leave as they are get copied)
    auto part = [&](auto rows, int first, int last) {
        int i = first;
#pragma nounroll
        do {
            const int P = Forward ? i : first + last - 1 - i;
            Chunk<T, RB, 1> x;
            node_reflectors<T, NC>(x, Vl, P, q, p);
            apply_panel<T, RB, decltype(rows)::value, KS, Forward>(4 * P, x, c, top, work, tau);
        } while (++i < last);
    };
    const bool more = NS > PL && (4 * PL < kMinColumns<NC> || np > PL);
    if constexpr (!Forward && NS > PL)
        if (more) part(std::integral_constant<int, RB>{}, PL, np);
    part(std::integral_constant<int, RL>{}, 0, np < PL ? np : PL);
    if constexpr (Forward && NS > PL)
        if (more) part(std::integral_constant<int, RB>{}, PL, np);
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
    __shared__ T top[4 * Slots<NC>::NS * kTopStride];
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
    triangle_to_lds<T, NC>(a.qs.Vn + (int64_t)id * NT, Vl);
    load_top<T, NC, NC, NC>(qL, top);
    zero_spare_rows<T, NC>(top);
    wave_sync();
    C c;
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int s = 0; s < NS; ++s) c.put(r, s, T(0));
    apply_node<T, NC, NS, false>(c, Vl, top, work, tau, a.n, q, p);
    wave_sync();
    store_top<T, NC, NC, NC>(top, qL);
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
    __shared__ T top[4 * Slots<NC>::NS * kTopStride];
    __shared__ __align__(16) T work[PanelLds<T, RPL>::kElems];
    const int lane = threadIdx.x;
    const int q = C::q(lane), p = C::p(lane);
    const int leaf = blockIdx.x;
    const int n = a.n;
    const int64_t r0 = (int64_t)leaf * a.leaf_rows;
    const int64_t r1 = (r0 + a.leaf_rows < a.m) ? r0 + a.leaf_rows : a.m;
    const T* qin = a.qs.qblk + (int64_t)leaf * NC * NC;
    load_top<T, NC, NC, NC>(qin, top);
    zero_spare_rows<T, NC>(top);
    wave_sync();
    if (r1 <= r0) return;
    const int64_t nchunks = (r1 - r0 + CH - 1) / CH;
    // panels past n hold no reflectors; the last one that does comes first
    const int plast = panels_of(n) - 1;
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
#pragma nounroll
        for (int P = plast; P >= 0; --P) {
            x = nx;
            const bool last = P == 0;
            load_reflectors<T, RPL>(nx, a.qs.V, a.qs.ldv, last ? r0 + tn * CH : cbase, last ? plast : P - 1, n, q, p);
            apply_panel<T, RPL, RPL, NS, false>(4 * P, x, c, top, work, tau);
        }
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
    __shared__ T top[4 * Slots<NC>::NS * kTopStride];
    __shared__ __align__(16) T work[PanelLds<T, RPL>::kElems];
    const LeafTreeArgs<T>& a = x.a;
    const int lane = threadIdx.x;
    const int q = C::q(lane), p = C::p(lane);
    const int leaf = blockIdx.x;
    const int n = a.n;
    const int64_t r0 = (int64_t)leaf * a.leaf_rows;
    const int64_t r1 = (r0 + a.leaf_rows < a.m) ? r0 + a.leaf_rows : a.m;
    for (int j = 0; j < NC; ++j) top[j * kTopStride + lane] = T(0);
    zero_spare_rows<T, NC>(top);
    wave_sync();
    const int64_t nchunks = r1 > r0 ? (r1 - r0 + CH - 1) / CH : 0;
    const int plast = panels_of(n) - 1;
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
#pragma nounroll
        for (int P = 0; P <= plast; ++P) {
            v = nv;
            const bool last = P == plast;
            load_reflectors<T, RPL>(nv, a.qs.V, a.qs.ldv, last ? r0 + tn * CH : cbase, last ? 0 : P + 1, n, q, p);
            apply_panel<T, RPL, RPL, KS, true>(4 * P, v, c, top, work, tau);
        }
    }
    wave_sync();
    T* out = x.tq + (int64_t)leaf * NC * kQtCols;
    store_top<T, NC, 4 * KS, kQtCols>(top, out);
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
    __shared__ T top[4 * Slots<NC>::NS * kTopStride];
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
    triangle_to_lds<T, NC>(a.qs.Vn + (int64_t)id * NT, Vl);
    load_top<T, NC, 4 * KS, kQtCols>(tl, top);
    zero_spare_rows<T, NC>(top);
    C c;
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int row = 16 * r + p;
            c.put(r, s, row < NC ? tr[row * kQtCols + 4 * s + q] : T(0));
        }
    wave_sync();
    apply_node<T, NC, KS, true>(c, Vl, top, work, tau, a.n, q, p);
    wave_sync();
    store_top<T, NC, 4 * KS, kQtCols>(top, tl);
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
