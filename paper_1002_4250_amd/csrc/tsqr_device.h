// tsqr_device.h -- gfx950 device code for the R factor of a tall-skinny matrix
// by Householder TSQR (Langou, arXiv:1002.4250, sections 2-3).
//
// Execution model (wavefronts of 64 lanes, four to a workgroup where there is
// more than one leaf):
//   * A leaf is a contiguous block of rows of A.  Its wavefront keeps the n-by-n
//     triangle R in LDS (packed by rows) and streams the block through
//     registers in chunks of 16*RPL rows.  Each chunk C is merged into R by
//     R := R-factor of [R; C] (the structured update of Table 3 with R2
//     replaced by a dense chunk: a flat tree inside the leaf; section 2 allows
//     any tree), four columns at a time on the matrix cores (tsqr_panel.h, with
//     the register layout and the arithmetic).
//   * Leaves then combine with the paper's operator qr(R1, R2) over a binary
//     tree pairing leaf i with i + 2^level (lower index on top): within a
//     workgroup through LDS, above that by whichever wavefront of the pair
//     arrives last (atomic ticket), so no wavefront ever waits on another.  A
//     merge is the same panel step on the lower triangle's rows (merge_panels).
//     Workgroups are numbered onto leaves so that tree siblings share an XCD
//     and its L2 (xcd_local_leaf).
//   * The root flips rows with a negative diagonal (section 2's positive
//     diagonal convention) and writes R.
//   * The operator's own entry point (Table 3) takes one column of R2 per lane
//     and one reflector at a time (merge_columns).
//
// What bounds it: instruction issue of one wavefront per SIMD.  A matrix
// instruction of one wavefront and a vector instruction of another do not
// overlap on a SIMD, so a panel costs its matrix instructions (16 cycles in
// FP64, 8 in FP32) plus about 5 cycles for each of some 300 others, most of
// them the four dependent reflectors.  A chunk of 128 rows at n = 50 in FP64
// takes 21 us on its own (about 3900 cycles a panel), a merge of two triangles
// 16 us.  One column at a time on the vector units the chunk took 37 us, and
// 2^22 x 50 1437 us per call in FP64 and 767 us in FP32; now 882 and 607 us.
#pragma once

#include <hip/hip_runtime.h>

#include <stdint.h>

#include <type_traits>
#include <utility>

#include "tsqr_internal.h"

namespace tsqr {
namespace dev {

constexpr int kWave = 64;

template <int NC>
struct Tri {
    static constexpr int kSize = NC * (NC + 1) / 2;
    // LDS copies get one wavefront of padding: a spare cell for branch-free
    // writes and room for column reads of lanes past the triangle
    static constexpr int kPadded = kSize + 64;
    // packed row-major upper triangle: row j starts at off(j), entry (j,k) at off(j)+k-j
    static constexpr __host__ __device__ int off(int j) { return j * NC - (j * (j - 1)) / 2; }
};

template <int NC>
struct Slots {
    static constexpr int NS = (NC + 3) / 4;     // column slots per lane
};

// The smallest column count that runs at a width: panels that begin before it always
// hold a column.  (33 to 40 columns run at 50 with a number of rows per lane that
// the width 40 is not compiled for.)
template <int NC>
constexpr int kMinColumns = NC <= 8 ? 1 : NC <= 16 ? 9 : NC <= 24 ? 17 : NC <= 32 ? 25 : NC <= 50 ? 33 : 51;
// The panels of n columns
__device__ __forceinline__ int panels_of(int n) { return (n + 3) / 4; }

template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(static_cast<F&&>(f));
    }
}

template <typename T> struct Limits;
template <> struct Limits<double> {
    static constexpr double tiny = 2.2250738585072014e-308;     // the smallest normal number
    static constexpr int tiny_high = 0x00100000;                // its high_word
};
template <> struct Limits<float> {
    static constexpr float tiny = 1.17549435e-38f;
    static constexpr int tiny_high = 0x00800000;
};

// ---- cross-lane primitives -------------------------------------------------

// Row rotations read a valid lane in every row, so no "old" value is needed.
template <int CTRL>
__device__ __forceinline__ double dpp_mov(double x)
{
    int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xF, 0xF, true);
    int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float x)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xF, 0xF, true));
}

// Fused multiply-add and absolute value in the element type (the generic
// builtins would take float operands through double).
__device__ __forceinline__ double fmadd(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fmadd(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double absv(double x) { return __builtin_fabs(x); }
__device__ __forceinline__ float absv(float x) { return __builtin_fabsf(x); }
// The hardware's maximum as it stands (a NaN gives the other operand); the
// builtin quiets its operands first, one more instruction each.  The operands are
// vector registers: a scalar register that a lane read has just written must not
// be read for two wait states, and the compiler sees to that outside inline
// assembly only.
__device__ __forceinline__ double max_raw(double a, double b)
{
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float max_raw(float a, float b)
{
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
// The word that holds sign, exponent and the leading bits: as an integer, its
// order is that of non-negative numbers, with every negative one below them
__device__ __forceinline__ int high_word(double x) { return __double2hiint(x); }
__device__ __forceinline__ int high_word(float x) { return __float_as_int(x); }
// The sign bit of x in place, and a non-negative x with that sign
__device__ __forceinline__ unsigned sign_of(double x) { return (unsigned)__double2hiint(x) & 0x80000000u; }
__device__ __forceinline__ unsigned sign_of(float x) { return (unsigned)__float_as_int(x) & 0x80000000u; }
__device__ __forceinline__ double with_sign(double x, unsigned s)
{
    return __hiloint2double((int)((unsigned)__double2hiint(x) ^ s), __double2loint(x));
}
__device__ __forceinline__ float with_sign(float x, unsigned s)
{
    return __int_as_float((int)((unsigned)__float_as_int(x) ^ s));
}

// Value of x held by the lane whose byte address (4 * lane) is src.
__device__ __forceinline__ double bpermute(int src, double x)
{
    int lo = __builtin_amdgcn_ds_bpermute(src, __double2loint(x));
    int hi = __builtin_amdgcn_ds_bpermute(src, __double2hiint(x));
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ float bpermute(int src, float x)
{
    return __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(x)));
}

// Value of x in lane `l` (l uniform), for every lane.
__device__ __forceinline__ double lane_value(double x, int l)
{
    const int lo = __builtin_amdgcn_readlane(__double2loint(x), l);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(x), l);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ float lane_value(float x, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
}

// This thread's lane in its wavefront (workgroups may hold several)
__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & (kWave - 1)); }

// Orders this wavefront's LDS accesses around a point without constraining
// arithmetic: LDS operations of one wavefront execute in order, so only the
// compiler has to be kept from moving them across.
__device__ __forceinline__ void lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Makes what this wavefront's lanes wrote to LDS visible to its other lanes.
// A wavefront's LDS operations execute in order, so this needs no barrier
// instruction, and the wavefronts of a workgroup need not reach it together.
__device__ __forceinline__ void wave_sync() { lds_order(); }

// ---- reflector scalars ---------------------------------------------------------

// With S = alpha^2 + sigma^2, nrm = sqrt(S) and sgn = sign(alpha) read from its
// sign bit:
//     beta = -sgn nrm,  tau = (beta - alpha)/beta = (|alpha| + nrm)/nrm,
//     s = 1/(alpha - beta) = sgn/(|alpha| + nrm),  tau*s = sgn/nrm.
// 1/nrm comes from the hardware reciprocal square root refined by two Newton
// steps, nrm = S/sqrt(S) with one Newton correction, 1/(|alpha| + nrm) from the
// hardware reciprocal with two Newton steps: a short dependent chain instead
// of two IEEE divisions and a square root.  (The FP64 hardware estimates are
// good to about 2^-24 on gfx950; one quadratic step leaves errors of tens of
// ulps, two reach the rounding level.)  A column whose sigma^2 is below
// the smallest normal number gives the identity reflector.
template <typename T>
struct Reflector {
    T beta, tau, s, ts;
};

__device__ __forceinline__ double hw_rsq(double x) { return __builtin_amdgcn_rsq(x); }
__device__ __forceinline__ float hw_rsq(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ double hw_rcp(double x) { return __builtin_amdgcn_rcp(x); }
__device__ __forceinline__ float hw_rcp(float x) { return __builtin_amdgcn_rcpf(x); }

template <typename T>
__device__ __forceinline__ Reflector<T> make_reflector(T alpha, T sigma2)
{
    const T S = fmadd(alpha, alpha, sigma2);
    T y = hw_rsq(S);
    const T hS = T(0.5) * S;
#pragma unroll
    for (int it = 0; it < 2; ++it) y = fmadd(y, fmadd(-hS * y, y, T(0.5)), y);
    T nrm = S * y;
    nrm = fmadd(T(0.5) * y, fmadd(-nrm, nrm, S), nrm);
    const T d = absv(alpha) + nrm;
    T q = hw_rcp(d);
#pragma unroll
    for (int it = 0; it < 2; ++it) q = fmadd(q, fmadd(-d, q, T(1)), q);
    const bool neg = __builtin_signbit(alpha);
    const bool ok = sigma2 >= Limits<T>::tiny;
    Reflector<T> r;
    r.beta = ok ? (neg ? nrm : -nrm) : alpha;
    r.tau = ok ? d * y : T(0);
    r.s = ok ? (neg ? -q : q) : T(0);
    r.ts = ok ? (neg ? -y : y) : T(0);
    return r;
}

// ---- one Householder step of a leaf -------------------------------------------

// Where a leaf prefetches its next chunk from.  A register slot holds four
// columns; once they are finished (after panel s) the whole slot is refilled
// with the next chunk's columns 4s..4s+3 by one wavefront-wide load per
// register, into registers no later panel of the current chunk reads, so no
// panel waits for the loads.  `col` is a per-lane running pointer to (row base
// + p, column 4s + q) of the next slot; lda and n pass through an opaque
// register copy so the compiler keeps that one pointer instead of precomputing
// one address per slot.
//
// Only a chunk whose rows all lie inside the leaf is prefetched, and the loads
// are branch-free (a lane whose column lies past n reads from a block of zeros
// instead), so that the number of loads in flight is known at compile time: with
// a branch around them the compiler waits for all of them at the top of the
// chunk loop, the last panel's included, a full memory latency per chunk.
static __device__ double kZerosF64[256];
static __device__ float kZerosF32[256];
__device__ __forceinline__ const double* zeros_for(const double*) { return kZerosF64; }
__device__ __forceinline__ const float* zeros_for(const float*) { return kZerosF32; }

template <typename T, int RPL, typename TIn = T>
struct Prefetch {
    const TIn* col;      // per lane: &A(base + p, 4s + q) for the next slot s to fill
    const TIn* zero;     // per lane: zero block + p
    int64_t lda4;        // uniform: 4 * lda
    int cols_left;       // per lane: n - (4s + q)
};

template <typename T, int RPL, typename TIn = T>
__device__ __forceinline__ Prefetch<T, RPL, TIn> make_prefetch(const TIn* A, int64_t lda, int n, int64_t base, int q,
                                                               int p)
{
    static_assert(16 * RPL <= 256, "zero block too small");
    Prefetch<T, RPL, TIn> pf;
    int ldlo = __builtin_amdgcn_readfirstlane((int)lda), ldhi = __builtin_amdgcn_readfirstlane((int)(lda >> 32));
    int nn = __builtin_amdgcn_readfirstlane(n);
    asm volatile("" : "+s"(ldlo), "+s"(ldhi), "+s"(nn));
    const int64_t ld = (int64_t)(((uint64_t)(uint32_t)ldhi << 32) | (uint32_t)ldlo);
    pf.col = A + base + p + (int64_t)q * ld;
    pf.zero = zeros_for(A) + p;
    pf.lda4 = 4 * ld;
    pf.cols_left = nn - q;
    return pf;
}

// Fill register slot `slot` with the next chunk's columns and advance.
template <typename T, int RPL, typename TIn, typename C>
__device__ __forceinline__ void prefetch_slot(C& c, int slot, Prefetch<T, RPL, TIn>& pf)
{
    const TIn* ptr = pf.cols_left > 0 ? pf.col : pf.zero;
#pragma unroll
    for (int r = 0; r < RPL; ++r) c.put(r, slot, (T)ptr[16 * r]);
    pf.col += pf.lda4;
    pf.cols_left -= 4;
}

// Where a leaf in the Q-factor mode writes the reflectors of its current
// chunk: column J of V gets the chunk part s*x of reflector J, tau[J] its tau.
// V has a row for every row of every chunk, so the rows of a partial last
// chunk past the end of A (whose entries are zero) are stored like the others.
template <typename T>
struct VSink {
    T* V;
    int64_t ldv;
    T* tau;
    int64_t cbase;    // first row of the chunk
};

// ---- the operator with one column per lane -------------------------------------
//
// R := qr([R1; R2]) for two NC x NC upper triangles, the operator of section 2
// in the structured form of Table 3 (only rows 0..J of R2 take part in step J).
// R1 is packed by rows in LDS (Rs, padded past the triangle); lane k holds
// column k of R2 in registers (v[i] = R2(i, k), zero below the diagonal).  In
// step J every lane fetches the pivot column R2(0:J, J) from lane J's
// registers (ds_bpermute) and forms its own dot product with it locally
// (lane J's is sigma^2, which all lanes then read from its register), so a
// step has no cross-lane reduction, and lane k > J updates R1(J, k) and its
// column.  One wavefront, bound by its chain of NC dependent steps.  With Keep it
// leaves the Householder vectors in v (lane J's column becomes s x, or stays x for
// an identity reflector) and the tau in tau_out.
template <typename T, int NC, bool Keep>
__device__ __forceinline__ void merge_columns(T (&v)[NC], T* Rs, T* tau_out, int n = NC)
{
    static_for<0, NC>([&](auto jc) {
        constexpr int J = decltype(jc)::value;
        if (J >= kMinColumns<NC> && J >= n) return;
        constexpr int OFF = Tri<NC>::off(J);
        // (an opaque copy, so that the compiler does not compute the masks of
        // all steps ahead and keep them)
        int lane = lane_id();
        asm volatile("" : "+v"(lane));
        const bool own = (lane > J) && (lane < NC);
        const int ridx = own ? OFF + lane - J : Tri<NC>::kSize;
        const T alpha = Rs[OFF];
        const T rjk = Rs[ridx];
        // every lane writes one cell of row J of R1: R1(J, k) for k > J, beta
        // for k = J (no branch), a spare cell otherwise
        const int ridx2 = own ? ridx : ((lane == J) ? OFF : Tri<NC>::kSize);
        // the pivot column, from lane J's registers to every lane
        T x[J + 1];
#pragma unroll
        for (int i = 0; i <= J; ++i) x[i] = bpermute(J << 2, v[i]);
        // this lane's dot product with the pivot column; for lane J it is
        // sigma^2 itself
        // (four partial sums keep the dependent chain short)
        T dd[4] = {x[0] * v[0], T(0), T(0), T(0)};
#pragma unroll
        for (int i = 1; i <= J; ++i) dd[i & 3] = fmadd(x[i], v[i], dd[i & 3]);
        const T d = (dd[0] + dd[1]) + (dd[2] + dd[3]);
        const Reflector<T> h = make_reflector(alpha, lane_value(d, J));
        const T w = fmadd(h.s, d, rjk);
        Rs[ridx2] = own ? fmadd(-h.tau, w, rjk) : ((lane == J) ? h.beta : rjk);
        const T f = own ? h.ts * w : T(0);
#pragma unroll
        for (int i = 0; i <= J; ++i) v[i] = fmadd(-f, x[i], v[i]);
        if constexpr (Keep) {
            const bool mine = (lane == J) && (h.tau != T(0));
#pragma unroll
            for (int i = 0; i <= J; ++i) v[i] = mine ? h.s * x[i] : v[i];
            if (lane == 0) tau_out[J] = h.tau;
        }
        lds_order();
    });
}

// Column `lane` of a packed NC x NC upper triangle (LDS or global) into
// registers, zero below the diagonal and past column NC.
template <typename T, int NC>
__device__ __forceinline__ void triangle_column(const T* tri, T (&v)[NC])
{
    int k = lane_id();
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        const int at = k + (Tri<NC>::off(i) - i);
        v[i] = tri[at < Tri<NC>::kSize ? at : Tri<NC>::kSize - 1];
    }
    asm volatile("" : "+v"(k));
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        v[i] = (i <= k && k < NC) ? v[i] : T(0);
    }
}

// Copy a packed triangle from global memory to LDS: all loads first, then
// all stores, so the loads are in flight together.
template <typename T, int NC>
__device__ __forceinline__ void triangle_to_lds(const T* __restrict__ src, T* dst)
{
    constexpr int NT = Tri<NC>::kSize;
    constexpr int U = (NT + kWave - 1) / kWave;
    const int lane = lane_id();
    T t[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int i = lane + u * kWave;
        t[u] = src[i < NT ? i : 0];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int i = lane + u * kWave;
        if (i < NT) dst[i] = t[u];
    }
}

}  // namespace dev
}  // namespace tsqr

#include "tsqr_panel.h"

namespace tsqr {
namespace dev {

// Widths up to which a merge with close columns takes one column per lane
constexpr int kColumnMerge = 16;

// ---- a merge of the tree ----------------------------------------------------------

// The columns (a bit for each) of the triangle Rs (LDS) that lie mostly in the
// span of those before them in their panel.  Two triangles of rows that are alike
// have about this growth in their merge: sum_i R(i, k)^2 over 2 R(k, k)^2.
template <typename T, int NC>
__device__ __forceinline__ uint64_t close_columns(const T* Rs)
{
    const int lane = lane_id();
    const int k = lane < NC ? lane : NC - 1;
    const T* d = Rs + Tri<NC>::off(k);               // R(k - i, k) is i (NC - k) + i (i - 1) / 2 before R(k, k)
    T sum = T(0);
#pragma unroll
    for (int i = 1; i < 4; ++i) {
        const bool in = i <= (k & 3);
        const T t = d[in ? -(i * (NC - k) + i * (i - 1) / 2) : 0];
        sum = in ? fmadd(t, t, sum) : sum;
    }
    return __builtin_amdgcn_ballot_w64(!(sum <= T(2 * kMaxGrowth) * (d[0] * d[0])));
}

// Whether R2 holds a NaN or an infinity
template <typename T, int RB, int NS>
__device__ __forceinline__ bool not_finite(const Chunk<T, RB, NS>& c)
{
    T t = T(0);
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int s = 0; s < NS; ++s) t = fmadd(c.get(r, s), T(0), t);
    return __builtin_amdgcn_ballot_w64(!(t == T(0))) != 0;
}

// Such an R2 for the panels.  Rows of the result above the first column k0 with a
// non-finite entry do not depend on R2's rows from k0 on, but a panel's products
// run over whole row blocks, and the zeros that it has there would not hide
// a NaN.  Column k0 as a NaN says the same without those rows.
template <typename T, int NC>
__device__ __forceinline__ void isolate_not_finite(Chunk<T, MergeRows<T, NC>::RB, Slots<NC>::NS>& c)
{
    constexpr int RB = MergeRows<T, NC>::RB, NS = Slots<NC>::NS;
    const int lane = lane_id();
    const int q = c.q(lane), p = c.p(lane);
    int k0 = NC;
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const uint64_t m = __builtin_amdgcn_ballot_w64(!(c.get(r, s) * T(0) == T(0)));
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int k = 4 * (s + merge_first<T>(r)) + j;
                if ((m & ((uint64_t)0x1111111111111111 << j)) != 0 && k < k0) k0 = k;
            }
        }
    if (k0 == 0) return;
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const T t = 4 * (s + merge_first<T>(r)) + q == k0 ? T(__builtin_nan("")) : (T)c.get(r, s);
            c.put(r, s, 16 * r + p < k0 ? t : T(0));
        }
}

// Tree node id: Rs := qr([Rs; R2]), Rs packed in LDS, R2 in c as well as, packed,
// at R2.  Panels that Rs calls close are done one column at a time.  In the narrow
// widths, where four panels hold little arithmetic, the whole merge is then done
// with one column per lane, which has the shorter chain; at 50 columns a
// single close panel would make it the slower way (20001 x 50, six decades,
// FP64: 279 us, 193 by panels).
template <typename T, int NC, bool WQ, typename Args>
__device__ __forceinline__ void merge_node(const Args& a, int id, const T* R2,
                                           Chunk<T, MergeRows<T, NC>::RB, Slots<NC>::NS>& c, T* Rs, T* work)
{
    T* Vn = WQ ? a.qs.Vn + (int64_t)id * Tri<NC>::kSize : nullptr;
    T* tau = WQ ? a.qs.tau_node + (int64_t)id * NC : nullptr;
    const uint64_t columns = close_columns<T, NC>(Rs);
    const bool bad = not_finite(c);
    unsigned close = 0;
    if (columns != 0 || bad) [[unlikely]] {
        if constexpr (NC <= kColumnMerge) {
            T v[NC];
            triangle_column<T, NC>(R2, v);
            merge_columns<T, NC, WQ>(v, Rs, tau, a.n);
            if constexpr (WQ) {
                int k = lane_id();
                asm volatile("" : "+v"(k));
#pragma unroll
                for (int i = 0; i < NC; ++i)
                    if (i <= k && k < NC) Vn[k + (Tri<NC>::off(i) - i)] = v[i];
            }
            return;
        }
        if (bad) isolate_not_finite<T, NC>(c);
#pragma unroll
        for (int P = 0; P < Slots<NC>::NS; ++P) close |= (columns >> 4 * P & 15) != 0 ? 1u << P : 0;
    }
    merge_panels<T, NC, WQ>(c, Rs, work, a.n, close, Vn, tau);
}

// ---- the fused leaf + tree kernel --------------------------------------------

// Copy a packed triangle from LDS to global memory, the reads first
template <typename T, int NC>
__device__ __forceinline__ void triangle_to_global(const T* src, T* __restrict__ dst)
{
    constexpr int NT = Tri<NC>::kSize;
    constexpr int U = (NT + kWave - 1) / kWave;
    const int lane = lane_id();
    T t[U];
#pragma unroll
    for (int u = 0; u < U; ++u) t[u] = src[lane + u * kWave < NT ? lane + u * kWave : 0];
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (lane + u * kWave < NT) dst[lane + u * kWave] = t[u];
}

// One chunk of a leaf: the panels in order, each followed by the loads of the
// next chunk's columns into its registers, which no later panel reads.  Panels
// past column n are left out (333333 x 20, Q and R in FP32: 286 us with them, 264
// without); their loads are not, so that their number is known.
template <typename T, int NC, int RPL, bool WQ, typename TIn>
__device__ __forceinline__ void leaf_chunk(Chunk<T, RPL, Slots<NC>::NS>& c, T* Rs, T* work, int q, int p,
                                           int n, unsigned& hard, Prefetch<T, RPL, TIn>& pf, const VSink<T>& vs)
{
    static_for<0, Slots<NC>::NS>([&](auto pc) {
        constexpr int P = decltype(pc)::value;
        if (4 * P < kMinColumns<NC> || 4 * P < n)
            panel_step<T, NC, RPL, RPL, P, WQ>(
                c, Rs, work, hard, [&](int rb, T v, const T(&tau)[4]) {
                    const int k = 4 * P + q;
                    if (k < n) vs.V[vs.cbase + 16 * rb + p + (int64_t)k * vs.ldv] = v;
                    if (rb == 0 && lane_id() < 4 && 4 * P + q < NC) vs.tau[4 * P + q] = of_column(tau, q);
                });
        prefetch_slot<T, RPL, TIn>(c, P, pf);
    });
}

// One leaf of one instance, then that instance's reduction tree: the body
// shared by the single-matrix kernel and the batched kernel.  `a` describes the
// instance (its matrix, leaf size and count, triangle slots, tree counters and
// output); `leaf` is this workgroup's leaf.  With WQ (the Q-factor mode) the
// leaf also writes its reflectors (a.qs.V, a.qs.tau_leaf), every merge those
// of the operator (a.qs.Vn, a.qs.tau_node), and the root the sign pattern of
// R's diagonal as the starting block of Q (a.qs.qblk, slot 0).  With
// a.stamps set, lane 0 writes the constant-rate clock at the start, at the
// end of the leaf phase and at exit, and the tree level at which it stopped
// (plus 100 for the root), to a.stamps[4 leaf + 0..3]: the split of the time
// between the leaves and the tree, measured.
template <typename T, int NC, int RPL, bool WQ = false, typename TIn = T>
__device__ __forceinline__ void leaf_phase(const LeafTreeArgs<T, TIn>& a, int leaf, T* Rs, T* red)
{
    constexpr int CH = 16 * RPL;                  // rows per chunk
    constexpr int NS = Slots<NC>::NS;
    const int lane = lane_id();
    // column 4s + q and row p + 16 r of register (r, s)
    using C = Chunk<T, RPL, NS>;
    const int q = C::q(lane), p = C::p(lane);
    const int64_t r0 = (int64_t)leaf * a.leaf_rows;
    const int64_t r1 = (r0 + a.leaf_rows < a.m) ? r0 + a.leaf_rows : a.m;
    const uint64_t t_start = a.stamps ? (uint64_t)wall_clock64() : 0;

    for (int i = lane; i < Tri<NC>::kPadded; i += kWave) Rs[i] = T(0);

    // step 1 of the method: the local factorisation of rows [r0, r1)
    if (r1 > r0) {
        C c;
        // Behind as many columns as the leaf has rows, rounding errors are left of
        // the others: those panels cannot be done at once (129 x 45 in
        // FP64: 73 us with the attempt, 61 without; 775 x 45 in FP32: 89 and 78)
        unsigned hard = r1 - r0 < a.n ? ~0u << ((int)(r1 - r0) / 4) : 0;
        wave_sync();
        const int64_t nfull = (r1 - r0) / CH, nchunks = (r1 - r0 + CH - 1) / CH;
        VSink<T> vs{};
        auto sink = [&](int64_t t) {
            if constexpr (WQ) {
                vs.V = a.qs.V;
                vs.ldv = a.qs.ldv;
                vs.cbase = r0 + t * CH;
                vs.tau = a.qs.tau_leaf + (vs.cbase / CH) * NC;
            }
        };
        // full chunks in a row are prefetched; the first one and a partial last
        // one are loaded here, row by row inside the leaf
        for (int64_t t = 0; t < nchunks;) {
#pragma unroll
            for (int r = 0; r < RPL; ++r) {
                const int64_t row = r0 + t * CH + p + 16 * r;
                const bool ok = row < r1;
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    const int k = 4 * s + q;
                    c.put(r, s, (ok && k < a.n) ? (T)a.A[row + (int64_t)k * a.lda] : T(0));
                }
            }
            // (where no full chunk follows, the prefetch reads the block of zeros: a
            // second copy of the chunk's code without it would cost more to fetch
            // than these loads)
            bool more;
            do {
                more = t + 1 < nfull;
                Prefetch<T, RPL, TIn> pf = make_prefetch<T, RPL, TIn>(
                    a.A, a.lda, more ? a.n : 0, more ? r0 + (t + 1) * CH : 0, q, p);
                sink(t);
                leaf_chunk<T, NC, RPL, WQ, TIn>(c, Rs, red, q, p, a.n, hard, pf, vs);
                ++t;
            } while (more);
        }
    }
    wave_sync();
    if (a.stamps && lane == 0) {
        a.stamps[4 * leaf] = t_start;
        a.stamps[4 * leaf + 1] = (uint64_t)wall_clock64();
    }
}

// The root, reached by leaf `leaf`'s wavefront at tree level `level`: positive
// diagonal, +0 below it, leading n-by-n block only (lane i writes row i, eight
// columns in flight).
template <typename T, int NC, bool WQ = false, typename TIn = T>
__device__ __forceinline__ void finish_root(const LeafTreeArgs<T, TIn>& a, int leaf, int level, const T* Rs)
{
    const int lane = lane_id();
    const int n = a.n;
    {
        const int i = lane < n ? lane : 0;
        const T* row = Rs + Tri<NC>::off(i) - i;
        const bool flip = __builtin_signbit(row[i]);
        for (int k0 = 0; k0 < n; k0 += 8) {
            T v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = row[k0 + u];      // past the row's end: inside the padding
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int k = k0 + u;
                const T x = k < i ? T(0) : (flip ? -v[u] : v[u]);
                if (lane < n && k < n) a.R[i + (int64_t)k * a.ldr] = x;
            }
        }
    }
    if (a.stamps && lane == 0) {
        a.stamps[4 * leaf + 2] = (uint64_t)wall_clock64();
        a.stamps[4 * leaf + 3] = (uint64_t)(100 + level);
    }
    if constexpr (WQ) {
        // R = D R_raw with D the diagonal of signs, so Q = Q_raw D: the tree
        // pass starts from [D; 0] (identity past column n)
        for (int idx = lane; idx < NC * NC; idx += kWave) {
            const int i = idx % NC, k = idx / NC;
            T d = T(0);
            if (i == k) d = (k < n && __builtin_signbit(Rs[Tri<NC>::off(k)])) ? T(-1) : T(1);
            a.qs.qblk[idx] = d;
        }
    }
}

// Step 2 from (node0, level0) on: the triangle of node node0 at tree level
// level0 is in Rs (this wavefront's leaf `leaf`, or the merge of the leaves
// below it); publish it, take the tickets up the tree, merge whenever this
// wavefront arrives second, and finish the root.
template <typename T, int NC, bool WQ = false, typename TIn = T>
__device__ __forceinline__ void tree_phase(const LeafTreeArgs<T, TIn>& a, int leaf, int node0, int level0, T* Rs,
                                           T* red)
{
    constexpr int NT = Tri<NC>::kSize;
    const int lane = lane_id();
    // step 2: binary reduction tree across leaves
    const int P = a.leaves;
    int node = node0;
    int level = level0;
    bool root = ((1 << level) >= P);
    if (!root) triangle_to_global<T, NC>(Rs, a.tri + (int64_t)node * NT);
    while (!root) {
        const int span = 1 << level;
        const bool is_left = (node & (2 * span - 1)) == 0;
        const int partner = is_left ? node + span : node - span;
        if (is_left && partner >= P) {          // no partner at this level: carry up
            ++level;
            root = (span * 2 >= P);
            continue;
        }
        const int left = is_left ? node : partner;
        const int id = left + span - 1;         // distinct for every (level, left) pair
        __threadfence();
        unsigned old = 0;
        if (lane == 0) old = atomicAdd(&a.tickets[id], 1u);
        old = (unsigned)__builtin_amdgcn_readfirstlane((int)old);
        if (old == 0) {                         // the partner will merge
            if (a.stamps && lane == 0) {
                a.stamps[4 * leaf + 2] = (uint64_t)wall_clock64();
                a.stamps[4 * leaf + 3] = (uint64_t)level;
            }
            return;
        }
        __threadfence();
        if (lane == 0) a.tickets[id] = 0u;      // both arrived: reset for the next call

        // the right (lower) operand in registers, the left one in LDS, so that
        // the lower index is on top
        Chunk<T, MergeRows<T, NC>::RB, Slots<NC>::NS> c;
        if (is_left) {
            triangle_chunk<T, NC>(a.tri + (int64_t)partner * NT, c);
        } else {
            triangle_chunk<T, NC>(Rs, c);
            wave_sync();
            triangle_to_lds<T, NC>(a.tri + (int64_t)partner * NT, Rs);
        }
        wave_sync();
        // (the right operand is in its slot in either case: its own wavefront put it there)
        merge_node<T, NC, WQ>(a, id, a.tri + (int64_t)(left + span) * NT, c, Rs, red);
        wave_sync();
        node = left;
        ++level;
        root = ((1 << level) >= P);
        if (!root) triangle_to_global<T, NC>(Rs, a.tri + (int64_t)node * NT);
    }

    finish_root<T, NC, WQ>(a, leaf, level, Rs);
}

// Workgroups are dispatched to the 8 XCDs in turn (workgroup g to XCD g mod 8),
// and each XCD has its own L2.  With P = 8a + b leaves, XCD x runs a + [x < b]
// workgroups; giving them the consecutive leaves starting at x a + min(x, b)
// makes tree siblings share an XCD at every level below the top three, so the
// stores, counters and loads of those merges stay in one L2.
constexpr int kXcds = 8;

__device__ __forceinline__ int xcd_local_leaf(int g, int P)
{
    const int a = P / kXcds, b = P % kXcds, x = g % kXcds;
    return x * a + (x < b ? x : b) + g / kXcds;
}

// Wavefronts per SIMD the register budget is held to: two where the chunk leaves
// room for the working set of a panel.  FP64 at 40 columns (160 registers) spilled
// up to 100 registers at two: at one, with half the leaves, Q and R of 10^6 x 40
// take 697 us (754 at two), 300000 x 40 with Q^T of ten columns 373 (426), R of 10^6 x
// 40 260 (271), of 4 10^6 x 40 605 (590).  156 registers (FP32, 50 columns, 12 rows)
// and FP32 at 64 columns (128) are better at two although the latter spills: R
// of 20001 x 64 188 us (215 at one), Q and R in FP64 at 32 columns (128) 10^6 x
// 32 580 (676).
template <typename T, int NC, int RPL>
struct LeafWaves {
    static constexpr int kChunkRegs = RPL * Slots<NC>::NS * (int)(sizeof(T) / 4);
    static constexpr int kPerSimd = kChunkRegs < 160 ? 2 : 1;
};

// A single leaf: no tree
template <typename T, int NC, int RPL, bool WQ = false>
__global__ void __launch_bounds__(kWave, (LeafWaves<T, NC, RPL>::kPerSimd)) tsqr_leaf_kernel(LeafTreeArgs<T> a)
{
    __shared__ T Rs[Tri<NC>::kPadded];
    __shared__ __align__(16) T red[PanelLds<T, RPL>::kElems];
    leaf_phase<T, NC, RPL, WQ>(a, 0, Rs, red);
    finish_root<T, NC, WQ>(a, 0, 0, Rs);
}

// Four leaves per workgroup, one wavefront each (one per SIMD of a compute
// unit at one wavefront per SIMD): the two lowest tree levels, whose partners
// then sit in the same workgroup, meet in LDS behind a workgroup barrier
// instead of through global memory, a release fence and a ticket.  Measured
// on a 1024-leaf tree, that global handoff costs 26 us at level 0 and 14 us at
// level 1, where every wavefront fences at once, against 2-6 us above.  The
// merges take the same operands in the same order (the lower index on top),
// so R is bit-identical to that of one leaf per workgroup, as the batched kernel
// has it.  The wavefronts of the last workgroup past the last leaf only keep
// the barriers; with at most four leaves no tree counter is touched.
template <typename T, int NC, int RPL, bool WQ = false>
__global__ void __launch_bounds__(4 * kWave, (LeafWaves<T, NC, RPL>::kPerSimd)) tsqr_leaf_tree4_kernel(LeafTreeArgs<T> a)
{
    __shared__ T Rs[4][Tri<NC>::kPadded];
    __shared__ __align__(16) T red[4][PanelLds<T, (RPL > 4 ? RPL : 4)>::kElems];
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));   // uniform per wavefront
    const int base = 4 * xcd_local_leaf(blockIdx.x, (a.leaves + 3) / 4);
    const int leaf = base + w;
    if (leaf < a.leaves) leaf_phase<T, NC, RPL, WQ>(a, leaf, Rs[w], red[w]);
    // level 0: leaf base + w (w even) takes base + w + 1 from below; level 1:
    // base takes base + 2.  One copy of the merge's code for both.
#pragma nounroll
    for (int level = 0; level < 2; ++level) {
        const int span = 1 << level;
        __syncthreads();
        if ((w & (2 * span - 1)) == 0) {
            if (leaf + span < a.leaves) {
                Chunk<T, MergeRows<T, NC>::RB, Slots<NC>::NS> c;
                triangle_chunk<T, NC>(Rs[w + span], c);
                merge_node<T, NC, WQ>(a, leaf + span - 1, Rs[w + span], c, Rs[w], red[w]);
            }
        } else if ((w & (span - 1)) == 0 && a.stamps && leaf < a.leaves && lane_id() == 0) {
            a.stamps[4 * leaf + 2] = (uint64_t)wall_clock64();
            a.stamps[4 * leaf + 3] = (uint64_t)level;
        }
    }
    // then the tree goes on through memory
    if (w == 0) tree_phase<T, NC, WQ>(a, leaf, base, 2, Rs[0], red[0]);
}

// Many independent instances in one launch: workgroup g takes tile
// tiles[g] = (instance, leaf); the tiles are ordered longest first so the
// hardware dispatcher starts the long leaves early and the short ones fill
// in.  Every instance has its own tree, so the tree of one instance overlaps
// the leaves of the others.
//
// With run_if set, the workgroups of an instance whose entry is 0 exit at once
// (the mixed-precision fallback: only instances whose correction failed are
// refactored, decided on the device).  With stamps set, workgroup g writes
// the constant-rate clock when it starts and when it is done (its leaf and
// whatever merges it performed) to stamps[2g], stamps[2g + 1], which measures
// the schedule.  TIn is the storage type of A.
template <typename T, int NC, int RPL, typename TIn = T>
__global__ void __launch_bounds__(kWave, (LeafWaves<T, NC, RPL>::kPerSimd)) tsqr_batch_kernel(BatchArgs<T, TIn> b)
{
    __shared__ T Rs[Tri<NC>::kPadded];
    __shared__ __align__(16) T red[PanelLds<T, (RPL > 4 ? RPL : 4)>::kElems];
    const uint64_t t_start = b.stamps ? (uint64_t)wall_clock64() : 0;
    const BatchTile t = b.tiles[blockIdx.x];
    if (b.run_if && b.run_if[t.inst] == 0) return;
    const BatchInstance in = b.inst[t.inst];
    LeafTreeArgs<T, TIn> a;
    a.A = b.A + in.a_off;
    a.m = in.m;
    a.lda = in.lda;
    a.n = b.n;
    a.leaf_rows = in.leaf_rows;
    a.leaves = in.leaves;
    a.tri = b.tri + in.tri_off;
    a.tickets = b.tickets + in.ticket_off;
    a.R = b.R + (int64_t)t.inst * b.ldr * b.n;
    a.ldr = b.ldr;
    a.qs = QStore<T>{};
    leaf_phase<T, NC, RPL, false, TIn>(a, t.leaf, Rs, red);
    tree_phase<T, NC, false, TIn>(a, t.leaf, t.leaf, 0, Rs, red);
    if (b.stamps && threadIdx.x == 0) {
        b.stamps[2 * blockIdx.x] = t_start;
        b.stamps[2 * blockIdx.x + 1] = (uint64_t)wall_clock64();
    }
}

// ---- the paper's operator as a single-workgroup kernel -------------------------

template <typename T, int NC>
__global__ void __launch_bounds__(kWave) qr_uppers_kernel(int n, T* R1, T* R2, T* tau)
{
    constexpr int NT = Tri<NC>::kSize;
    __shared__ T Rs[Tri<NC>::kPadded];
    __shared__ T R2s[Tri<NC>::kPadded];
    __shared__ T taus[NC];
    const int lane = threadIdx.x;
    for (int idx = lane; idx < NT; idx += kWave) {
        // packed index -> (row, column)
        int i = 0;
        while (Tri<NC>::off(i + 1) <= idx) ++i;
        const int k = i + (idx - Tri<NC>::off(i));
        const bool in = i < n && k < n;
        Rs[idx] = in ? R1[i + (int64_t)k * n] : T(0);
        R2s[idx] = in ? R2[i + (int64_t)k * n] : T(0);
    }
    wave_sync();
    T v[NC];
    triangle_column<T, NC>(R2s, v);
    wave_sync();
    merge_columns<T, NC, true>(v, Rs, taus);
    wave_sync();
    for (int idx = lane; idx < n * n; idx += kWave) {
        const int i = idx % n, k = idx / n;
        if (k >= i) R1[idx] = Rs[Tri<NC>::off(i) + (k - i)];
    }
#pragma unroll
    for (int i = 0; i < NC; ++i)
        if (i <= lane && lane < n) R2[i + (int64_t)lane * n] = v[i];
    if (lane < n) tau[lane] = taus[lane];
}

}  // namespace dev
}  // namespace tsqr
