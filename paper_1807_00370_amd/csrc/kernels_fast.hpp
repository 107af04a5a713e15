// One-wave kernels of a reduction level for block sizes 9 to 32 (elimination,
// back substitution) and up to 64 (reduced-system products).  Same
// arithmetic and outputs as the work-group kernels in kernels.hpp; the
// difference is the mapping onto a single wave64:
//
//   k_reduce_m  the products P^H P, Q^H Q, P^H Q, P^H g, Q^H g of Eq.
//               (Formulas) on MFMA (16x16x4, real-pair 4-multiply complex
//               form), operands loaded from HBM straight into the MFMA lane
//               layout; diagonal blocks are written as their lower triangle
//               only (the Hermitian reading every consumer uses).
//   k_elim_mf   (8 < m <= 32) the Cholesky by 16 x 16 tiles (tile_chol), then
//               the substitutions on MFMA with the inverse diagonal tiles.
//   k_back_mf   w = g - Q x_{p-d} - P x_{p+d} on MFMA, then L^H x = w tile by
//               tile on MFMA with the inverse diagonal tiles.
#pragma once

#include "kernels.hpp"

namespace crs {

typedef double d4v __attribute__((ext_vector_type(4)));
typedef float f4v __attribute__((ext_vector_type(4)));

template <class T>
struct MF;
template <>
struct MF<double> {
    using v4 = d4v;
    static __device__ __forceinline__ v4 mma(double a, double b, v4 c)
    {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    // output row of accumulator register v in a lane with kr = lane / 16
    static __device__ __forceinline__ int row(int kr, int v) { return kr + 4 * v; }
};
template <>
struct MF<float> {
    using v4 = f4v;
    static __device__ __forceinline__ v4 mma(float a, float b, v4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int kr, int v) { return 4 * kr + v; }
};

template <class T>
__device__ __forceinline__ cx<T> czero()
{
    return cx<T>{T(0), T(0)};
}

// *p where ok, else zero.  The load is issued in every lane (from q, a valid
// address, where ok is false), so no branch surrounds it and the compiler's
// count of the wave's memory operations in flight stays exact: a wait for
// one group of a software pipeline's loads then does not also wait for the
// group issued after it.
template <class T>
__device__ __forceinline__ cx<T> ld_or0(const cx<T>* p, const cx<T>* q, bool ok)
{
    const cx<T> v = *(ok ? p : q);
    return ok ? v : czero<T>();
}

// 1 / sqrt(d) from the hardware reciprocal square root and one Newton step
// (relative error about the unit roundoff); NaN for d < 0, inf for d = 0.
__device__ __forceinline__ double rsqrt_nr(double d)
{
    const double r = __builtin_amdgcn_rsq(d);
    return r * fma(-0.5 * d * r, r, 1.5);
}
__device__ __forceinline__ float rsqrt_nr(float d)
{
    const float r = __builtin_amdgcn_rsqf(d);
    return r * fmaf(-0.5f * d * r, r, 1.5f);
}

// Orders the LDS accesses of one wave: stores before the call are seen by
// loads after it from any lane of the same wave (a wave's LDS operations
// complete in order; the fences keep the compiler from moving them).
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Value of x in lane N of each 16-lane row, in every lane of that row: one
// data-parallel move per dword pair (the row broadcast of the gfx9 matrix
// GPUs), no scalar registers and no LDS round trip.
template <int N>
__device__ __forceinline__ double row_bcast(double x)
{
    return __builtin_amdgcn_update_dpp(x, x, 0x150 + N, 0xf, 0xf, true);
}
template <int N>
__device__ __forceinline__ float row_bcast(float x)
{
    const int v = __float_as_int(x);
    return __int_as_float(__builtin_amdgcn_update_dpp(v, v, 0x150 + N, 0xf, 0xf, true));
}

// MFMA 16x16x4 lane layout (wave64, checked on gfx950): lane l supplies
// A[l % 16][l / 16] and B[l / 16][l % 16]; accumulator register v of lane l
// holds D[row][l % 16] with row = 4 (l / 16) + v for the f32 instruction and
// row = l / 16 + 4 v for the f64 instruction (MF<T>::row).

// Operands are loaded four k-steps at a time, one group ahead of the MFMAs
// that consume the previous group; the scheduling barrier keeps the compiler
// from hoisting every load of the tile to the top (register pressure).
constexpr int kGroup = 4;

// Accumulators of the three-multiplication (3M) complex product: with
// a = op(A), b = op(B) split into real and imaginary parts,
//   t1 += Re a Re b,  t2 += Im a Im b,  t3 += (Re a + Im a)(Re b + Im b),
// and the product is Re = t1 - t2, Im = t3 - t1 - t2: three real MFMAs per
// complex contraction step instead of four.  The real part is the 4M one;
// the imaginary part carries an absolute error of a few units of roundoff
// times sum_t (|Re a| + |Im a|)(|Re b| + |Im b|) (normwise stable, not
// componentwise; Higham, Accuracy and Stability of Numerical Algorithms,
// Section 23.2.4).  For real data t2 = 0 and t3 = t1 bit for bit, so the
// imaginary part is exactly zero.
//
// RE (real data: every imaginary part is zero): only t1 is formed, one real
// MFMA per contraction step, Re = t1 and Im = 0 -- the same values the 3M
// form gives for real data (t2 = 0, t3 = t1), with a third of the MFMAs.
template <class T, int RM, int RN, bool RE = false>
struct Acc3 {
    using v4 = typename MF<T>::v4;
    v4 t1[RM][RN], t2[RE ? 1 : RM][RE ? 1 : RN], t3[RE ? 1 : RM][RE ? 1 : RN];
    __device__ __forceinline__ void zero()
    {
#pragma unroll
        for (int i = 0; i < RM; ++i)
#pragma unroll
            for (int j = 0; j < RN; ++j) {
                t1[i][j] = v4{0, 0, 0, 0};
                if constexpr (!RE)
                    t2[i][j] = t3[i][j] = v4{0, 0, 0, 0};
            }
    }
    __device__ __forceinline__ T re(int i, int j, int v) const
    {
        if constexpr (RE)
            return t1[i][j][v];
        else
            return t1[i][j][v] - t2[i][j][v];
    }
    __device__ __forceinline__ T im(int i, int j, int v) const
    {
        if constexpr (RE)
            return T(0);
        else
            return t3[i][j][v] - t1[i][j][v] - t2[i][j][v];
    }
    // acc(i, j) += a b for one contraction step of real-pair operands
    __device__ __forceinline__ void step(int i, int j, T ar, T ai, T br, T bi)
    {
        t1[i][j] = MF<T>::mma(ar, br, t1[i][j]);
        if constexpr (!RE) {
            t2[i][j] = MF<T>::mma(ai, bi, t2[i][j]);
            t3[i][j] = MF<T>::mma(ar + ai, br + bi, t3[i][j]);
        }
    }
};

// (cr, ci) += X^H Y on the 16 x 16 tile with rows cx0.. (columns of X) and
// columns cy0.. (columns of Y); X, Y row-major, contraction over their first
// kd rows.  Out-of-range rows and columns read as zero.
template <class T, int KS>
__device__ __forceinline__ void tile_hn(typename MF<T>::v4& cr, typename MF<T>::v4& ci,
                                        const cx<T>* __restrict__ X, int ldx, int ncx, int cx0,
                                        const cx<T>* __restrict__ Y, int ldy, int ncy, int cy0,
                                        int kd)
{
    constexpr int G = KS < kGroup ? KS : kGroup, NG = KS / G;
    const int lane = threadIdx.x & 63, kr = lane >> 4, cc = lane & 15;
    const int ax = cx0 + cc, by = cy0 + cc;
    const bool okx = ax < ncx, oky = by < ncy;
    const cx<T>* xb = X + (kr * ldx + ax);
    const cx<T>* yq = Y + (kr * ldy + by);
    const int sx = 4 * ldx, sy = 4 * ldy;
    cx<T> xa[2][G], yb[2][G];
    auto load = [&](int g, int b) {
#pragma unroll
        for (int u = 0; u < G; ++u) {
            const int ks = g * G + u, t = 4 * ks + kr;
            xa[b][u] = ld_or0(xb + ks * sx, X, t < kd && okx);
            yb[b][u] = ld_or0(yq + ks * sy, Y, t < kd && oky);
        }
    };
    load(0, 0);
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        if (g + 1 < NG)
            load(g + 1, (g + 1) & 1);
#pragma unroll
        for (int u = 0; u < G; ++u) {
            const cx<T> a = xa[g & 1][u], b = yb[g & 1][u];
            cr = MF<T>::mma(a.r, b.r, cr);
            cr = MF<T>::mma(a.i, b.i, cr);
            ci = MF<T>::mma(a.r, b.i, ci);
            ci = MF<T>::mma(-a.i, b.r, ci);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// acc += X Y in the 3M form on the tile with rows rx0.. (rows of X) and columns
// cy0.. (columns of Y); contraction over kd columns of X / rows of Y.
template <class T, int KS>
__device__ __forceinline__ void tile_nn3(Acc3<T, 1, 1>& acc, const cx<T>* __restrict__ X, int ldx,
                                         int nrx, int rx0, const cx<T>* __restrict__ Y, int ldy,
                                         int ncy, int cy0, int kd)
{
    constexpr int G = KS < kGroup ? KS : kGroup, NG = KS / G;
    const int lane = threadIdx.x & 63, kr = lane >> 4, cc = lane & 15;
    const int ar = rx0 + cc, by = cy0 + cc;
    const bool okx = ar < nrx, oky = by < ncy;
    const cx<T>* xb = X + (ar * ldx + kr);
    const cx<T>* yq = Y + (kr * ldy + by);
    const int sy = 4 * ldy;
    cx<T> xa[2][G], yb[2][G];
    auto load = [&](int g, int b) {
#pragma unroll
        for (int u = 0; u < G; ++u) {
            const int ks = g * G + u, t = 4 * ks + kr;
            xa[b][u] = ld_or0(xb + 4 * ks, X, t < kd && okx);
            yb[b][u] = ld_or0(yq + ks * sy, Y, t < kd && oky);
        }
    };
    load(0, 0);
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        if (g + 1 < NG)
            load(g + 1, (g + 1) & 1);
#pragma unroll
        for (int u = 0; u < G; ++u) {
            const cx<T> a = xa[g & 1][u], b = yb[g & 1][u];
            acc.t1[0][0] = MF<T>::mma(a.r, b.r, acc.t1[0][0]);
            acc.t2[0][0] = MF<T>::mma(a.i, b.i, acc.t2[0][0]);
            acc.t3[0][0] = MF<T>::mma(a.r + a.i, b.r + b.i, acc.t3[0][0]);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// --------------------------------------------------- 16 x 16 tiles in registers

// Cholesky factor L and inverse D = L^{-1} of one 16 x 16 tile by one wave, on
// registers and MFMA.  Lane (kr, cc) = (lane / 16, lane % 16) keeps the four
// entries u = kr + 4 v of row cc of the tile: this is the accumulator layout
// of the FP64 16x16x4 instruction for the transposed tile, and register v
// over the four lane groups is the panel of the columns 4 v .. 4 v + 3.  Per
// panel of four columns:
//   - every lane gathers its row's four panel entries (lane swaps) and
//     factors the panel on its own row, pivots and finished columns coming by
//     row broadcasts;
//   - beside it lane group k eliminates column k of the panel's identity,
//     which leaves M = [D_pp; -L_below D_pp], one entry per lane;
//   - one 4-term product on MFMA adds the panel's products to the sums of the
//     whole tile, W += L_p L_p^H (the lane's own entry of L_p is both
//     operands), and one more forms all of D, D_{p..} = M D_p (the lane's own
//     accumulator is the right operand).
// Every entry's products are summed from zero and subtracted from it once, when
// its column is factored: sums that start from the entry round every product
// at the diagonal's size, and the error of a solve was 5 to 8 % larger (m = 16:
// 6.67e-16 against 6.98e-16, m = 32: 7.55e-16 against 8.09e-16).
// A panel's chain is four pivots long; the 16 x 16 updates leave it.  The
// chain of dependent FP64 operations bounds it.  Measured, one wave: 5740 cycles
// for L and D of FP64 complex data, 3040 of real data; a column at a time on the
// vector unit, every lane on its whole row, 8700 with twice the instructions
// (complex).  The diagonal step of the tiled Cholesky went from 7.8 to about 2.5 us
// by it.  Panels past the block's edge are left out (a test per column instead
// cost 1 % at m = 32).
//
// The tile is factored in double for every type; for float the columns are
// rounded to float as they are finished, so that D is the inverse of the L
// that is stored.
template <class T>
__device__ __forceinline__ double round_to(double x)
{
    return sizeof(T) == 8 ? x : (double)(float)x;
}

// o[g] = x of the lane with the same cc in lane group g.
__device__ __forceinline__ void gather_groups(double x, double (&o)[4])
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(x);
    unsigned w[2] = {(unsigned)b, (unsigned)(b >> 32)}, q[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        // odd 16-lane rows of the first operand swap with even rows of the
        // second, then upper and lower halves
        const auto t = __builtin_amdgcn_permlane16_swap(w[i], w[i], false, false);
        const auto e = __builtin_amdgcn_permlane32_swap(t[0], t[0], false, false);
        const auto d = __builtin_amdgcn_permlane32_swap(t[1], t[1], false, false);
        q[i][0] = e[0];
        q[i][1] = d[0];
        q[i][2] = e[1];
        q[i][3] = d[1];
    }
#pragma unroll
    for (int g = 0; g < 4; ++g)
        o[g] = __longlong_as_double((long long)(((unsigned long long)q[1][g] << 32) | q[0][g]));
}

template <bool RE>
__device__ __forceinline__ void gather_groups(const cx<double> x, cx<double> (&o)[4])
{
    double r[4], i[4] = {0, 0, 0, 0};
    gather_groups(x.r, r);
    if constexpr (!RE)
        gather_groups(x.i, i);
#pragma unroll
    for (int g = 0; g < 4; ++g)
        o[g] = cx<double>{r[g], i[g]};
}

// Column C = 4 P + J of the panel's identity: row C is scaled by the inverse
// pivot, the rows below subtract their L_rC times it.
template <int C, bool RE>
__device__ __forceinline__ void tile_inv_col(cx<double>& q, const cx<double> l, double inv, int r)
{
    const cx<double> z{row_bcast<C>(q.r) * inv, RE ? 0.0 : row_bcast<C>(q.i) * inv};
    const cx<double> lm{r > C ? l.r : 0.0, RE ? 0.0 : (r > C ? l.i : 0.0)};
    cx<double> t{fma(-lm.r, z.r, q.r), 0.0};
    if constexpr (!RE) {
        t.r = fma(lm.i, z.i, t.r);
        t.i = fma(-lm.r, z.i, q.i);
        t.i = fma(-lm.i, z.r, t.i);
    }
    q.r = r == C ? z.r : t.r;
    if constexpr (!RE)
        q.i = r == C ? z.i : t.i;
}

template <class T, bool RE, int P, int J>
__device__ __forceinline__ void tile_chol_col(const cx<double> (&s)[4], cx<double> (&c)[4], cx<double>& q,
                                              int r, int mr, unsigned long long& fail)
{
    constexpr int C = 4 * P + J;
    const cx<double> x{(sizeof(T) == 8 ? s[J].r : 0.0) - c[J].r,
                       RE ? 0.0 : (sizeof(T) == 8 ? s[J].i : 0.0) - c[J].i};
    const double d = row_bcast<C>(x.r);
    const double inv = round_to<T>(rsqrt_nr(d));
    fail |= C < mr ? __ballot(!(d > 0.0)) : 0ull;
    asm volatile("" : "+s"(fail)); // compared now, not with all 16 pivots kept
    const cx<double> l{round_to<T>(x.r * inv), RE ? 0.0 : round_to<T>(x.i * inv)};
    auto add = [&](cx<double>& w, double ur, double ui) { // w += l conj(u)
        w.r = fma(l.r, ur, w.r);
        if constexpr (!RE) {
            w.r = fma(l.i, ui, w.r);
            w.i = fma(l.i, ur, w.i);
            w.i = fma(-l.r, ui, w.i);
        }
    };
    if constexpr (J < 1)
        add(c[1], row_bcast<4 * P + 1>(l.r), RE ? 0.0 : row_bcast<4 * P + 1>(l.i));
    if constexpr (J < 2)
        add(c[2], row_bcast<4 * P + 2>(l.r), RE ? 0.0 : row_bcast<4 * P + 2>(l.i));
    if constexpr (J < 3)
        add(c[3], row_bcast<4 * P + 3>(l.r), RE ? 0.0 : row_bcast<4 * P + 3>(l.i));
    tile_inv_col<C, RE>(q, l, inv, r);
    c[J] = l;
}

// D over panel P: rows of the panel are replaced, the rows below updated.
template <bool RE, int P>
__device__ __forceinline__ void tile_inv_panel(d4v& er, d4v& ei, const cx<double> q)
{
    const double br = er[P], bi = RE ? 0.0 : ei[P];
    er[P] = 0.0;
    er = MF<double>::mma(q.r, br, er);
    if constexpr (!RE) {
        ei[P] = 0.0;
        ei = MF<double>::mma(q.r, bi, ei);
        er = MF<double>::mma(-q.i, bi, er);
        ei = MF<double>::mma(q.i, br, ei);
    }
}

// The panel's entries s and the sums c of the products to subtract from them
// (T = float: c holds both, in double).
template <class T, bool RE, bool HW, int P>
__device__ __forceinline__ void tile_chol_panel(const cx<double> s, d4v& wr, d4v& wi, d4v& er, d4v& ei,
                                                cx<double> (&L)[4], int r, int g, int mr,
                                                unsigned long long& fail)
{
    cx<double> a[4], c[4], q{r == 4 * P + g ? 1.0 : 0.0, 0.0};
    if constexpr (sizeof(T) == 4)
        gather_groups<RE>(cx<double>{wr[P] - s.r, wi[P] - s.i}, c);
    else {
        gather_groups<RE>(s, a);
        if constexpr (HW || P > 0)
            gather_groups<RE>(cx<double>{wr[P], wi[P]}, c);
        else
            c[0] = c[1] = c[2] = c[3] = czero<double>();
    }
    tile_chol_col<T, RE, P, 0>(a, c, q, r, mr, fail);
    tile_chol_col<T, RE, P, 1>(a, c, q, r, mr, fail);
    tile_chol_col<T, RE, P, 2>(a, c, q, r, mr, fail);
    tile_chol_col<T, RE, P, 3>(a, c, q, r, mr, fail);
    const bool b0 = g & 1, b1 = g & 2;
    cx<double> l;
    l.r = b1 ? (b0 ? c[3].r : c[2].r) : (b0 ? c[1].r : c[0].r);
    l.i = RE ? 0.0 : (b1 ? (b0 ? c[3].i : c[2].i) : (b0 ? c[1].i : c[0].i));
    L[P] = l;
    if constexpr (P < 3) {
        wr = MF<double>::mma(l.r, l.r, wr);
        if constexpr (!RE) {
            wi = MF<double>::mma(l.r, l.i, wi);
            wr = MF<double>::mma(l.i, l.i, wr);
            wi = MF<double>::mma(-l.i, l.r, wi);
        }
    }
    tile_inv_panel<RE, P>(er, ei, q);
    __builtin_amdgcn_sched_barrier(0);
}

__device__ __forceinline__ void tile_identity(d4v& er, d4v& ei, int r, int g)
{
#pragma unroll
    for (int v = 0; v < 4; ++v)
        er[v] = g + 4 * v == r ? 1.0 : 0.0;
    ei = d4v{0, 0, 0, 0};
}

// s: the lane's entries (cc, kr + 4 v) of the tile (those right of the
// diagonal may hold anything), wr + i wi: of the products to subtract from it
// (HW: not all zero) -> L: the same entries of the factor, the diagonal as {L_rr, 1 / L_rr}; e:
// entries (kr + 4 v, cc) of D.  Returns true if one of the first mr pivots is
// not > 0 (the same in every lane).
template <class T, bool RE = false, bool HW = true>
__device__ __forceinline__ bool tile_chol(const cx<double> (&s)[4], d4v wr, d4v wi, cx<double> (&L)[4],
                                          cx<double> (&e)[4], int mr)
{
    const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
    d4v er, ei;
    tile_identity(er, ei, r, g);
    unsigned long long fail = 0;
    L[1] = L[2] = L[3] = czero<double>();
    mr = __builtin_amdgcn_readfirstlane(mr);
    // panels past the block's edge hold identity rows, which D has already
    tile_chol_panel<T, RE, HW, 0>(s[0], wr, wi, er, ei, L, r, g, mr, fail);
    if (mr > 4) {
        tile_chol_panel<T, RE, HW, 1>(s[1], wr, wi, er, ei, L, r, g, mr, fail);
        if (mr > 8) {
            tile_chol_panel<T, RE, HW, 2>(s[2], wr, wi, er, ei, L, r, g, mr, fail);
            if (mr > 12)
                tile_chol_panel<T, RE, HW, 3>(s[3], wr, wi, er, ei, L, r, g, mr, fail);
        }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        e[v] = cx<double>{er[v], ei[v]};
        if (g + 4 * v == r) // the inverse pivot is D's diagonal
            L[v].i = er[v];
    }
    return fail != 0;
}
template <class T, bool RE = false>
__device__ __forceinline__ bool tile_chol(const cx<double> (&s)[4], cx<double> (&L)[4],
                                          cx<double> (&e)[4], int mr)
{
    return tile_chol<T, RE, false>(s, d4v{0, 0, 0, 0}, d4v{0, 0, 0, 0}, L, e, mr);
}

// Storage of a factor of 8 < m <= 32 (in LDS and in the workspace): the packed
// lower triangle, row r at r (r + 1) / 2, with L_10 in its place and the
// inverse diagonal tiles D_I in place of L_II.  D_I is as large as L_II, and
// no later pass needs L_II itself.

// The lane's entries (cc, kr + 4 v) of diagonal tile I of such a triangle of
// A (entries right of the diagonal: the diagonal's), identity rows past m.
template <class T>
__device__ __forceinline__ void tile_load(const cx<T>* sL, int I, int m, cx<double> (&s)[4])
{
    const int lane = threadIdx.x & 63, kr = lane >> 4, r = lane & 15, gi = 16 * I + r;
    const cx<T>* row = sL + gi * (gi + 1) / 2 + 16 * I;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        s[v] = cvt<double>(row[min(kr + 4 * v, r)]);
        if (gi >= m)
            s[v] = cx<double>{kr + 4 * v == r ? 1.0 : 0.0, 0.0};
    }
}
// D_I (entries (kr + 4 v, cc), as tile_chol leaves them) into the triangle.
template <class T>
__device__ __forceinline__ void tile_store(cx<T>* sL, int I, int m, const cx<double> (&e)[4])
{
    const int lane = threadIdx.x & 63, kr = lane >> 4, cc = lane & 15;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int q = kr + 4 * v, gi = 16 * I + q;
        if (gi < m && cc <= q)
            sL[gi * (gi + 1) / 2 + 16 * I + cc] = cvt<T>(e[v]);
    }
}
// Operands of the MFMA products: D_I[cc][MF::row(kr, v)] (adj: the conjugate
// of D_I[MF::row(kr, v)][cc]).  Rows past m are identity rows.
template <class T, bool adj>
__device__ __forceinline__ void tile_operand(const cx<T>* sL, int I, int m, cx<T> (&aD)[4])
{
    const int lane = threadIdx.x & 63, kr = lane >> 4, cc = lane & 15;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int q = MF<T>::row(kr, v), i = adj ? q : cc, j = adj ? cc : q, gi = 16 * I + i;
        const cx<T> x = sL[gi * (gi + 1) / 2 + 16 * I + min(i, j)];
        const bool ok = gi < m && j <= i;
        aD[v] = ok ? cx<T>{x.r, adj ? -x.i : x.i} : cx<T>{gi >= m && i == j ? T(1) : T(0), T(0)};
    }
}
// The packed triangle between memory and LDS, a lane's elements e = lane +
// 64 q: all loads issued before the first is used; lanes past the end move the
// last element (the same value), so no branch holds one back.
template <class T, int MT>
__device__ __forceinline__ void packed_load(cx<T>* sL, const cx<T>* __restrict__ L, int m)
{
    constexpr int NE = (MT * (MT + 1) / 2 + 63) / 64;
    const int lane = threadIdx.x & 63, np = m * (m + 1) / 2;
    cx<T> x[NE];
#pragma unroll
    for (int q = 0; q < NE; ++q)
        x[q] = L[min(lane + 64 * q, np - 1)];
#pragma unroll
    for (int q = 0; q < NE; ++q)
        sL[min(lane + 64 * q, np - 1)] = x[q];
    wave_lds_sync();
}

// ---------------------------------------------------------------- k_elim_mf

// Elimination for block sizes 8 < m <= 32 on MFMA.  The Cholesky runs by 16 x
// 16 tiles: tile_chol of the first gives L_00 and D_0 = L_00^{-1}, then L_10 =
// A_10 D_0^H, S_11 = A_11 - L_10 L_10^H and tile_chol again.  Each 16-column
// strip G of [B_p^H | B_{p-d} | y_p] is solved tile by tile, X_0 = D_0 G_0 and
// X_1 = D_1 (G_1 - L_10 X_0): register v of a lane's accumulator holds row
// MF::row(kr, v) of its column, which is the right operand of contraction
// step v when the left operand supplies column MF::row(kr, v), so the
// products chain through the accumulators.  Right-hand sides are read from
// memory straight into that layout, the first strip's before the Cholesky,
// each next strip while the current one is solved.
//
// What is stored is L_10 and the D tiles in place of L's diagonal tiles: the
// later passes (right-hand side alone, back substitution) start with the
// operands they need and invert nothing.  A level of 64 blocks, m = 32, FP64
// complex, k = 16: 18.2 -> 14.4 us with the matrix, 8.0 -> 5.9 us without; 8192
// blocks (bound by HBM): 158 -> 153 us and 49 -> 41 us.  A and the factor move through LDS so that every access to memory is
// linear: the same loads straight into the tile layout (64-byte pieces) cost
// 30 % at 8192 blocks.
//
// The register budget is held to three waves per SIMD (168 VGPRs for FP64,
// m = 32, no spills).
//
// nsplit waves share a block: wave sp solves strips sp, sp + nsplit, ...
// Each of them factors the block itself (a few microseconds of latency,
// no cross-wave synchronisation); wave 0 alone stores L and raises the
// breakdown flag.  Levels with few blocks use nsplit > 1 to shorten the
// chain of strips that one wave walks through.
template <class T, int MT, class EI = cx<T>>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3, 8))) void k_elim_mf(const Seg* __restrict__ segs, int nseg,
                                                   int64_t total, int nsplit,
                                                   const EI* __restrict__ inA,
                                                   const EI* __restrict__ inB,
                                                   const EI* __restrict__ iny,
                                                   cx<T>* __restrict__ W,
                                                   unsigned long long* __restrict__ flags,
                                                   int with_mat, int with_rhs)
{
    static_assert(MT == 16 || MT == 32, "one or two 16-row tiles");
    using v4 = typename MF<T>::v4;
    constexpr int S = MT / 16;
    constexpr int NP = MT * (MT + 1) / 2;
    __shared__ cx<T> sL[NP]; // packed A, then the factor
    const int lane = threadIdx.x, kr = lane >> 4, cc = lane & 15;
    const int64_t w = blockIdx.x / nsplit;
    const int sp = (int)(blockIdx.x - w * nsplit);
    if (w >= total)
        return;
    const Seg& s = segs[find_seg(segs, nseg, w)];
    const int64_t t = w - s.w0;
    const int p = s.e0 + (int)t * s.es;
    const int m = s.m, k = s.k, d = s.d;
    const int64_t mm = (int64_t)m * m, mk = (int64_t)m * k;
    const bool hasPrev = p - d >= 0, hasNext = p + d < s.n;
    if ((flags[s.sys] >> 40) < (unsigned long long)s.level)
        return; // broke down at an earlier level: nothing left to do
    cx<T>* Lg = W + s.oL + t * mm;

    // strips: S of B_p^H (into P), S of B_{p-d} (into Q), ceil(k / 16) of y_p
    const int nP = (with_mat && hasNext) ? S : 0;
    const int nQ = (with_mat && hasPrev) ? S : 0;
    const int nst = nP + nQ + (with_rhs ? (k + 15) / 16 : 0);
    const EI* Bp = inB + s.oB + (int64_t)p * mm;
    const EI* Bq = inB + s.oB + (int64_t)(p - d) * mm;
    const EI* yp = iny + s.oy + (int64_t)p * mk;
    // element (r, c) of strip st's source is base[r * sr + c * sc], conjugated
    // for B_p^H
#define CRS_LOAD_STRIP(st, g)                                                                      \
    do {                                                                                           \
        const int src_ = (st) < nP ? 0 : ((st) < nP + nQ ? 1 : 2);                                 \
        const int c_ = 16 * (src_ == 0 ? (st) : (src_ == 1 ? (st) - nP : (st) - nP - nQ)) + cc;    \
        const EI* base_ = src_ == 0 ? Bp : (src_ == 1 ? Bq : yp);                              \
        const int sr_ = src_ == 0 ? 1 : (src_ == 1 ? m : k), sc_ = src_ == 0 ? m : 1;               \
        const bool okc_ = c_ < (src_ == 2 ? k : m);                                                \
        const T cj_ = src_ == 0 ? T(-1) : T(1);                                                    \
        const EI* col_ = base_ + (okc_ ? c_ : 0) * sc_;                                        \
        _Pragma("unroll") for (int I_ = 0; I_ < S; ++I_)                                           \
            _Pragma("unroll") for (int v_ = 0; v_ < 4; ++v_)                                       \
            {                                                                                      \
                const int r_ = 16 * I_ + MF<T>::row(kr, v_);                                       \
                const bool ok_ = okc_ && r_ < m;                                                   \
                const cx<T> x_ = cvt<T>(col_[(ok_ ? r_ : 0) * sr_]);                               \
                g[I_][v_] = ok_ ? cx<T>{x_.r, cj_ * x_.i} : czero<T>();                            \
            }                                                                                      \
    } while (0)
    cx<T> gn[S][4];

    cx<T> aL[4], aD[S][4]; // left operands: L_10, then the D tiles
    const int i1 = 16 + cc;
    cx<T>* row1 = sL + i1 * (i1 + 1) / 2; // row i1 of the triangle
    if (with_mat) {
        const EI* Ap = inA + s.oA + (int64_t)p * mm;
        const int np = m * (m + 1) / 2;
        constexpr int NE = (NP + 63) / 64;
        EI av[NE];
#pragma unroll
        for (int q = 0; q < NE; ++q) {
            const int e = min(lane + 64 * q, np - 1), r = tri_row(e);
            av[q] = Ap[r * m + e - r * (r + 1) / 2];
        }
        // the first strip's loads return during the factorization
        if (sp < nst)
            CRS_LOAD_STRIP(sp, gn);
#pragma unroll
        for (int q = 0; q < NE; ++q)
            sL[min(lane + 64 * q, np - 1)] = cvt<T>(av[q]);
        wave_lds_sync();
        cx<double> t[4], L[4], e[4];
        tile_load<T>(sL, 0, m, t);
        bool fail = tile_chol<T>(t, L, e, m);
        tile_store<T>(sL, 0, m, e);
        wave_lds_sync();
        tile_operand<T, false>(sL, 0, m, aD[0]);
        if constexpr (S == 2) {
            // L_10 as a left operand: conj(L_10)^T = D_0 A_10^H comes out of
            // the products with row MF::row(kr, v) of column cc in register
            // v, which is conj(L_10[cc][MF::row(kr, v)])
            v4 zr = {0, 0, 0, 0}, zi = {0, 0, 0, 0};
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const cx<T> x = row1[MF<T>::row(kr, v)], d = aD[0][v];
                const T br = i1 < m ? x.r : T(0), bi = i1 < m ? -x.i : T(0);
                zr = MF<T>::mma(d.r, br, zr);
                zi = MF<T>::mma(d.r, bi, zi);
                zr = MF<T>::mma(-d.i, bi, zr);
                zi = MF<T>::mma(d.i, br, zi);
            }
            wave_lds_sync();
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                aL[v] = cx<T>{zr[v], -zi[v]};
                if (i1 < m)
                    row1[MF<T>::row(kr, v)] = aL[v];
            }
            wave_lds_sync();
            // L_10 L_10^H, to be subtracted from A_11, in the layout of
            // tile_chol: the lane's entries of L_10 are both operands
            tile_load<T>(sL, 1, m, t);
            d4v pr = {0, 0, 0, 0}, pi = {0, 0, 0, 0};
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const cx<double> x = sizeof(T) == 8 ? cvt<double>(aL[v])
                                                    : (i1 < m ? cvt<double>(row1[kr + 4 * v]) : czero<double>());
                pr = MF<double>::mma(x.r, x.r, pr);
                pi = MF<double>::mma(x.r, x.i, pi);
                pr = MF<double>::mma(x.i, x.i, pr);
                pi = MF<double>::mma(-x.i, x.r, pi);
            }
            fail |= tile_chol<T>(t, pr, pi, L, e, m - 16);
            tile_store<T>(sL, 1, m, e);
            wave_lds_sync();
            tile_operand<T, false>(sL, 1, m, aD[1]);
        }
        if (sp == 0 && lane == 0 && fail)
            atomicMin(&flags[s.sys], fail_key(s.level, s.ob0 + s.obs * p));
    } else {
        packed_load<T, MT>(sL, Lg, m);
        if (sp < nst)
            CRS_LOAD_STRIP(sp, gn);
#pragma unroll
        for (int I = 0; I < S; ++I)
            tile_operand<T, false>(sL, I, m, aD[I]);
    }
    if constexpr (S == 2) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const cx<T> x = row1[MF<T>::row(kr, v)];
            aL[v] = i1 < m ? x : czero<T>();
        }
    }

#pragma unroll 1
    for (int st = sp; st < nst; st += nsplit) {
        cx<T> g[S][4];
#pragma unroll
        for (int I = 0; I < S; ++I)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                g[I][v] = gn[I][v];
        // the next strip (the current one again after the last): issued in
        // every pass, so the wait for this strip's loads does not wait for it
        CRS_LOAD_STRIP(st + nsplit < nst ? st + nsplit : st, gn);
        // X_0 = D_0 G_0 (3M products, combined before they chain on)
        v4 x0r, x0i;
        {
            Acc3<T, 1, 1> p;
            p.zero();
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const cx<T> a = aD[0][v], b = g[0][v];
                p.t1[0][0] = MF<T>::mma(a.r, b.r, p.t1[0][0]);
                p.t2[0][0] = MF<T>::mma(a.i, b.i, p.t2[0][0]);
                p.t3[0][0] = MF<T>::mma(a.r + a.i, b.r + b.i, p.t3[0][0]);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                x0r[v] = p.re(0, 0, v);
                x0i[v] = p.im(0, 0, v);
            }
        }
        v4 x1r = {0, 0, 0, 0}, x1i = {0, 0, 0, 0};
        if (S == 2) {
            // T = L_10 X_0, then X_1 = D_1 (G_1 - T)
            Acc3<T, 1, 1> p;
            p.zero();
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const cx<T> a = aL[v];
                p.t1[0][0] = MF<T>::mma(a.r, x0r[v], p.t1[0][0]);
                p.t2[0][0] = MF<T>::mma(a.i, x0i[v], p.t2[0][0]);
                p.t3[0][0] = MF<T>::mma(a.r + a.i, x0r[v] + x0i[v], p.t3[0][0]);
            }
            Acc3<T, 1, 1> q;
            q.zero();
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const cx<T> a = aD[S - 1][v];
                const T br = g[S - 1][v].r - p.re(0, 0, v), bi = g[S - 1][v].i - p.im(0, 0, v);
                q.t1[0][0] = MF<T>::mma(a.r, br, q.t1[0][0]);
                q.t2[0][0] = MF<T>::mma(a.i, bi, q.t2[0][0]);
                q.t3[0][0] = MF<T>::mma(a.r + a.i, br + bi, q.t3[0][0]);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                x1r[v] = q.re(0, 0, v);
                x1i[v] = q.im(0, 0, v);
            }
        }
        const int src = st < nP ? 0 : (st < nP + nQ ? 1 : 2);
        const int c = 16 * (src == 0 ? st : (src == 1 ? st - nP : st - nP - nQ)) + cc;
        const int ld = src == 2 ? k : m;
        cx<T>* out = src == 0 ? W + s.oP + t * mm : (src == 1 ? W + s.oQ + t * mm : W + s.og + t * mk);
        if (c < ld) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r0 = MF<T>::row(kr, v);
                if (r0 < m)
                    out[r0 * ld + c] = cx<T>{x0r[v], x0i[v]};
                if (S == 2 && 16 + r0 < m)
                    out[(16 + r0) * ld + c] = cx<T>{x1r[v], x1i[v]};
            }
        }
    }
    // the factor last: no load waits behind these stores
    if (with_mat && sp == 0)
        for (int e = lane; e < m * (m + 1) / 2; e += 64)
            Lg[e] = sL[e];
}

#undef CRS_LOAD_STRIP

// --------------------------------------------------------------- k_reduce_m

// MFMA operand tile: 16 columns [c0, c0 + 16) of a row-major matrix with
// kd rows, loaded once in the lane layout shared by the A and B operands
// (lane l holds rows 4 s + l / 16, column c0 + l % 16, s < KS).
template <class T, int KS>
struct OpTile {
    cx<T> v[KS];
    __device__ __forceinline__ void load(const cx<T>* __restrict__ X, int ld, int ncol, int c0,
                                         int kd)
    {
        const int lane = threadIdx.x & 63, kr = lane >> 4, cc = lane & 15;
        const bool ok = c0 + cc < ncol;
        const cx<T>* b = X + (kr * ld + c0 + cc);
#pragma unroll
        for (int s = 0; s < KS; ++s)
            v[s] = (ok && 4 * s + kr < kd) ? b[4 * s * ld] : czero<T>();
    }
    __device__ __forceinline__ void zero()
    {
#pragma unroll
        for (int s = 0; s < KS; ++s)
            v[s] = czero<T>();
    }
};

// acc += A^H B for operand tiles A (rows of the result) and B (columns) in the
// 3M form.
template <class T, int KS>
__device__ __forceinline__ void mma_hn3(Acc3<T, 1, 1>& acc, const OpTile<T, KS>& A,
                                        const OpTile<T, KS>& B)
{
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const T ar = A.v[s].r, ai = -A.v[s].i, br = B.v[s].r, bi = B.v[s].i;
        acc.t1[0][0] = MF<T>::mma(ar, br, acc.t1[0][0]);
        acc.t2[0][0] = MF<T>::mma(ai, bi, acc.t2[0][0]);
        acc.t3[0][0] = MF<T>::mma(ar + ai, br + bi, acc.t3[0][0]);
    }
}

// Reduced system for a kept block q with eliminated neighbours l, r:
//   A'_q = A_q - P_l^H P_l - Q_r^H Q_r,  B'_q = -P_r^H Q_r,
//   y'_q = y_q - P_l^H g_l - Q_r^H g_r.
// Each 16-column operand tile is loaded from memory once and reused by every
// output tile that needs it (NT16 = MT / 16 tiles per m x m operand).
template <class T, int MT, class EI = cx<T>>
__global__ __launch_bounds__(64, 2) void k_reduce_m(const Seg* __restrict__ segs, int nseg,
                                                    int64_t total, const EI* __restrict__ inA,
                                                    const EI* __restrict__ iny,
                                                    cx<T>* __restrict__ W,
                                                    const unsigned long long* __restrict__ flags,
                                                    int with_mat, int with_rhs)
{
    static_assert(MT == 16 || MT == 32, "one or two operand tiles");
    using v4 = typename MF<T>::v4;
    using Tile = OpTile<T, MT / 4>;
    constexpr int NT16 = MT / 16, NV = NT16 * (NT16 + 1) / 2;
    const int lane = threadIdx.x, kr = lane >> 4, cc = lane & 15;
    const int64_t w = blockIdx.x;
    if (w >= total)
        return;
    const Seg& s = segs[find_seg(segs, nseg, w)];
    const int64_t t = w - s.w0;
    const int q = s.k0 + (int)t * s.ks;
    const int m = s.m, k = s.k, d = s.d, n = s.n;
    const int l = q - d, r = q + d;
    const bool hasL = l >= 0, hasR = r < n;
    const int64_t tl = hasL ? (l - s.e0) / s.es : 0, tr = hasR ? (r - s.e0) / s.es : 0;
    const int64_t oi = s.out_by_pos ? q : t;
    const int64_t mm = (int64_t)m * m, mk = (int64_t)m * k;
    if ((flags[s.sys] >> 40) <= (unsigned long long)s.level)
        return;
    const cx<T>* Pl = W + s.oP + tl * mm;
    const cx<T>* Qr = W + s.oQ + tr * mm;
    const cx<T>* Pr = W + s.oP + tr * mm;
    const cx<T>* gl = W + s.og + tl * mk;
    const cx<T>* gr = W + s.og + tr * mk;
    const v4 z4 = {0, 0, 0, 0};

    // right-hand side columns beyond the first 16 are handled in later chunks
    const int kc0 = with_rhs ? (k < 16 ? k : 16) : 0;
    Tile X[NT16], G;
    Acc3<T, 1, 1> av[NV], ay[NT16];
#pragma unroll
    for (int i = 0; i < NV; ++i)
        av[i].zero();
#pragma unroll
    for (int i = 0; i < NT16; ++i)
        ay[i].zero();

    // phase 1: P_l^H P_l and P_l^H g_l;  phase 2: Q_r^H Q_r and Q_r^H g_r
#pragma unroll
    for (int ph = 0; ph < 2; ++ph) {
        const bool on = ph == 0 ? hasL : hasR;
        if (!on)
            continue;
        const cx<T>* Xm = ph == 0 ? Pl : Qr;
        const cx<T>* Gm = ph == 0 ? gl : gr;
#pragma unroll
        for (int i = 0; i < NT16; ++i)
            X[i].load(Xm, m, m, 16 * i, m);
        if (kc0)
            G.load(Gm, k, kc0, 0, m);
        if (with_mat) {
#pragma unroll
            for (int i = 0, v = 0; i < NT16; ++i)
#pragma unroll
                for (int j = 0; j <= i; ++j, ++v)
                    mma_hn3<T, MT / 4>(av[v], X[i], X[j]);
        }
        if (kc0) {
#pragma unroll
            for (int i = 0; i < NT16; ++i)
                mma_hn3<T, MT / 4>(ay[i], X[i], G);
        }
    }
    // the epilogues load the four A_q or y_q elements of a tile together, in
    // every lane (element 0 stands in), before their stores: one round trip
    // per tile instead of one per element waiting behind the previous store
    if (with_mat) {
        const EI* Aq = inA + s.oA + q * mm;
        cx<T>* Vo = W + s.oAo + oi * mm;
#pragma unroll
        for (int i = 0, v = 0; i < NT16; ++i)
#pragma unroll
            for (int j = 0; j <= i; ++j, ++v) {
                cx<T> xa[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int a = 16 * i + MF<T>::row(kr, u), b = 16 * j + cc;
                    xa[u] = cvt<T>(Aq[(a < m && b <= a) ? a * m + b : 0]);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int a = 16 * i + MF<T>::row(kr, u), b = 16 * j + cc;
                    if (a < m && b <= a) {
                        cx<T> o{xa[u].r - av[v].re(0, 0, u), xa[u].i - av[v].im(0, 0, u)};
                        if (a == b)
                            o.i = T(0);
                        Vo[a * m + b] = o;
                    }
                }
            }
    }
    if (kc0) {
        const EI* yq = iny + s.oy + q * mk;
        cx<T>* yo = W + s.oyo + oi * mk;
#pragma unroll
        for (int i = 0; i < NT16; ++i) {
            cx<T> xy[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int a = 16 * i + MF<T>::row(kr, u), c = cc;
                xy[u] = cvt<T>(yq[(a < m && c < kc0) ? a * k + c : 0]);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int a = 16 * i + MF<T>::row(kr, u), c = cc;
                if (a < m && c < kc0)
                    yo[a * k + c] = cx<T>{xy[u].r - ay[i].re(0, 0, u), xy[u].i - ay[i].im(0, 0, u)};
            }
        }
    }
    // phase 3: B'_q = -P_r^H Q_r (Q_r tiles are still in X when hasR)
    if (with_mat && hasR && r + d < n) {
        Tile Pt[NT16];
#pragma unroll
        for (int i = 0; i < NT16; ++i)
            Pt[i].load(Pr, m, m, 16 * i, m);
        cx<T>* Fo = W + s.oBo + oi * mm;
#pragma unroll
        for (int i = 0; i < NT16; ++i)
#pragma unroll
            for (int j = 0; j < NT16; ++j) {
                Acc3<T, 1, 1> af;
                af.zero();
                mma_hn3<T, MT / 4>(af, Pt[i], X[j]);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int a = 16 * i + MF<T>::row(kr, u), b = 16 * j + cc;
                    if (a < m && b < m)
                        Fo[a * m + b] = cx<T>{-af.re(0, 0, u), -af.im(0, 0, u)};
                }
            }
    }
    // remaining right-hand-side chunks (k > 16)
    if (with_rhs && k > 16) {
        const EI* yq = iny + s.oy + q * mk;
        cx<T>* yo = W + s.oyo + oi * mk;
        for (int c0 = 16; c0 < k; c0 += 16) {
#pragma unroll
            for (int i = 0; i < NT16; ++i) {
                Acc3<T, 1, 1> ac;
                ac.zero();
                if (hasL) {
                    Tile A1, G1;
                    A1.load(Pl, m, m, 16 * i, m);
                    G1.load(gl, k, k, c0, m);
                    mma_hn3<T, MT / 4>(ac, A1, G1);
                }
                if (hasR) {
                    Tile A1, G1;
                    A1.load(Qr, m, m, 16 * i, m);
                    G1.load(gr, k, k, c0, m);
                    mma_hn3<T, MT / 4>(ac, A1, G1);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int a = 16 * i + MF<T>::row(kr, u), c = c0 + cc;
                    if (a < m && c < k) {
                        const cx<T> x = cvt<T>(yq[a * k + c]);
                        yo[a * k + c] = cx<T>{x.r - ac.re(0, 0, u), x.i - ac.im(0, 0, u)};
                    }
                }
            }
        }
    }
}

// --------------------------------------------------------------- k_reduce_t

template <class T, int MT, class EI = cx<T>>
__global__ __launch_bounds__(64, (MT >= 64 ? 2 : 4)) void k_reduce_t(const Seg* __restrict__ segs, int nseg,
                                                 int64_t total, const EI* __restrict__ inA,
                                                 const EI* __restrict__ iny,
                                                 cx<T>* __restrict__ W,
                                                 const unsigned long long* __restrict__ flags,
                                                 int with_mat, int with_rhs)
{
    using v4 = typename MF<T>::v4;
    constexpr int NT16 = MT / 16, KS = MT / 4;
    const int lane = threadIdx.x, kr = lane >> 4, cc = lane & 15;

    {
        const int64_t w = blockIdx.x;
        if (w >= total)
            return;
        const Seg& s = segs[find_seg(segs, nseg, w)];
        const int64_t t = w - s.w0;
        const int q = s.k0 + (int)t * s.ks;
        const int m = s.m, k = s.k, d = s.d, n = s.n;
        const int l = q - d, r = q + d;
        const bool hasL = l >= 0, hasR = r < n;
        const int64_t tl = hasL ? (l - s.e0) / s.es : 0, tr = hasR ? (r - s.e0) / s.es : 0;
        const int64_t oi = s.out_by_pos ? q : t;
        const int64_t mm = (int64_t)m * m, mk = (int64_t)m * k;
        if ((flags[s.sys] >> 40) <= (unsigned long long)s.level)
            return;
        const cx<T>* Pl = W + s.oP + tl * mm;
        const cx<T>* Qr = W + s.oQ + tr * mm;
        const cx<T>* Pr = W + s.oP + tr * mm;
        if (with_mat) {
            const EI* Aq = inA + s.oA + q * mm;
            cx<T>* Vo = W + s.oAo + oi * mm;
#pragma unroll 1
            for (int ti = 0; ti < NT16; ++ti) {
                if (16 * ti >= m)
                    break;
#pragma unroll 1
                for (int tj = 0; tj <= ti; ++tj) {
                    v4 cr = {0, 0, 0, 0}, ci = {0, 0, 0, 0};
                    if (hasL)
                        tile_hn<T, KS>(cr, ci, Pl, m, m, 16 * ti, Pl, m, m, 16 * tj, m);
                    if (hasR)
                        tile_hn<T, KS>(cr, ci, Qr, m, m, 16 * ti, Qr, m, m, 16 * tj, m);
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int i = 16 * ti + MF<T>::row(kr, v), j = 16 * tj + cc;
                        if (i < m && j <= i) {
                            const cx<T> a = cvt<T>(Aq[i * m + j]);
                            cx<T> o{a.r - cr[v], a.i - ci[v]};
                            if (i == j)
                                o.i = T(0);
                            Vo[i * m + j] = o;
                        }
                    }
                }
            }
            if (hasR && r + d < n) {
                cx<T>* Fo = W + s.oBo + oi * mm;
    #pragma unroll 1
            for (int ti = 0; ti < NT16; ++ti) {
                    if (16 * ti >= m)
                        break;
#pragma unroll 1
                    for (int tj = 0; tj < NT16; ++tj) {
                        if (16 * tj >= m)
                            break;
                        v4 cr = {0, 0, 0, 0}, ci = {0, 0, 0, 0};
                        tile_hn<T, KS>(cr, ci, Pr, m, m, 16 * ti, Qr, m, m, 16 * tj, m);
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const int i = 16 * ti + MF<T>::row(kr, v), j = 16 * tj + cc;
                            if (i < m && j < m)
                                Fo[i * m + j] = cx<T>{-cr[v], -ci[v]};
                        }
                    }
                }
            }
        }
        if (with_rhs) {
            const cx<T>* gl = W + s.og + tl * mk;
            const cx<T>* gr = W + s.og + tr * mk;
            const EI* yq = iny + s.oy + q * mk;
            cx<T>* vo = W + s.oyo + oi * mk;
#pragma unroll 1
            for (int ti = 0; ti < NT16; ++ti) {
                if (16 * ti >= m)
                    break;
#pragma unroll 1
                for (int c0 = 0; c0 < k; c0 += 16) {
                    v4 cr = {0, 0, 0, 0}, ci = {0, 0, 0, 0};
                    if (hasL)
                        tile_hn<T, KS>(cr, ci, Pl, m, m, 16 * ti, gl, k, k, c0, m);
                    if (hasR)
                        tile_hn<T, KS>(cr, ci, Qr, m, m, 16 * ti, gr, k, k, c0, m);
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int i = 16 * ti + MF<T>::row(kr, v), c = c0 + cc;
                        if (i < m && c < k) {
                            const cx<T> a = cvt<T>(yq[i * k + c]);
                            vo[i * k + c] = cx<T>{a.r - cr[v], a.i - ci[v]};
                        }
                    }
                }
            }
        }
    }
}

// ---------------------------------------------------------------- k_back_mf

// Back substitution for block sizes 8 < m <= 32 on MFMA: per 16-column strip
// of x_p, w = g - Q x_{p-d} - P x_{p+d} stays in the accumulators and the
// block upper triangular L^H x = w is solved tile by tile,
// x_1 = D_1^H w_1, x_0 = D_0^H (w_0 - L_10^H x_1), with the products chained
// through the accumulators as in k_elim_mf (D_I = L_II^{-1} is stored in L_II's
// place).
template <class T, int MT>
__global__ __launch_bounds__(64, 2) void k_back_mf(const Seg* __restrict__ segs, int nseg,
                                                   int64_t total, const cx<T>* __restrict__ W,
                                                   cx<T>* __restrict__ X,
                                                   const unsigned long long* __restrict__ flags,
                                                   cx<double>* __restrict__ U, int upd)
{
    static_assert(MT == 16 || MT == 32, "one or two 16-row tiles");
    using v4 = typename MF<T>::v4;
    constexpr int S = MT / 16, KS = MT / 4;
    constexpr int NP = MT * (MT + 1) / 2;
    __shared__ cx<T> sL[NP]; // the packed factor
    const int lane = threadIdx.x, kr = lane >> 4, cc = lane & 15;
    const int64_t w = blockIdx.x;
    if (w >= total)
        return;
    const Seg& s = segs[find_seg(segs, nseg, w)];
    const int64_t t = w - s.w0;
    const int p = s.e0 + (int)t * s.es;
    const int m = s.m, k = s.k, d = s.d;
    const bool hasPrev = p - d >= 0, hasNext = p + d < s.n;
    const int64_t mm = (int64_t)m * m, mk = (int64_t)m * k;
    cx<T>* xp = X + s.ox + (s.xo + s.xs * p) * mk;
    cx<double>* up = upd ? U + s.oU + p * mk : nullptr;
    if (flags[s.sys] != kNoFail) {
        const T nan = T(NAN);
        for (int e = lane; e < m * k; e += 64) {
            put_x<T>(xp, up, upd ? 1 : 0, e, cx<T>{nan, nan});
            if (upd && hasNext)
                put_x<T>(xp, up + d * mk, 1, e, cx<T>{nan, nan});
        }
        return;
    }
    const cx<T>* xm = X + s.ox + (s.xo + s.xs * (p - d)) * mk;
    const cx<T>* xn = X + s.ox + (s.xo + s.xs * (p + d)) * mk;
    if (upd && hasNext)
        put_kept<T>(xn, up + d * mk, upd, lane, mk, 64);
    const cx<T>* L = W + s.oL + t * mm;
    const cx<T>* P = W + s.oP + t * mm;
    const cx<T>* Q = W + s.oQ + t * mm;
    const cx<T>* g = W + s.og + t * mk;
    packed_load<T, MT>(sL, L, m);
    // left operands (L_10^H)[i][u] = conj(L[16 + u][i]) and D_I^H
    cx<T> aLh[4], aDh[S][4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int u = 16 + MF<T>::row(kr, v);
        const cx<T> a = (S == 2 && u < m) ? sL[u * (u + 1) / 2 + cc] : czero<T>();
        aLh[v] = cx<T>{a.r, -a.i};
    }
#pragma unroll
    for (int I = 0; I < S; ++I)
        tile_operand<T, true>(sL, I, m, aDh[I]);
#pragma unroll 1
    for (int c0 = 0; c0 < k; c0 += 16) {
        const int cw = min(16, k - c0);
        // w_I = g_I - Q_I x_{p-d} - P_I x_{p+d} in the accumulator layout
        T wr[S][4], wi[S][4];
#pragma unroll
        for (int I = 0; I < S; ++I) {
            Acc3<T, 1, 1> acc;
            acc.zero();
            if (hasPrev)
                tile_nn3<T, KS>(acc, Q, m, m, 16 * I, xm + c0, k, cw, 0, m);
            if (hasNext)
                tile_nn3<T, KS>(acc, P, m, m, 16 * I, xn + c0, k, cw, 0, m);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = 16 * I + MF<T>::row(kr, v);
                const cx<T> gv = (r < m && cc < cw) ? g[r * k + c0 + cc] : czero<T>();
                wr[I][v] = gv.r - acc.re(0, 0, v);
                wi[I][v] = gv.i - acc.im(0, 0, v);
            }
        }
        // bottom tile first: x_{S-1} = D_{S-1}^H w_{S-1}
        v4 x1r = {0, 0, 0, 0}, x1i = {0, 0, 0, 0};
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const cx<T> a = aDh[S - 1][v];
            x1r = MF<T>::mma(a.r, wr[S - 1][v], x1r);
            x1r = MF<T>::mma(-a.i, wi[S - 1][v], x1r);
            x1i = MF<T>::mma(a.r, wi[S - 1][v], x1i);
            x1i = MF<T>::mma(a.i, wr[S - 1][v], x1i);
        }
        v4 x0r = x1r, x0i = x1i;
        if (S == 2) {
            // w_0 -= L_10^H x_1, x_0 = D_0^H w_0
            v4 tr = {0, 0, 0, 0}, ti = {0, 0, 0, 0};
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const cx<T> a = aLh[v];
                tr = MF<T>::mma(a.r, x1r[v], tr);
                tr = MF<T>::mma(-a.i, x1i[v], tr);
                ti = MF<T>::mma(a.r, x1i[v], ti);
                ti = MF<T>::mma(a.i, x1r[v], ti);
            }
            x0r = v4{0, 0, 0, 0};
            x0i = v4{0, 0, 0, 0};
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const cx<T> a = aDh[0][v];
                const T br = wr[0][v] - tr[v], bi = wi[0][v] - ti[v];
                x0r = MF<T>::mma(a.r, br, x0r);
                x0r = MF<T>::mma(-a.i, bi, x0r);
                x0i = MF<T>::mma(a.r, bi, x0i);
                x0i = MF<T>::mma(a.i, br, x0i);
            }
        }
        if (cc < cw) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r0 = MF<T>::row(kr, v);
                if (r0 < m)
                    put_x<T>(xp, up, upd, r0 * k + c0 + cc, cx<T>{x0r[v], x0i[v]});
                if (S == 2 && 16 + r0 < m)
                    put_x<T>(xp, up, upd, (16 + r0) * k + c0 + cc, cx<T>{x1r[v], x1i[v]});
            }
        }
    }
}

} // namespace crs
