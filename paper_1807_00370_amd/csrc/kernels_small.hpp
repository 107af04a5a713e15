// Kernels of a reduction level for block sizes up to 8: several blocks share a
// wave, so that a level costs what its bytes cost (a block of m = 8 is 1 KiB
// per matrix; a work-group of 256 lanes per block left most of them idle).
//
//   k_elim_s    one column of [A_p | B_p^H | B_{p-d} | y_p] per lane, MT lanes
//               per operand: 2 blocks per wave for MT = 8, 4 for MT = 4.  The
//               elimination that factors A_p is applied to every column.
//   k_reduce_s  the products of a kept block as one 16 x 16 MFMA tile
//               [Q_r | P_r]^H [Q_r | g_r] + [P_l | 0]^H [P_l | g_l]: A', B'
//               and y' together (two blocks side by side for MT = 4).
//   k_back_s    one row of an eliminated block per lane, 64 / MT blocks (or
//               right-hand-side columns of a block) per wave.
//
// Launches of few waves deal a block's columns of y over 2^ss waves (2^cs lane
// groups in k_back_s); in the elimination with the matrix each of them factors
// the block and wave 0 alone stores the factor, P, Q and the first columns.
//
// Rows and columns from m to MT are padded with the identity (A) or zero.
//
// All three are bound by HBM at levels with many blocks and by the latency of
// their loads below.  Measured against the kernels they replaced (one wave per
// block in the elimination, a work-group of 256 per block in the others),
// N = 131071, m = 8, k = 1, FP64 complex, level 0 / all levels of a solve, us:
//   elimination        141 -> 91 / 376 -> 279   (390 MB: 4.3 TB/s)
//   reduction          390 -> 74 / 813 -> 220   (340 MB: 4.6 TB/s)
//   back substitution  374 -> 48 / 739 -> 134   (183 MB: 3.8 TB/s)
// and N = 64, m = 4, k = 1: 87 -> 57 us of kernels.  The elimination of FP64
// complex blocks of 5..8 keeps 6 registers in scratch (28 bytes a lane).
#pragma once

#include "kernels_fast.hpp"

namespace crs {

// ok ? a : b by component (a choice between two array elements would choose
// between their addresses and put the arrays into scratch memory).
template <class T>
__device__ __forceinline__ cx<T> pick(bool ok, const cx<T> a, const cx<T> b)
{
    return cx<T>{ok ? a.r : b.r, ok ? a.i : b.i};
}

// Value of x in lane R of each group of MT lanes (MT = 4 or 8).
template <int MT, int R>
__device__ __forceinline__ int group_bcast(int x)
{
    if constexpr (MT == 4)
        return __builtin_amdgcn_update_dpp(x, x, 0x55 * R, 0xf, 0xf, true); // quad permute
    const int lo = __builtin_amdgcn_update_dpp(x, x, 0x150 + R, 0xf, 0x3, false);
    return __builtin_amdgcn_update_dpp(lo, x, 0x158 + R, 0xf, 0xc, false);
}
template <int MT, int R>
__device__ __forceinline__ float group_bcast(float x)
{
    return __int_as_float(group_bcast<MT, R>(__float_as_int(x)));
}
template <int MT, int R>
__device__ __forceinline__ double group_bcast(double x)
{
    const long long v = __double_as_longlong(x);
    const unsigned lo = (unsigned)group_bcast<MT, R>((int)v);
    const unsigned hi = (unsigned)group_bcast<MT, R>((int)(v >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// ----------------------------------------------------------------- k_elim_s

// The elimination from step C on of one column x (rows C..MT-1), with column C
// of L in l (diagonal {L_CC, 1 / L_CC}); the next column of L is read a step
// ahead, and no earlier (registers).
template <class T, int MT, int C>
__device__ __forceinline__ void col_solve(cx<T> (&x)[MT], const cx<T>* sL, const cx<T> (&l)[MT])
{
    cx<T> ln[MT];
#pragma unroll
    for (int r = 0; r < MT; ++r)
        ln[r] = C + 1 < MT && r > C ? sL[(C + 1) * MT + r] : czero<T>();
    const T inv = l[C].i;
    x[C] = cx<T>{x[C].r * inv, x[C].i * inv};
#pragma unroll
    for (int r = C + 1; r < MT; ++r)
        msub(x[r], l[r], x[C]);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (C + 1 < MT)
        col_solve<T, MT, C + 1>(x, sL, ln);
}
template <class T, int MT>
__device__ __forceinline__ void col_solve(cx<T> (&x)[MT], const cx<T>* sL)
{
    cx<T> l[MT];
#pragma unroll
    for (int r = 0; r < MT; ++r)
        l[r] = sL[r];
    col_solve<T, MT, 0>(x, sL, l);
}

// Column C of the factorization: lane j = C of the A part owns it (rows
// C..MT-1 of its x, unscaled); it publishes the scaled column in LDS and
// every column right of it, of every operand, takes the step.  own: this
// lane's column of A is done (its x keeps the unscaled column, iv its inverse
// pivot).
template <class T, int MT, int C>
__device__ __forceinline__ void factor_steps(cx<T> (&x)[MT], cx<T>* sL, T& iv, bool inA, int j,
                                             int m, bool& fail)
{
    if constexpr (C < MT) {
        const T d = x[C].r;
        const T inv = rsqrt_nr(d);
        cx<T>* col = sL + C * MT;
        if (inA && j == C) {
            col[C] = cx<T>{d * inv, inv};
#pragma unroll
            for (int r = C + 1; r < MT; ++r)
                col[r] = cx<T>{x[r].r * inv, x[r].i * inv};
            iv = inv;
            fail = C < m && !(d > T(0));
        }
        wave_lds_sync();
        cx<T> l[MT];
#pragma unroll
        for (int r = C; r < MT; ++r)
            l[r] = col[r];
        __builtin_amdgcn_sched_barrier(0); // one column of L in registers at a time
        const bool act = !inA || j > C;
        const T s = act ? l[C].i : T(1);
        x[C] = cx<T>{x[C].r * s, x[C].i * s};
        const cx<T> f = pick(act, x[C], czero<T>());
#pragma unroll
        for (int r = C + 1; r < MT; ++r)
            msub(x[r], l[r], f);
        factor_steps<T, MT, C + 1>(x, sL, iv, inA, j, m, fail);
    }
}

// MAT: with the matrix (and the first MT columns of y_p); else the columns of
// y_p against the stored factor.  That form is an instance of its own: it
// needs 191 registers for FP64, MT = 8, where both in one kernel spilled at any
// bound that the matrix pass runs well with (N = 131071, m = 8, k = 1, stored
// factors 740 -> 458 us).
template <class T, int MT, bool MAT, class EI = cx<T>>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MAT ? 3 : 2, 8))) void k_elim_s(const Seg* __restrict__ segs, int nseg, int64_t total, int ss,
                                                const EI* __restrict__ inA, const EI* __restrict__ inB,
                                                const EI* __restrict__ iny, cx<T>* __restrict__ W,
                                                unsigned long long* __restrict__ flags, int with_rhs)
{
    constexpr int LB = 4 * MT, NB = 64 / LB; // lanes per block, blocks per wave
    constexpr int LT = MT + 1;
    // a block's A_p and B_p for the transposition, then its factor
    __shared__ cx<T> sAll[4][NB][MAT ? 2 * MT * LT : MT * MT];
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int blk = lane / LB, cl = lane % LB, part = cl / MT, j = cl % MT;
    const int64_t wi = (int64_t)blockIdx.x * (blockDim.x >> 6) + wv;
    const int nsplit = 1 << ss, sp = (int)wi & (nsplit - 1); // waves per block, this one
    const int64_t w = (wi >> ss) * NB + blk;
    bool live = w < total;
    const Seg& s = segs[find_seg(segs, nseg, live ? w : 0)];
    const int64_t t = live ? w - s.w0 : 0;
    const int p = s.e0 + (int)t * s.es;
    const int m = s.m, k = s.k, d = s.d;
    const int mm = m * m, mk = m * k;
    const bool hasPrev = p - d >= 0, hasNext = p + d < s.n;
    // a system that broke down at an earlier level stores nothing (the loads
    // do not wait for its flag)
    const bool in = live;
    live = live && (flags[s.sys] >> 40) >= (unsigned long long)s.level;
    cx<T>* Lg = W + s.oL + t * mm;
    cx<T>* sL = sAll[wv][blk];
    const EI* yp = iny + s.oy + (int64_t)p * mk;
    cx<T>* gp = W + s.og + t * mk;
    // the columns of y_p beyond those that a matrix pass takes along, one per
    // lane of the block
    const int c0 = (MAT ? MT : 0) + sp * LB + cl, kc = with_rhs ? k : 0;
    cx<T> yc[MT];
    auto load_col = [&](int c) {
#pragma unroll
        for (int r = 0; r < MT; ++r) {
            const bool ok = c < kc && r < m;
            const cx<T> v = cvt<T>(yp[ok ? r * k + c : 0]);
            yc[r] = pick(ok, v, czero<T>());
        }
    };
    if constexpr (MAT) {
        // element r of the lane's column: A_p's (from the lower triangle),
        // B_p^H's, B_{p-d}'s or y_p's.  Every lane loads down its column of
        // the stored block, so that a load covers MT consecutive elements of
        // each block; what has to be read along rows (A_p above the diagonal,
        // B_p^H) crosses through LDS.
        const EI* Ap = inA + s.oA + (int64_t)p * mm;
        const EI* src = part == 0 ? Ap
                                  : part == 3 ? yp : inB + s.oB + (int64_t)(part == 1 ? p : p - d) * mm;
        const bool on = in && j < (part == 3 ? k : m) &&
                        (part == 0 || (sp == 0 && (part == 1 ? hasNext : part == 2 ? hasPrev : with_rhs != 0)));
        const int ld = part == 3 ? k : m;
        EI in[MT];
#pragma unroll
        for (int r = 0; r < MT; ++r)
            in[r] = (on && r < m ? src : Ap)[on && r < m ? r * ld + j : 0];
        cx<T> x[MT];
#pragma unroll
        for (int r = 0; r < MT; ++r) {
            const cx<T> v = cvt<T>(in[r]);
            x[r] = pick(on && r < m, v, czero<T>());
        }
        cx<T>* st = sL + (part & 1) * MT * LT;
        if (part < 2) {
#pragma unroll
            for (int r = 0; r < MT; ++r)
                st[r * LT + j] = x[r];
        }
        wave_lds_sync();
#pragma unroll
        for (int r = 0; r < MT; ++r) {
            const cx<T> v = st[j * LT + r];
            if (part == 1 || (part == 0 && r < j))
                x[r] = cx<T>{v.r, -v.i};
            if (part == 0 && r == j)
                x[r] = cx<T>{on ? x[r].r : T(1), T(0)};
        }
        wave_lds_sync();
        T iv = T(1);
        bool fail = false;
        factor_steps<T, MT, 0>(x, sL, iv, part == 0, j, m, fail);
        if (fail && live && sp == 0)
            atomicMin(&flags[s.sys], fail_key(s.level, s.ob0 + s.obs * p));
        if (on && live && sp == 0) {
            if (part == 0) {
                // packed lower triangle, the inverse pivot in the imaginary
                // slot of the diagonal
#pragma unroll
                for (int r = 0; r < MT; ++r)
                    if (r >= j && r < m)
                        Lg[r * (r + 1) / 2 + j] = cx<T>{x[r].r * iv, r == j ? iv : x[r].i * iv};
            } else {
                cx<T>* out = part == 3 ? gp : W + (part == 1 ? s.oP : s.oQ) + t * mm;
#pragma unroll
                for (int r = 0; r < MT; ++r)
                    if (r < m)
                        out[r * ld + j] = x[r];
            }
        }
    } else {
        // the packed factor, dealt over the block's lanes, into columns (lanes
        // past the end move the last element); what the padded rows and
        // columns hold reaches no stored row
        constexpr int NE = (MT * (MT + 1) / 2 + LB - 1) / LB;
        const int np = m * (m + 1) / 2;
        cx<T> l[NE];
#pragma unroll
        for (int q = 0; q < NE; ++q)
            l[q] = Lg[min(cl + LB * q, np - 1)];
        load_col(c0); // beside L
#pragma unroll
        for (int q = 0; q < NE; ++q) {
            const int e = min(cl + LB * q, np - 1), r = tri_row(e);
            sL[(e - r * (r + 1) / 2) * MT + r] = l[q];
        }
        wave_lds_sync();
    }
    for (int c = c0; live && c < kc; c += LB * nsplit) {
        if (MAT || c > c0)
            load_col(c);
        col_solve<T, MT>(yc, sL);
#pragma unroll
        for (int r = 0; r < MT; ++r)
            if (r < m)
                gp[r * k + c] = yc[r];
    }
}

// --------------------------------------------------------------- k_reduce_s

// The 16 columns of the operand tile are MT columns of Q_r and MT of P_r for
// each of the NB = 8 / MT blocks; the right operand has g's first MT columns
// in P_r's place.  Accumulator entries whose row and column belong to one
// block are its A' (Q, Q), B' (P, Q) and y' (Q, g); columns of y' beyond MT
// follow in chunks of 16 / NB.  The products take the four-multiplication
// complex form.
template <class T, int MT, class EI = cx<T>>
__global__ __launch_bounds__(256) void k_reduce_s(const Seg* __restrict__ segs, int nseg,
                                                  int64_t total, int ss, const EI* __restrict__ inA,
                                                  const EI* __restrict__ iny, cx<T>* __restrict__ W,
                                                  const unsigned long long* __restrict__ flags,
                                                  int with_mat, int with_rhs)
{
    using v4 = typename MF<T>::v4;
    constexpr int NB = 8 / MT, KS = MT / 4, CW = 16 / NB;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int kr = lane >> 4, cc = lane & 15;
    const int64_t wi = (int64_t)blockIdx.x * (blockDim.x >> 6) + wv;
    const int nsplit = 1 << ss, sp = (int)wi & (nsplit - 1); // waves per block, this one
    const int64_t w = (wi >> ss) * NB + (NB == 1 ? 0 : cc / CW);
    bool live = w < total;
    const Seg& s = segs[find_seg(segs, nseg, live ? w : 0)];
    const int64_t t = live ? w - s.w0 : 0;
    const int q = s.k0 + (int)t * s.ks;
    const int m = s.m, k = s.k, d = s.d, n = s.n;
    const int l = q - d, r = q + d;
    const int64_t oi = s.out_by_pos ? q : t;
    const int mm = m * m, mk = m * k;
    // (the loads do not wait for the flag)
    const bool hasL = live && l >= 0, hasR = live && r < n, hasF = hasR && r + d < n;
    const bool in = live;
    live = live && (flags[s.sys] >> 40) > (unsigned long long)s.level;
    const int64_t tl = hasL ? (l - s.e0) / s.es : 0, tr = hasR ? (r - s.e0) / s.es : 0;
    const cx<T>* Pl = W + s.oP + tl * mm;
    const cx<T>* Qr = W + s.oQ + tr * mm;
    const cx<T>* Pr = W + s.oP + tr * mm;
    const cx<T>* gl = W + s.og + tl * mk;
    const cx<T>* gr = W + s.og + tr * mk;
    const EI* Aq = inA + s.oA + q * (int64_t)mm;
    const EI* yq = iny + s.oy + q * (int64_t)mk;
    cx<T>* Vo = W + s.oAo + oi * mm;
    cx<T>* Fo = W + s.oBo + oi * mm;
    cx<T>* yo = W + s.oyo + oi * mk;
    const bool second = (cc / MT) & 1; // P_r / g columns
    const int col = cc % MT;
    const int kc = with_rhs && sp == 0 ? min(k, MT) : 0;
    if (sp)
        with_mat = 0;
    // operands: left Q_r | P_r and P_l | 0, right Q_r | g_r and P_l | g_l
    cx<T> xr[KS], yr[KS], xl[KS], yl[KS];
#pragma unroll
    for (int u = 0; u < KS; ++u) {
        const int tt = 4 * u + kr;
        const bool okm = tt < m && col < m, okg = tt < m && col < kc;
        const cx<T> a = ld_or0((second ? Pr : Qr) + tt * m + col, W,
                               okm && (second ? hasF && with_mat : hasR));
        const cx<T> b = ld_or0(Pl + tt * m + col, W, okm && hasL && !second);
        const cx<T> gx = ld_or0(gr + tt * k + col, W, okg && hasR && second);
        const cx<T> gy = ld_or0(gl + tt * k + col, W, okg && hasL && second);
        xr[u] = a;
        yr[u] = second ? gx : a;
        xl[u] = b;
        yl[u] = second ? gy : b;
    }
    // what the results are subtracted from: A_q for (Q, Q), y_q for (Q, g)
    cx<T> base[4];
    bool put[4];
    cx<T>* dst[4];
    bool diag[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int i = MF<T>::row(kr, v), a = i % MT;
        const bool same = NB == 1 || i / CW == cc / CW, rowP = (i / MT) & 1;
        const bool isA = same && !rowP && !second && with_mat && in && a < m && col <= a;
        const bool isF = same && rowP && !second && with_mat && hasF && a < m && col < m;
        const bool isY = same && !rowP && second && in && a < m && col < kc;
        const EI* src = isA ? Aq + a * m + col : isY ? yq + a * k + col : yq;
        base[v] = cvt<T>(*(isA || isY ? src : (with_mat ? inA + s.oA : iny + s.oy)));
        if (!(isA || isY))
            base[v] = czero<T>();
        diag[v] = isA && a == col;
        put[v] = live && (isA || isF || isY);
        dst[v] = isA ? Vo + a * m + col : isF ? Fo + a * m + col : yo + a * k + col;
    }
    v4 cr = {0, 0, 0, 0}, ci = {0, 0, 0, 0};
    auto mul = [&](const cx<T> a, const cx<T> b) { // += conj(a) b
        cr = MF<T>::mma(a.r, b.r, cr);
        ci = MF<T>::mma(a.r, b.i, ci);
        cr = MF<T>::mma(a.i, b.i, cr);
        ci = MF<T>::mma(-a.i, b.r, ci);
    };
#pragma unroll
    for (int u = 0; u < KS; ++u)
        mul(xl[u], yl[u]);
#pragma unroll
    for (int u = 0; u < KS; ++u)
        mul(xr[u], yr[u]);
#pragma unroll
    for (int v = 0; v < 4; ++v)
        if (put[v])
            *dst[v] = cx<T>{base[v].r - cr[v], diag[v] ? T(0) : base[v].i - ci[v]};
    if (!with_rhs)
        return;
    // the chunks of columns beyond MT; wave 0 of several has had the matrix
    for (int c0 = MT + CW * (sp ? sp - 1 : nsplit - 1); __any(c0 < k); c0 += CW * nsplit) {
        const int c = c0 + cc % CW;
        cr = v4{0, 0, 0, 0};
        ci = v4{0, 0, 0, 0};
        cx<T> br[KS], bl[KS];
#pragma unroll
        for (int u = 0; u < KS; ++u) {
            const int tt = 4 * u + kr;
            bl[u] = ld_or0(gl + tt * k + c, W, tt < m && c < k && hasL);
            br[u] = ld_or0(gr + tt * k + c, W, tt < m && c < k && hasR);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = MF<T>::row(kr, v), a = i % MT;
            put[v] = (NB == 1 || i / CW == cc / CW) && !((i / MT) & 1) && live && a < m && c < k;
            base[v] = cvt<T>(yq[put[v] ? a * k + c : 0]);
        }
#pragma unroll
        for (int u = 0; u < KS; ++u)
            mul(xl[u], bl[u]);
#pragma unroll
        for (int u = 0; u < KS; ++u)
            mul(xr[u], br[u]);
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (put[v])
                yo[(MF<T>::row(kr, v) % MT) * k + c] = cx<T>{base[v].r - cr[v], base[v].i - ci[v]};
    }
}

// ----------------------------------------------------------------- k_back_s

// L^H x = w: row R's unknown, then its part of the rows above.
template <class T, int MT, int R>
__device__ __forceinline__ void back_steps(cx<T>& w, const cx<T> (&L)[MT], T iv, int r)
{
    if constexpr (R >= 0) {
        const cx<T> x{group_bcast<MT, R>(w.r * iv), group_bcast<MT, R>(w.i * iv)};
        cx<T> u = w;
        msub_ca(u, L[R], x); // L[R] = L_Rr
        w = pick(r < R, u, pick(r == R, x, w));
        back_steps<T, MT, R - 1>(w, L, iv, r);
    }
}

// Value of x in lane r ^ B of the group (B = 1, 2) or lane 7 - r (B = 4).
template <int B>
__device__ __forceinline__ int group_swap(int x)
{
    constexpr int ctrl = B == 1 ? 0xb1 : B == 2 ? 0x4e : 0x141; // quad permutes, half-row mirror
    return __builtin_amdgcn_update_dpp(x, x, ctrl, 0xf, 0xf, true);
}
template <int B>
__device__ __forceinline__ float group_swap(float x)
{
    return __int_as_float(group_swap<B>(__float_as_int(x)));
}
template <int B>
__device__ __forceinline__ double group_swap(double x)
{
    const long long v = __double_as_longlong(x);
    const unsigned lo = (unsigned)group_swap<B>((int)v);
    const unsigned hi = (unsigned)group_swap<B>((int)(v >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// v[u] summed over the 2 B lanes of the group, u = this lane's row: each
// step hands the half of the values whose rows lie with the other lane over
// to it and adds what comes back (the mirror pairs lane r with 7 - r, so the
// following steps within a quad meet every pair).
template <int B, class T, int N>
__device__ __forceinline__ cx<T> group_scatter(const cx<T> (&v)[N], int r)
{
    static_assert(N == 2 * B, "one value per lane");
    const bool up = r & B;
    cx<T> h[B];
#pragma unroll
    for (int u = 0; u < B; ++u) {
        const cx<T> keep = pick(up, v[u + B], v[u]), give = pick(up, v[u], v[u + B]);
        h[u] = cx<T>{keep.r + group_swap<B>(give.r), keep.i + group_swap<B>(give.i)};
    }
    if constexpr (B == 1)
        return h[0];
    else
        return group_scatter<B / 2>(h, r);
}

// Lanes: row r = lane % MT, then 2^cs right-hand-side columns, then blocks.
// A lane loads column r of Q_p and P_p (a load covers MT consecutive elements
// of each block; rows per lane would touch one line per lane and load), forms
// its column's products with x_{p-d} and x_{p+d} for all MT rows, and the
// group scatters the sums.
template <class T, int MT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 8))) void k_back_s(const Seg* __restrict__ segs, int nseg, int64_t total,
                                                int cs, const cx<T>* __restrict__ W,
                                                cx<T>* __restrict__ X,
                                                const unsigned long long* __restrict__ flags,
                                                cx<double>* __restrict__ U, int upd)
{
    const int64_t id = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / MT;
    const int r = threadIdx.x % MT, cg = (int)(id & ((1 << cs) - 1));
    const int64_t w = id >> cs;
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
    const int step = 1 << cs;
    if (flags[s.sys] != kNoFail) {
        const T nan = T(NAN);
        if (r < m)
            for (int c = cg; c < k; c += step) {
                put_x<T>(xp, up, upd ? 1 : 0, r * k + c, cx<T>{nan, nan});
                if (upd && hasNext)
                    put_x<T>(xp, up + d * mk, 1, r * k + c, cx<T>{nan, nan});
            }
        return;
    }
    const cx<T>* xm = X + s.ox + (s.xo + s.xs * (p - d)) * mk;
    const cx<T>* xn = X + s.ox + (s.xo + s.xs * (p + d)) * mk;
    if (upd && hasNext)
        put_kept<T>(xn, up + d * mk, upd, cg * MT + r, mk, MT << cs);
    const cx<T>* L = W + s.oL + t * mm;
    const cx<T>* P = W + s.oP + t * mm;
    const cx<T>* Q = W + s.oQ + t * mm;
    const cx<T>* g = W + s.og + t * mk;
    // columns r of Q, P and L (below the diagonal)
    cx<T> qc[MT], pc[MT], lc[MT];
    const bool okr = r < m;
#pragma unroll
    for (int u = 0; u < MT; ++u) {
        qc[u] = ld_or0(Q + u * m + r, W, okr && u < m && hasPrev);
        pc[u] = ld_or0(P + u * m + r, W, okr && u < m && hasNext);
        lc[u] = ld_or0(L + u * (u + 1) / 2 + r, W, u < m && r <= u);
    }
    T iv = T(1);
#pragma unroll
    for (int u = 0; u < MT; ++u)
        iv = u == r && okr ? lc[u].i : iv;
#pragma unroll 1
    for (int c = cg; c < k; c += step) {
        const cx<T> am = ld_or0(xm + r * k + c, X, okr && hasPrev);
        const cx<T> an = ld_or0(xn + r * k + c, X, okr && hasNext);
        cx<T> v = ld_or0(g + r * k + c, W, okr);
        cx<T> z[MT];
#pragma unroll
        for (int u = 0; u < MT; ++u) {
            z[u] = czero<T>();
            msub(z[u], qc[u], am);
            msub(z[u], pc[u], an);
        }
        const cx<T> z0 = group_scatter<MT / 2>(z, r);
        v = cx<T>{v.r + z0.r, v.i + z0.i};
        back_steps<T, MT, MT - 1>(v, lc, iv, r);
        if (okr)
            put_x<T>(xp, up, upd, r * k + c, v);
    }
}

} // namespace crs
