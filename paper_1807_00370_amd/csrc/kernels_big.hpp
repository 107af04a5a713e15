// Kernels of a reduction level for block sizes 32 < m <= 256 (the block 2D
// Poisson workload has m = 256).  A block no longer fits in LDS, so every
// step is cut into 16 x 16 MFMA tiles whose operands stream from L2 (the
// streaming products in the three-multiplication complex form, Acc3):
//
//   k_potrf_reg   one work-group per eliminated block, the block held in its
//                 registers: right-looking Cholesky L_p = chol(A_p) by
//                 16-column panels.  Each 16 x 16 diagonal tile is factored
//                 and inverted by one wave (tile_chol); its inverse
//                 D_I = L_II^{-1} is kept for the substitutions.
//   k_potrf_rl    the same from memory, for FP64 complex blocks above 128.
//   k_trsm_reg    one wave per (eliminated block, 16-column strip of
//                 [B_p^H | B_{p-d} | y_p]), four strips of a block per
//                 work-group: blocked forward substitution
//                 X_I = D_I (G_I - L[I][<I] X_{<I}), the Section 4 recipe
//                 L \ G for the three operands of Eq. (Formulas), the strip
//                 in registers and L staged in LDS column by column.
//   k_trsm_strip  the same, one wave per work-group with the finished rows
//                 re-read, for FP64 complex blocks above 128.
//   k_reduce_big  one wave per (kept block, 16 or 32 wide tile) of the reduced
//                 system A' = A_q - P_l^H P_l - Q_r^H Q_r (lower triangle),
//                 B' = -P_r^H Q_r, y' = y_q - P_l^H g_l - Q_r^H g_r; with
//                 16 x 16 tiles it also serves the levels of m <= 32 that
//                 hold few blocks.
//   k_reduce_lds  A' and B' for blocks above 64: one work-group of four
//                 waves per 64 x 64 tile, operand panels staged in LDS.
//   k_back_big    one work-group per (eliminated block, 16-column strip of
//                 x_p), one wave per row tile: blocked back substitution of
//                 L^H x_p = g_p - Q_p x_{p-d} - P_p x_{p+d}.
//   k_grad_big    one wave per (block row, 32 x 32 tile) of the adjoint's
//                 gradient blocks.
//
// Storage for these sizes: L_p as a full m x m row-major slot (lower
// triangle used; the diagonal holds {L_cc, 1 / L_cc} like every other
// factor) and the inverse diagonal tiles D_I (16 x 16 row-major, lower
// triangular) at Seg::oD.  A trailing partial tile is padded with the
// identity, so the padding never reaches a stored value.
#pragma once

#include "kernels_fast.hpp"

namespace crs {

// Work item of this work-group when the 1-D grid (a multiple of 8 groups) is
// dealt round-robin over the 8 XCDs: consecutive items then run on one XCD,
// whose L2 holds the operands they share.
__device__ __forceinline__ int64_t xcd_item()
{
    const int64_t b = blockIdx.x, q = gridDim.x >> 3;
    return (b & 7) * q + (b >> 3);
}

// Operand of a wave-level product: element (o, t) at p[o * so + t * st] for
// o < no (zero beyond), where o is the row of a left operand or the column
// of a right operand and t the contraction index.
template <class T>
struct WOp {
    const cx<T>* p;
    int so, st, no;
};

// (cr, ci)[a][b] += opA(A) opB(B) over kd contraction steps for the RM x RN
// tiles of 16 x 16: rows 16 a + i of the left operand, columns 16 b + j of the
// right one; CA / CB conjugate the operand.  Operands are loaded G k-steps at
// a time, one group ahead of the MFMAs that consume the previous group.
template <class T, int RM, int RN, bool CA, bool CB, int G>
__device__ __forceinline__ void wave_mm(typename MF<T>::v4 (&cr)[RM][RN],
                                        typename MF<T>::v4 (&ci)[RM][RN], const WOp<T> A,
                                        const WOp<T> B, int kd)
{
    const int lane = threadIdx.x & 63, kr = lane >> 4, cc = lane & 15;
    const int ng = (kd + 4 * G - 1) / (4 * G);
    if (ng <= 0)
        return;
    const cx<T>* pa[RM];
    const cx<T>* pb[RN];
    bool oa[RM], ob[RN];
#pragma unroll
    for (int i = 0; i < RM; ++i) {
        const int o = 16 * i + cc;
        oa[i] = o < A.no;
        pa[i] = A.p + ((oa[i] ? o : 0) * A.so + kr * A.st);
    }
#pragma unroll
    for (int j = 0; j < RN; ++j) {
        const int o = 16 * j + cc;
        ob[j] = o < B.no;
        pb[j] = B.p + ((ob[j] ? o : 0) * B.so + kr * B.st);
    }
    const int sa = 4 * A.st, sb = 4 * B.st;
    cx<T> xa0[RM][G], yb0[RN][G], xa1[RM][G], yb1[RN][G];
    auto load = [&](cx<T>(&xa)[RM][G], cx<T>(&yb)[RN][G], int g) {
#pragma unroll
        for (int u = 0; u < G; ++u) {
            const int ks = g * G + u;
            const bool ok = 4 * ks + kr < kd;
#pragma unroll
            for (int i = 0; i < RM; ++i)
                xa[i][u] = ld_or0(pa[i] + ks * sa, A.p, ok && oa[i]);
#pragma unroll
            for (int j = 0; j < RN; ++j)
                yb[j][u] = ld_or0(pb[j] + ks * sb, B.p, ok && ob[j]);
        }
    };
    auto comp = [&](const cx<T>(&xa)[RM][G], const cx<T>(&yb)[RN][G]) {
#pragma unroll
        for (int u = 0; u < G; ++u)
#pragma unroll
            for (int i = 0; i < RM; ++i)
#pragma unroll
                for (int j = 0; j < RN; ++j) {
                    const T ar = xa[i][u].r, ai = CA ? -xa[i][u].i : xa[i][u].i;
                    const T br = yb[j][u].r, bi = CB ? -yb[j][u].i : yb[j][u].i;
                    cr[i][j] = MF<T>::mma(ar, br, cr[i][j]);
                    cr[i][j] = MF<T>::mma(-ai, bi, cr[i][j]);
                    ci[i][j] = MF<T>::mma(ar, bi, ci[i][j]);
                    ci[i][j] = MF<T>::mma(ai, br, ci[i][j]);
                }
    };
    load(xa0, yb0, 0);
    for (int g = 0; g < ng; g += 2) {
        if (g + 1 < ng)
            load(xa1, yb1, g + 1);
        comp(xa0, yb0);
        __builtin_amdgcn_sched_barrier(0);
        if (g + 1 < ng) {
            if (g + 2 < ng)
                load(xa0, yb0, g + 2);
            comp(xa1, yb1);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// acc += opA(A) opB(B) in the 3M form (one real MFMA per step for real
// data, RE), operands as in wave_mm.
template <class T, int RM, int RN, bool CA, bool CB, int G, bool RE = false>
__device__ __forceinline__ void wave_mm3(Acc3<T, RM, RN, RE>& acc, const WOp<T> A, const WOp<T> B,
                                         int kd)
{
    const int lane = threadIdx.x & 63, kr = lane >> 4, cc = lane & 15;
    const int ng = (kd + 4 * G - 1) / (4 * G);
    if (ng <= 0)
        return;
    const cx<T>* pa[RM];
    const cx<T>* pb[RN];
    bool oa[RM], ob[RN];
#pragma unroll
    for (int i = 0; i < RM; ++i) {
        const int o = 16 * i + cc;
        oa[i] = o < A.no;
        pa[i] = A.p + ((oa[i] ? o : 0) * A.so + kr * A.st);
    }
#pragma unroll
    for (int j = 0; j < RN; ++j) {
        const int o = 16 * j + cc;
        ob[j] = o < B.no;
        pb[j] = B.p + ((ob[j] ? o : 0) * B.so + kr * B.st);
    }
    const int sa = 4 * A.st, sb = 4 * B.st;
    cx<T> xa0[RM][G], yb0[RN][G], xa1[RM][G], yb1[RN][G];
    auto load = [&](cx<T>(&xa)[RM][G], cx<T>(&yb)[RN][G], int g) {
#pragma unroll
        for (int u = 0; u < G; ++u) {
            const int ks = g * G + u;
            const bool ok = 4 * ks + kr < kd;
#pragma unroll
            for (int i = 0; i < RM; ++i)
                xa[i][u] = ld_or0(pa[i] + ks * sa, A.p, ok && oa[i]);
#pragma unroll
            for (int j = 0; j < RN; ++j)
                yb[j][u] = ld_or0(pb[j] + ks * sb, B.p, ok && ob[j]);
        }
    };
    auto comp = [&](const cx<T>(&xa)[RM][G], const cx<T>(&yb)[RN][G]) {
#pragma unroll
        for (int u = 0; u < G; ++u) {
            T ar[RM], ai[RM], as[RM], br[RN], bi[RN], bs[RN];
#pragma unroll
            for (int i = 0; i < RM; ++i) {
                ar[i] = xa[i][u].r;
                ai[i] = CA ? -xa[i][u].i : xa[i][u].i;
                as[i] = ar[i] + ai[i];
            }
#pragma unroll
            for (int j = 0; j < RN; ++j) {
                br[j] = yb[j][u].r;
                bi[j] = CB ? -yb[j][u].i : yb[j][u].i;
                bs[j] = br[j] + bi[j];
            }
#pragma unroll
            for (int i = 0; i < RM; ++i)
#pragma unroll
                for (int j = 0; j < RN; ++j) {
                    acc.t1[i][j] = MF<T>::mma(ar[i], br[j], acc.t1[i][j]);
                    if constexpr (!RE) {
                        acc.t2[i][j] = MF<T>::mma(ai[i], bi[j], acc.t2[i][j]);
                        acc.t3[i][j] = MF<T>::mma(as[i], bs[j], acc.t3[i][j]);
                    }
                }
        }
    };
    load(xa0, yb0, 0);
    for (int g = 0; g < ng; g += 2) {
        if (g + 1 < ng)
            load(xa1, yb1, g + 1);
        comp(xa0, yb0);
        __builtin_amdgcn_sched_barrier(0);
        if (g + 1 < ng) {
            if (g + 2 < ng)
                load(xa0, yb0, g + 2);
            comp(xa1, yb1);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

template <class T, int RM, int RN>
__device__ __forceinline__ void zero_acc(typename MF<T>::v4 (&cr)[RM][RN],
                                         typename MF<T>::v4 (&ci)[RM][RN])
{
#pragma unroll
    for (int i = 0; i < RM; ++i)
#pragma unroll
        for (int j = 0; j < RN; ++j) {
            cr[i][j] = typename MF<T>::v4{0, 0, 0, 0};
            ci[i][j] = typename MF<T>::v4{0, 0, 0, 0};
        }
}

// The diagonal step of panel I of the tiled Cholesky, run by one wave: the
// tile S_II (lower triangle in sT, leading dimension 17) is factored and
// inverted in the registers (tile_chol).  L_II goes to L (diagonal
// {L_cc, 1 / L_cc}), D_I to Dg and to sD (leading dimension 17).  Returns
// true on a pivot that is not > 0.
template <class T>
__device__ __forceinline__ bool potrf_diag_tile(cx<T>* sT, cx<T>* sD, cx<T>* __restrict__ Lg,
                                                cx<T>* __restrict__ Dg, int m, int I)
{
    const int lane = threadIdx.x & 63, kr = lane >> 4, c0 = 16 * I;
    const int r = lane & 15, gi = c0 + r;
    cx<double> t[4], l[4], e[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int u = kr + 4 * v;
        t[v] = cvt<double>(sT[r * 17 + u]);
        if (gi >= m)
            t[v] = cx<double>{u == r ? 1.0 : 0.0, 0.0};
    }
    const bool fail = tile_chol<T>(t, l, e, m - c0);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int u = kr + 4 * v;
        const cx<T> d = cvt<T>(e[v]);
        sD[u * 17 + r] = d;
        Dg[I * 256 + u * 16 + r] = d;
        if (gi < m && u <= r)
            Lg[(int64_t)gi * m + c0 + u] = cvt<T>(l[v]);
    }
    return fail;
}

// -------------------------------------------------------------- k_potrf_rl

// Right-looking tiled Cholesky from memory, for the FP64 complex blocks above
// 128 that do not fit k_potrf_reg: one work-group of eight waves per block, whose
// chain of panels sets the time.  Per 16-column panel I: the waves form the tiles
// below the diagonal, L_RI = S_RI D_I^H, into L and into LDS; then wave 0
// runs ahead on the next panel -- S_JJ -= L_JI L_JI^H for J = I + 1, straight
// into LDS, and the diagonal step of panel J (potrf_diag_tile: L_JJ, D_J) --
// while the other seven waves update the remaining trailing tiles
// S_RC -= L_RI L_CI^H (I < C <= R) in place in the L slot, eight tiles per
// batch of loads, both product operands from LDS.  The diagonal steps, a
// chain of one wave, thus overlap the trailing updates instead of idling
// the work-group.  Panel 0 reads the tiles of A (Hermitian reading: lower
// triangle, the diagonal's imaginary parts dropped when a diagonal tile is
// factored) and writes every lower tile of the slot once; later panels read
// and update the slot.  Every panel's products are summed from zero and
// subtracted once, as in k_potrf_reg: real data gives the same bits in both.
//
// A left-looking form (one sum over all panels, other bits) was as fast in
// launches of more than 256 blocks: N = 600, 1023, 4096, m = 200 6705, 9389, 28835
// us a solve with it, 6689, 9364, 29020 without; m = 256, N = 4096 42.98 and 43.37
// ms.
template <class T, class EI>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 8))) void k_potrf_rl(const Seg* __restrict__ segs, int nseg,
                                                  int64_t total, const EI* __restrict__ inA,
                                                  cx<T>* __restrict__ W,
                                                  unsigned long long* __restrict__ flags)
{
    constexpr int kMaxS = 16; // m <= 256
    constexpr int TB = 8;     // trailing tiles per batch of loads
    __shared__ cx<T> sT[16 * 17]; // diagonal tile S_I (row-major, leading dimension 17)
    __shared__ cx<T> sD[16 * 17]; // D_I (leading dimension 17)
    __shared__ cx<T> sP[(kMaxS - 1) * 256]; // L_RI of R > I: tile R - I - 1, 16 x 16 row-major
    __shared__ int sFail;
    const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63, kr = lane >> 4, cc = lane & 15;
    const int nw = blockDim.x >> 6;
    const int64_t w = blockIdx.x;
    if (w >= total)
        return;
    const Seg& s = segs[find_seg(segs, nseg, w)];
    const int64_t t = w - s.w0;
    const int p = s.e0 + (int)t * s.es;
    const int m = s.m, S = (m + 15) >> 4;
    if ((flags[s.sys] >> 40) < (unsigned long long)s.level)
        return;
    const int64_t mm = (int64_t)m * m;
    const EI* Ap = inA + s.oA + (int64_t)p * mm;
    cx<T>* Lg = W + s.oL + t * mm;
    cx<T>* Dg = W + s.oD + t * (int64_t)S * 256;
    // element (i, j) of the lower triangle as panel I finds it, zero unless
    // ok; the load is issued in every lane (element (0, 0) stands in), so a
    // wave's count of memory operations in flight stays exact
    auto cur_el = [&](int I, int i, int j, bool ok) -> cx<T> {
        const int64_t e = ok ? (int64_t)i * m + j : 0;
        const cx<T> v = I == 0 ? cvt<T>(Ap[e]) : Lg[e];
        return ok ? v : czero<T>();
    };
    if (tid == 0)
        sFail = 0;
    bool fail = false;
    // panel 0's diagonal step (later ones run ahead, during the previous
    // panel's trailing updates)
    if (wv == 0) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = kr * 4 + v;
            const cx<T> e = cur_el(0, i, cc, cc <= i && i < m);
            if (cc <= i && i < m)
                sT[i * 17 + cc] = e;
        }
        wave_lds_sync();
        fail |= potrf_diag_tile<T>(sT, sD, Lg, Dg, m, 0);
    }
    __syncthreads();
    for (int I = 0; I < S; ++I) {
        const int c0 = 16 * I, kd = min(16, m - c0);
        // tiles below the diagonal: L_RI = S_RI D_I^H, to L and to LDS.
        // Contraction step q: lane (kr, cc) supplies S_RI[cc][4 q + kr] and
        // conj(D_I[cc][4 q + kr])
        for (int R = I + 1 + wv; R < S; R += nw) {
            cx<T> sa[4], db[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i = 16 * R + cc, tc = 4 * q + kr;
                sa[q] = cur_el(I, i, c0 + tc, i < m && tc < kd);
                db[q] = tc < kd ? sD[cc * 17 + tc] : czero<T>();
            }
            Acc3<T, 1, 1> acc;
            acc.zero();
#pragma unroll
            for (int q = 0; q < 4; ++q)
                acc.step(0, 0, sa[q].r, sa[q].i, db[q].r, -db[q].i);
            cx<T>* tp = sP + (R - I - 1) * 256;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int ii = MF<T>::row(kr, v), i = 16 * R + ii, j = c0 + cc;
                const cx<T> l{acc.re(0, 0, v), acc.im(0, 0, v)};
                const bool in = i < m && j < m;
                if (in)
                    Lg[(int64_t)i * m + j] = l;
                tp[ii * 16 + cc] = in ? l : czero<T>();
            }
        }
        __syncthreads();
        if (I + 1 < S) {
            const int nt = S - I - 1, ntile = nt * (nt + 1) / 2;
            if (wv == 0) {
                // look-ahead: S_JJ -= L_JI L_JI^H for J = I + 1 (sP tile 0),
                // straight into sT, then the diagonal step of panel J
                const int J = I + 1, cJ = 16 * J;
                Acc3<T, 1, 1> acc;
                acc.zero();
                const int ta = cc * 16 + kr;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const cx<T> a = sP[ta + 4 * q];
                    acc.step(0, 0, a.r, a.i, a.r, -a.i);
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = MF<T>::row(kr, v), gi = cJ + i, gj = cJ + cc;
                    const bool ok = cc <= i && gi < m;
                    const cx<T> o = cur_el(I, gi, gj, ok);
                    if (ok)
                        sT[i * 17 + cc] = cx<T>{o.r - acc.re(0, 0, v), o.i - acc.im(0, 0, v)};
                }
                wave_lds_sync();
                fail |= potrf_diag_tile<T>(sT, sD, Lg, Dg, m, J);
            } else {
                // the other trailing tiles S_RC -= L_RI L_CI^H, I < C <= R, row
                // by row (tile 0 is the look-ahead's), TB at a time: their
                // loads issued together before the stores, in every lane
                auto tile_rc = [&](int e, int& R, int& C) {
                    int r = (int)((sqrtf(8.0f * e + 1.0f) - 1.0f) * 0.5f);
                    while (r * (r + 1) / 2 > e)
                        --r;
                    while ((r + 1) * (r + 2) / 2 <= e)
                        ++r;
                    R = I + 1 + r;
                    C = I + 1 + (e - r * (r + 1) / 2);
                };
                const int nwt = nw - 1;
                for (int eb = wv; eb < ntile; eb += nwt * TB) {
                    cx<T> cur[TB][4];
#pragma unroll
                    for (int b = 0; b < TB; ++b) {
                        const int e = eb + nwt * b;
                        int R = I + 1, C = I + 1;
                        if (e < ntile)
                            tile_rc(e, R, C);
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const int i = 16 * R + MF<T>::row(kr, v), j = 16 * C + cc;
                            cur[b][v] = cur_el(I, i, j, e < ntile && i < m && j <= i);
                        }
                    }
#pragma unroll
                    for (int b = 0; b < TB; ++b) {
                        const int e = eb + nwt * b;
                        if (e >= ntile)
                            break;
                        int R, C;
                        tile_rc(e, R, C);
                        Acc3<T, 1, 1> acc;
                        acc.zero();
                        const int ta = (R - I - 1) * 256 + cc * 16 + kr, tb = (C - I - 1) * 256 + cc * 16 + kr;
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const cx<T> a = sP[ta + 4 * q], bb = sP[tb + 4 * q];
                            acc.step(0, 0, a.r, a.i, bb.r, -bb.i);
                        }
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const int i = 16 * R + MF<T>::row(kr, v), j = 16 * C + cc;
                            if (i < m && j <= i)
                                Lg[(int64_t)i * m + j] =
                                    cx<T>{cur[b][v].r - acc.re(0, 0, v), cur[b][v].i - acc.im(0, 0, v)};
                        }
                    }
                }
            }
        }
        __syncthreads();
    }
    if (wv == 0 && lane == 0 && fail)
        sFail = 1;
    __syncthreads();
    if (tid == 0 && sFail)
        atomicMin(&flags[s.sys], fail_key(s.level, s.ob0 + s.obs * p));
}

// Element of an exchanged tile in LDS: real data keeps the real part only.
template <class T, bool RE>
struct lds_el {
    using type = cx<T>;
    static __device__ __forceinline__ type to(const cx<T> v) { return v; }
    static __device__ __forceinline__ cx<T> from(const type v) { return v; }
};
template <class T>
struct lds_el<T, true> {
    using type = T;
    static __device__ __forceinline__ type to(const cx<T> v) { return v.r; }
    static __device__ __forceinline__ cx<T> from(const type v) { return cx<T>{v, T(0)}; }
};

// ------------------------------------------------------------- k_potrf_reg

// Tiled Cholesky with the whole block in the registers of one work-group, for
// every tiled block but FP64 complex ones above 128 (whose 544 KB at m = 256
// exceed a CU's 512 KB of registers).  The accumulators hold the upper tiles
// V_KI = A_IK^H, K <= I <= S - 1 < SM, of which wave w of SM / 2 owns the tile
// columns w and S - 1 - w: S + 1 tiles, the same for every wave.  Right-looking
// over J: U_JI = D_J V_JI (= L_IJ^H) for I > J, then V_KI -= U_JK^H U_JI.  In
// this form both operands of every product lie in the lanes as accumulators
// do (see the note in k_elim_mf), so the tiles U_JK pass from their owners to
// the other waves through LDS in lane order, and only D_J is transposed.  The
// owner of column J + 1 finishes its diagonal tile first and factors it
// (tile_chol) while the others update: two barriers per J, no read of L.
//
// One block's chain of diagonal steps bounds it, about 6 us each at m = 64 and at
// m = 256.  us per launch, from memory -> here:
//   few blocks   FP64 complex m = 64 43 -> 23, m = 128 89 -> 55; FP64 real m = 256
//                296 -> 96; FP32 complex m = 256 272 -> 144
//   600 blocks   FP64 complex m = 128 266 -> 147, FP32 complex m = 256 647 -> 443
// The complex instances of eight tile columns in FP64 and of sixteen in FP32 do
// not fit altogether: they keep about 70 and 30 of their 256 registers in scratch
// (176 and 104 bytes a lane), and the figures above are with that.
// The products are summed from zero and subtracted once per J, as k_potrf_rl
// does: real data gives the same bits in both.
template <class T, int SM, class EI = cx<T>, bool RE = false>
__global__ __launch_bounds__(32 * SM) __attribute__((amdgpu_waves_per_eu(2, 8))) void k_potrf_reg(
    const Seg* __restrict__ segs, int nseg, int64_t total, const EI* __restrict__ inA,
    cx<T>* __restrict__ W, unsigned long long* __restrict__ flags)
{
    using v4 = typename MF<T>::v4;
    using EL = lds_el<T, RE>;
    __shared__ typename EL::type sU[SM * 256]; // U_JK: register v of lane l at (4 K + v) 64 + l
    __shared__ typename EL::type sD[16 * 17];  // D_J
    __shared__ cx<T> sT[sizeof(T) == 4 ? 16 * 17 : 1];
    const int tid = threadIdx.x, lane = tid & 63, kr = lane >> 4, cc = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t w = blockIdx.x;
    if (w >= total)
        return;
    const Seg& s = segs[find_seg(segs, nseg, w)];
    const int64_t t = w - s.w0;
    const int p = s.e0 + (int)t * s.es;
    const int m = s.m, S = (m + 15) >> 4;
    if ((flags[s.sys] >> 40) < (unsigned long long)s.level)
        return;
    const int64_t mm = (int64_t)m * m;
    const EI* Ap = inA + s.oA + (int64_t)p * mm;
    cx<T>* Lg = W + s.oL + t * mm;
    cx<T>* Dg = W + s.oD + t * (int64_t)S * 256;
    // the wave's columns (-1: none); tile (K, b) in slot K, tile (K, a) in slot
    // SM - K, which never meet
    const int b = wv <= S - 1 - wv ? S - 1 - wv : -1, a = wv < S - 1 - wv ? wv : -1;
    v4 vr[SM + 1], vi[RE ? 1 : SM + 1];
    auto load = [&](v4& xr, v4& xi, int K, int I) {
        const int i = 16 * I + cc;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int j = 16 * K + MF<T>::row(kr, v);
            const bool ok = i < m && j <= i; // the lower triangle of A only
            const cx<T> x = cvt<T>(Ap[ok ? i * m + j : 0]);
            xr[v] = ok ? x.r : i == j ? T(1) : T(0);
            if constexpr (!RE)
                xi[v] = ok ? -x.i : T(0);
        }
    };
#pragma unroll
    for (int K = 0; K <= SM; ++K) {
        vr[K] = v4{0, 0, 0, 0};
        if constexpr (!RE)
            vi[K] = v4{0, 0, 0, 0};
    }
#pragma unroll
    for (int K = 0; K < SM; ++K) {
        if (K <= b)
            load(vr[K], vi[RE ? 0 : K], K, b);
        if (K < SM / 2 && K <= a)
            load(vr[SM - K], vi[RE ? 0 : SM - K], K, a);
    }
    bool fail = false;
    // diagonal step of column J (the owner's wave) on its finished tile
    auto diag = [&](int J, const v4 xr, const v4 xi) {
        cx<double> e[4], l[4], x[4];
        if constexpr (sizeof(T) == 4) { // rows 4 kr + v: through LDS
#pragma unroll
            for (int v = 0; v < 4; ++v)
                sT[cc * 17 + MF<T>::row(kr, v)] = cx<T>{xr[v], RE ? T(0) : -xi[v]};
            wave_lds_sync();
#pragma unroll
            for (int v = 0; v < 4; ++v)
                x[v] = cvt<double>(sT[cc * 17 + kr + 4 * v]);
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v)
                x[v] = cx<double>{xr[v], RE ? 0.0 : -xi[v]};
        }
        fail |= tile_chol<T, RE>(x, l, e, m - 16 * J);
        const int gi = 16 * J + cc;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int u = kr + 4 * v;
            const cx<T> d = cvt<T>(e[v]);
            sD[u * 17 + cc] = EL::to(d);
            Dg[J * 256 + u * 16 + cc] = d;
            if (gi < m && u <= cc)
                Lg[gi * m + 16 * J + u] = cvt<T>(l[v]);
        }
    };
    if (wv == 0)
        diag(0, vr[SM], vi[RE ? 0 : SM]);
    for (int J = 0;; ++J) {
        __syncthreads(); // D_J is there, U of J - 1 is read
        if (J + 1 == S)
            break;
        // U_JI of the wave's columns, to LDS and to L
        if (b > J) {
            cx<T> d[4];
#pragma unroll
            for (int v = 0; v < 4; ++v)
                d[v] = EL::from(sD[cc * 17 + MF<T>::row(kr, v)]);
            auto solve = [&](int I, const v4 xr, const v4 xi) {
                v4 ur = {0, 0, 0, 0}, ui = {0, 0, 0, 0};
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    ur = MF<T>::mma(d[v].r, xr[v], ur);
                    if constexpr (!RE) {
                        ui = MF<T>::mma(d[v].r, xi[v], ui);
                        ur = MF<T>::mma(d[v].i, -xi[v], ur);
                        ui = MF<T>::mma(d[v].i, xr[v], ui);
                    }
                }
                const int gi = 16 * I + cc;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    sU[(4 * I + v) * 64 + lane] = EL::to(cx<T>{ur[v], ui[v]});
                    if (gi < m)
                        Lg[gi * m + 16 * J + MF<T>::row(kr, v)] = cx<T>{ur[v], RE ? T(0) : -ui[v]};
                }
            };
#pragma unroll
            for (int K = 0; K < SM; ++K)
                if (K == J) {
                    solve(b, vr[K], vi[RE ? 0 : K]);
                    if (K < SM / 2 && a > J)
                        solve(a, vr[SM - K], vi[RE ? 0 : SM - K]);
                }
        }
        __syncthreads();
        if (b <= J)
            continue;
        auto operand = [&](int K, cx<T>(&x)[4]) {
#pragma unroll
            for (int v = 0; v < 4; ++v)
                x[v] = EL::from(sU[(4 * K + v) * 64 + lane]);
        };
        // the product is summed from zero and subtracted once
        auto update = [&](v4& xr, v4& xi, const cx<T>(&l)[4], const cx<T>(&r)[4]) {
            v4 pr = {0, 0, 0, 0}, pi = {0, 0, 0, 0};
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                pr = MF<T>::mma(l[v].r, r[v].r, pr);
                if constexpr (!RE) {
                    pi = MF<T>::mma(l[v].r, r[v].i, pi);
                    pr = MF<T>::mma(l[v].i, r[v].i, pr);
                    pi = MF<T>::mma(l[v].i, -r[v].r, pi);
                }
            }
            // subtracted here: hipcc 7.2 has moved this past the next branch,
            // where it no longer waits for the matrix unit
            xr -= pr;
            asm volatile("" : "+v"(xr));
            if constexpr (!RE) {
                xi -= pi;
                asm volatile("" : "+v"(xi));
            }
        };
        const int J1 = J + 1;
        if (b == J1 || a == J1) {
            cx<T> u[4];
            operand(J1, u);
            v4 xr = {0, 0, 0, 0}, xi = {0, 0, 0, 0};
#pragma unroll
            for (int K = 1; K < SM; ++K)
                if (K == J1) {
                    if (K < SM / 2 && a == J1) {
                        xr = vr[SM - K];
                        if constexpr (!RE)
                            xi = vi[SM - K];
                    } else {
                        xr = vr[K];
                        if constexpr (!RE)
                            xi = vi[K];
                    }
                }
            update(xr, xi, u, u);
            diag(J1, xr, xi);
        }
        if (b > J1) {
            cx<T> ub[4], ua[4], x[4], xn[4];
            operand(b, ub);
            operand(a > 0 ? a : 0, ua);
            operand(J1, xn);
#pragma unroll
            for (int K = 1; K < SM; ++K) {
                if (K > J && K <= b) {
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        x[v] = xn[v];
                    operand(K + 1 < SM ? K + 1 : K, xn);
                    update(vr[K], vi[RE ? 0 : K], x, ub);
                    if (K < SM / 2 && K <= a && a > J1)
                        update(vr[SM - K], vi[RE ? 0 : SM - K], x, ua);
                }
            }
        }
    }
    if (lane == 0 && fail)
        atomicMin(&flags[s.sys], fail_key(s.level, s.ob0 + s.obs * p));
}

// -------------------------------------------------------------- k_trsm_reg

// Forward substitutions L \ [B_p^H | B_{p-d} | y_p] of the tiled blocks: a
// work-group of four waves per (block, four 16-column strips), one strip per
// wave with all its row tiles of W = L X (at most SM) in accumulator registers.
// Right-looking over the columns J of L: X_J = D_J (G_J - W_J) (the result is
// the right operand as it lies, see the note in k_elim_mf), then
// W_I += L_IJ X_J for every I > J -- independent accumulators, so the matrix unit
// never waits for its own result.  Column J of L and D_J, the left operands of all
// four strips,
// come through LDS once per work-group, column J + 1 being fetched (into
// registers, then the other LDS buffer) while J is used: one barrier per
// column.  Tiles are stored 16 x 17 so that the operand reads (16 rows, four
// columns) fall on different banks.
//
// FP64 MFMA is the largest part of its time (busy 36 to 44 % for real data at m =
// 256, 39 % for complex data at m = 64): 16 (four-multiplication form; real data 4)
// instructions of 64 cycles per 16 x 16 product against four LDS reads and a
// quarter of a tile from L2; the rest waits at the barrier of each column.  Against one wave per strip (or two) that reads
// its finished rows back from memory, N = 4096, m = 256 real: 13.2 -> 4.9 ms
// per solve; FP64 complex N = 16384, m = 64, k = 32, solve and adjoint: 2.54 -> 2.05
// ms.  Eight waves per group halve the passes over L above 128 and were
// slower all the same (6.8 ms): one barrier then holds up eight strips.
// Waves per SIMD that the accumulators of SM row tiles (and the column in
// flight) leave room for.
template <class T, bool RE, int SM>
constexpr int trsm_waves()
{
    return SM == 16 ? (RE || sizeof(T) == 4 ? 2 : 1) : SM == 8 ? (RE || sizeof(T) == 4 ? 3 : 2)
                                                               : (RE || sizeof(T) == 4 ? 4 : 3);
}

template <class T, int SM, class EI = cx<T>, bool RE = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(trsm_waves<T, RE, SM>(), 8))) void k_trsm_reg(
    const Seg* __restrict__ segs, int nseg, int64_t total, int ngrp, int per, int with_mat, int with_rhs,
    const EI* __restrict__ inB, const EI* __restrict__ iny, cx<T>* __restrict__ W,
    const unsigned long long* __restrict__ flags)
{
    using v4 = typename MF<T>::v4;
    using EL = lds_el<T, RE>;
    constexpr int TS = 16 * 17; // a tile in LDS
    __shared__ typename EL::type sC[2][SM * TS]; // D_J, then L_IJ of I > J
    const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63, kr = lane >> 4, cc = lane & 15;
    const int64_t li = xcd_item();
    const int64_t w = li / ngrp;
    if (w >= total)
        return;
    const int grp = (int)(li - w * ngrp);
    const Seg& s = segs[find_seg(segs, nseg, w)];
    const int64_t t = w - s.w0;
    const int p = s.e0 + (int)t * s.es;
    const int m = s.m, k = s.k, d = s.d, S = (m + 15) >> 4;
    if ((flags[s.sys] >> 40) < (unsigned long long)s.level)
        return;
    const int64_t mm = (int64_t)m * m, mk = (int64_t)m * k;
    // the block's strips: S of B_p^H and S of B_{p-d} where it has those
    // neighbours, then those of y_p; this wave's is per grp + wv
    const int nP = with_mat && p + d < s.n ? S : 0, nQ = with_mat && p - d >= 0 ? S : 0;
    const int nst = nP + nQ + (with_rhs ? (k + 15) >> 4 : 0);
    if (per * grp >= nst)
        return;
    const int u = per * grp + wv;
    const bool on = wv < per && u < nst;
    const int src = !on || u < nP ? 0 : u < nP + nQ ? 1 : 2;
    const int c0 = 16 * (src == 0 ? u : src == 1 ? u - nP : u - nP - nQ);
    const int nc = on ? min(16, (src == 2 ? k : m) - c0) : 0;
    const cx<T>* Lg = W + s.oL + t * mm;
    const cx<T>* Dg = W + s.oD + t * (int64_t)S * 256;
    // thread tid moves element (tid / 16, tid % 16) of every tile of a column
    const int er = tid >> 4, ec = tid & 15;
    cx<T> cn[SM];
    auto fetch = [&](int J) {
        cn[0] = Dg[J * 256 + tid];
#pragma unroll
        for (int q = 1; q < SM; ++q) {
            cn[q] = czero<T>();
            if (16 * (J + q) < m) // uniform
                cn[q] = Lg[(int64_t)min(16 * (J + q) + er, m - 1) * m + min(16 * J + ec, m - 1)];
        }
    };
    auto put = [&](int J) {
#pragma unroll
        for (int q = 0; q < SM; ++q) {
            const bool ok = q == 0 || 16 * (J + q) + er < m;
            if (q == 0 || 16 * (J + q) < m)
                sC[J & 1][q * TS + er * 17 + ec] =
                    EL::to(cx<T>{ok ? cn[q].r : T(0), ok ? cn[q].i : T(0)});
        }
    };
    fetch(0);
    // right-hand side: element (r, c) is G[r * gr + (c0 + c) * gc], conjugated
    // for B_p^H
    const EI* G = src == 2 ? iny + s.oy + (int64_t)p * mk
                           : inB + s.oB + (int64_t)(src == 0 ? p : p - d) * mm;
    const int gr = src == 0 ? 1 : src == 1 ? m : k, gc = src == 0 ? m : 1;
    const int ldo = src == 2 ? k : m;
    cx<T>* out = W + (src == 0 ? s.oP : src == 1 ? s.oQ : s.og) + t * (src == 2 ? mk : mm) + c0 + cc;
    // every element set on every path: hipcc 7.2 has dropped the real part of a
    // value that only some paths to its use defined
    v4 wr[SM], wi[RE ? 1 : SM];
#pragma unroll
    for (int I = 0; I < SM; ++I) {
        wr[I] = v4{0, 0, 0, 0};
        if (!RE)
            wi[I] = v4{0, 0, 0, 0};
    }
    // rows of the right-hand side for column J, fetched a column ahead
    const EI* Gc = G + (c0 + min(cc, max(nc, 1) - 1)) * gc;
    const bool okc = cc < nc;
    EI gn[4] = {};
    auto rows = [&](int J) {
        if (nc > 0) { // uniform within the wave; without a strip there is no G
#pragma unroll
            for (int v = 0; v < 4; ++v)
                gn[v] = Gc[min(16 * J + MF<T>::row(kr, v), m - 1) * gr];
        }
    };
    rows(0);
    put(0);
    __syncthreads();
    // the columns by recursion: the compiler leaves a loop of this size rolled,
    // and the accumulators need constant indices
    auto column = [&](auto self, auto Jc) {
        constexpr int J = decltype(Jc)::value;
        if (J >= S)
            return;
        const typename EL::type* col = sC[J & 1] + cc * 17;
        // w = G_J - W_J
        v4 gr4, gi4 = {0, 0, 0, 0};
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const cx<T> x = cvt<T>(gn[v]);
            const bool ok = okc && 16 * J + MF<T>::row(kr, v) < m;
            gr4[v] = ok ? x.r - wr[J][v] : T(0);
            if constexpr (!RE)
                gi4[v] = ok ? (src == 0 ? -x.i : x.i) - wi[J][v] : T(0);
        }
        if (J + 1 < S) {
            fetch(J + 1);
            rows(J + 1);
        }
        cx<T> a[4], an[4];
        v4 xr = {0, 0, 0, 0}, xi = {0, 0, 0, 0}, ni;
#pragma unroll
        for (int v = 0; v < 4; ++v)
            an[v] = czero<T>();
        auto operand = [&](int q, cx<T>(&x)[4]) { // left operand of tile q of the column
#pragma unroll
            for (int v = 0; v < 4; ++v)
                x[v] = EL::from(col[q * TS + MF<T>::row(kr, v)]);
        };
        if (nc > 0) {
            operand(0, a);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                xr = MF<T>::mma(a[v].r, gr4[v], xr);
                if constexpr (!RE) {
                    xi = MF<T>::mma(a[v].r, gi4[v], xi);
                    xr = MF<T>::mma(a[v].i, -gi4[v], xr);
                    xi = MF<T>::mma(a[v].i, gr4[v], xi);
                }
            }
        }
        ni = -xi;
        if (J + 1 < SM && nc > 0) {
            operand(1, an);
#pragma unroll
            for (int I = J + 1; I < SM; ++I) {
                if (I >= S)
                    break;
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    a[v] = an[v];
                if (I + 1 < SM)
                    operand(I + 1 - J, an);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    wr[I] = MF<T>::mma(a[v].r, xr[v], wr[I]);
                    if constexpr (!RE) {
                        wi[I] = MF<T>::mma(a[v].r, xi[v], wi[I]);
                        wr[I] = MF<T>::mma(a[v].i, ni[v], wr[I]);
                        wi[I] = MF<T>::mma(a[v].i, xr[v], wi[I]);
                    }
                }
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = 16 * J + MF<T>::row(kr, v);
            if (r < m && cc < nc)
                out[(int64_t)r * ldo] = cx<T>{xr[v], RE ? T(0) : xi[v]};
        }
        if (J + 1 < S)
            put(J + 1);
        __syncthreads();
        if constexpr (J + 1 < SM)
            self(self, std::integral_constant<int, J + 1>{});
    };
    column(column, std::integral_constant<int, 0>{});
}

// -------------------------------------------------------------- k_trsm_few

// The right-hand sides alone in FP32, few strips a block: a strip of k_trsm_reg
// is one wave's chain of S (S + 1) / 2 tile products, with idle waves beside
// it.  Here a work-group has one strip and one wave per row tile (blockDim = 64 x
// the largest tile count of the launch): wave J forms X_J = D_J (G_J - W_J) and
// passes it on through LDS, the waves I > J add L_IJ X_J to their W_I.  A tile of
// L has one reader then and comes straight from memory, a column ahead.  The
// products and their order are those of k_trsm_reg: the same bits.
template <class T, class EI = cx<T>, bool RE = false>
__global__ __launch_bounds__(1024) void k_trsm_few(const Seg* __restrict__ segs, int nseg,
                                                   int64_t total, int nstrip,
                                                   const EI* __restrict__ iny, cx<T>* __restrict__ W,
                                                   const unsigned long long* __restrict__ flags)
{
    using v4 = typename MF<T>::v4;
    __shared__ cx<T> sX[2][256]; // X_J: register v of lane l at 64 v + l
    const int lane = threadIdx.x & 63, kr = lane >> 4, cc = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t li = xcd_item();
    const int64_t w = li / nstrip;
    const int c0 = 16 * (int)(li - w * nstrip);
    if (w >= total)
        return;
    const Seg& s = segs[find_seg(segs, nseg, w)];
    const int64_t t = w - s.w0;
    const int p = s.e0 + (int)t * s.es;
    const int m = s.m, k = s.k, S = (m + 15) >> 4;
    if (c0 >= k || (flags[s.sys] >> 40) < (unsigned long long)s.level)
        return;
    const int64_t mm = (int64_t)m * m, mk = (int64_t)m * k;
    const int nc = min(16, k - c0);
    // the wave's tile; one past the block's edge (a smaller block in a launch
    // of larger ones) reads no L and stores nothing
    const int r0 = 16 * wv, row = r0 + cc;
    const bool own = wv < S;
    const cx<T>* Lr = W + s.oL + t * mm + (int64_t)min(row, m - 1) * m;
    const cx<T>* Dg = W + s.oD + t * (int64_t)S * 256 + min(wv, S - 1) * 256 + cc * 16;
    const EI* G = iny + s.oy + (int64_t)p * mk + c0 + min(cc, nc - 1);
    cx<T>* out = W + s.og + t * mk + c0 + cc;
    cx<T> a[4], an[4], d[4], g[4];
    auto fetch = [&](int J) { // L_IJ, J < I = wv < S: columns below 16 I < m
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const cx<T> x = Lr[16 * J + MF<T>::row(kr, v)];
            an[v] = cx<T>{row < m ? x.r : T(0), row < m ? x.i : T(0)};
        }
    };
#pragma unroll
    for (int v = 0; v < 4; ++v)
        an[v] = czero<T>();
    if (own && wv > 0)
        fetch(0);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int rr = MF<T>::row(kr, v);
        const bool ok = cc < nc && r0 + rr < m;
        d[v] = Dg[rr];
        const cx<T> x = cvt<T>(G[(int64_t)min(r0 + rr, m - 1) * k]);
        g[v] = cx<T>{ok ? x.r : T(0), ok ? x.i : T(0)};
    }
    v4 wr = {0, 0, 0, 0}, wi = {0, 0, 0, 0};
    for (int J = 0; J < S; ++J) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
            a[v] = an[v];
        if (own && wv > J + 1)
            fetch(J + 1);
        if (wv == J) {
            v4 xr = {0, 0, 0, 0}, xi = {0, 0, 0, 0};
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const bool ok = cc < nc && r0 + MF<T>::row(kr, v) < m;
                const T br = ok ? g[v].r - wr[v] : T(0), bi = ok ? g[v].i - wi[v] : T(0);
                xr = MF<T>::mma(d[v].r, br, xr);
                if constexpr (!RE) {
                    xi = MF<T>::mma(d[v].r, bi, xi);
                    xr = MF<T>::mma(d[v].i, -bi, xr);
                    xi = MF<T>::mma(d[v].i, br, xi);
                }
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = r0 + MF<T>::row(kr, v);
                const cx<T> x{xr[v], RE ? T(0) : xi[v]};
                sX[J & 1][64 * v + lane] = x;
                if (r < m && cc < nc)
                    out[(int64_t)r * k] = x;
            }
        }
        __syncthreads();
        if (own && wv > J) {
            cx<T> x[4];
#pragma unroll
            for (int v = 0; v < 4; ++v)
                x[v] = sX[J & 1][64 * v + lane];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                wr = MF<T>::mma(a[v].r, x[v].r, wr);
                if constexpr (!RE) {
                    wi = MF<T>::mma(a[v].r, x[v].i, wi);
                    wr = MF<T>::mma(a[v].i, -x[v].i, wr);
                    wi = MF<T>::mma(a[v].i, x[v].r, wi);
                }
            }
        }
    }
}

// ------------------------------------------------------------ k_trsm_strip

// One wave per (eliminated block, 16-column strip), sweeping the row tiles of
// its strip without barriers: X_I = D_I (G_I - L_I X) with the finished rows of
// X read back as the right operand.  Serves FP64 complex blocks above 128, for
// which the accumulators of k_trsm_reg (256 registers of 512, and scratch)
// leave one wave per SIMD: N = 1023, m = 200, 2.52 ms per solve here, 2.80
// there.  GD contraction steps per load group: eight for launches of few blocks.
template <class T, class EI, int GD>
__global__ __launch_bounds__(64) void k_trsm_strip(const Seg* __restrict__ segs, int nseg,
                                                 int64_t total, int nstrip, int with_mat,
                                                 int with_rhs, const EI* __restrict__ inB,
                                                 const EI* __restrict__ iny,
                                                 cx<T>* __restrict__ W,
                                                 const unsigned long long* __restrict__ flags)
{
    using v4 = typename MF<T>::v4;
    const int lane = threadIdx.x, kr = lane >> 4, cc = lane & 15;
    const int64_t li = xcd_item();
    const int64_t w = li / nstrip;
    int u = (int)(li - w * nstrip);
    if (w >= total)
        return;
    const Seg& s = segs[find_seg(segs, nseg, w)];
    const int64_t t = w - s.w0;
    const int p = s.e0 + (int)t * s.es;
    const int m = s.m, k = s.k, d = s.d, S = (m + 15) >> 4;
    if ((flags[s.sys] >> 40) < (unsigned long long)s.level)
        return;
    const int64_t mm = (int64_t)m * m, mk = (int64_t)m * k;
    int src = 2;
    if (with_mat) {
        if (u < 2 * S)
            src = u < S ? 0 : 1;
        else
            u -= 2 * S;
    }
    int c0;
    if (src == 2) {
        c0 = 16 * u;
        if (!with_rhs || c0 >= k)
            return;
    } else {
        c0 = 16 * (src == 0 ? u : u - S);
        if (src == 0 ? p + d >= s.n : p - d < 0)
            return;
    }
    const int nc = min(16, (src == 2 ? k : m) - c0);
    // element (r, c) of the right-hand side is G[r * gr + c * gc]
    const EI* G;
    int gr, gc;
    cx<T>* out;
    if (src == 0) {
        G = inB + s.oB + (int64_t)p * mm; // B_p^H: conjugated below
        gr = 1;
        gc = m;
        out = W + s.oP + t * mm;
    } else if (src == 1) {
        G = inB + s.oB + (int64_t)(p - d) * mm;
        gr = m;
        gc = 1;
        out = W + s.oQ + t * mm;
    } else {
        G = iny + s.oy + (int64_t)p * mk;
        gr = k;
        gc = 1;
        out = W + s.og + t * mk;
    }
    const int ldo = src == 2 ? k : m;
    const cx<T>* Lg = W + s.oL + t * mm;
    const cx<T>* Dg = W + s.oD + t * (int64_t)S * 256;
    for (int I = 0; I < S; ++I) {
        const int r0 = 16 * I;
        Acc3<T, 1, 1, false> acc;
        acc.zero();
        wave_mm3<T, 1, 1, false, false, GD, false>(acc, WOp<T>{Lg + (int64_t)r0 * m, m, 1, m - r0},
                                                   WOp<T>{out + c0, 1, ldo, nc}, r0);
        // w = G_I - acc stays in the accumulator layout: register v of lane
        // (kr, cc) holds row MF::row(kr, v) of column cc, which is the right
        // operand of contraction step v once the left operand D_I supplies
        // column MF::row(kr, v) of its row cc
        Acc3<T, 1, 1, false> x;
        x.zero();
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int rr = MF<T>::row(kr, v), r = r0 + rr;
            const cx<T> a = Dg[I * 256 + cc * 16 + rr];
            cx<T> g = (r < m && cc < nc) ? cvt<T>(G[r * gr + (c0 + cc) * gc]) : czero<T>();
            if (src == 0)
                g.i = -g.i;
            x.step(0, 0, a.r, a.i, g.r - acc.re(0, 0, v), g.i - acc.im(0, 0, v));
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = r0 + MF<T>::row(kr, v);
            if (r < m && cc < nc)
                out[(int64_t)r * ldo + c0 + cc] = cx<T>{x.re(0, 0, v), x.im(0, 0, v)};
        }
        __syncthreads(); // the rows just stored are the next tiles' operands
    }
}

// ------------------------------------------------------------ k_reduce_big

// One wave per output tile of TT = 16 TW rows and columns of a kept block
// (NT = ceil(m / TT)): with_mat gives the NT (NT + 1) / 2 lower tiles of A'
// and the NT^2 tiles of B', with_rhs the NT ceil(k / TT) tiles of y' after
// them.  TW = 2 serves the right-hand sides of blocks above 64 (k > 16);
// TW = 1 the blocks of 32 < m <= 64, the right-hand sides with k <= 16 of
// larger blocks, and the levels of m <= 32 with too few blocks to fill the
// GPU one wave per block.
template <class T, int TW, class EI = cx<T>, bool RE = false>
__global__ __launch_bounds__(64) void k_reduce_big(const Seg* __restrict__ segs, int nseg,
                                                   int64_t total, int ntile, int with_mat,
                                                   int with_rhs, const EI* __restrict__ inA,
                                                   const EI* __restrict__ iny,
                                                   cx<T>* __restrict__ W,
                                                   const unsigned long long* __restrict__ flags)
{
    using v4 = typename MF<T>::v4;
    const int lane = threadIdx.x, kr = lane >> 4, cc = lane & 15;
    const int64_t li = xcd_item();
    const int64_t w = li / ntile;
    int u = (int)(li - w * ntile);
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
        return; // the level's elimination broke down: stop this system
    constexpr int TT = 16 * TW;
    const int NT = (m + TT - 1) / TT, nV = NT * (NT + 1) / 2, nF = NT * NT;
    int kind, ti, tj;
    if (with_mat && u < nV + nF) {
        if (u < nV) {
            kind = 0;
            ti = tri_row(u);
            tj = u - ti * (ti + 1) / 2;
        } else {
            kind = 1;
            u -= nV;
            ti = u / NT;
            tj = u % NT;
            if (!hasR || r + d >= n)
                return;
        }
    } else {
        if (with_mat)
            u -= nV + nF;
        const int Tk = (k + TT - 1) / TT;
        if (!with_rhs || u >= NT * Tk)
            return;
        kind = 2;
        ti = u / Tk;
        tj = u % Tk;
    }
    const cx<T>* Pl = W + s.oP + tl * mm;
    const cx<T>* Qr = W + s.oQ + tr * mm;
    const cx<T>* Pr = W + s.oP + tr * mm;
    const int i0 = TT * ti, j0 = TT * tj;
    // 16 x 16 tiles: the elements of A_q (kind 0) or y_q (kind 2) this lane
    // subtracts from, loaded first and in every lane (element 0 stands in):
    // the loads overlap the products and none waits behind a store of the
    // tile (32 x 32 tiles, short of registers, load each before its store)
    cx<T> xo[TW][TW][4];
    auto load_xo = [&] {
        if (kind == 1)
            return;
        const EI* src = kind == 0 ? inA + s.oA + q * mm : iny + s.oy + q * mk;
        const int ld = kind == 0 ? m : k;
#pragma unroll
        for (int a = 0; a < TW; ++a)
#pragma unroll
            for (int b = 0; b < TW; ++b)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = i0 + 16 * a + MF<T>::row(kr, v), j = j0 + 16 * b + cc;
                    const bool ok = i < m && (kind == 0 ? j <= i : j < k);
                    xo[a][b][v] = cvt<T>(src[ok ? i * ld + j : 0]);
                }
    };
    if constexpr (TW == 1)
        load_xo();
    Acc3<T, TW, TW, RE> acc;
    acc.zero();
    if (kind == 0) {
        if (hasL)
            wave_mm3<T, TW, TW, true, false, 2 / TW, RE>(acc, WOp<T>{Pl + i0, 1, m, m - i0},
                                             WOp<T>{Pl + j0, 1, m, m - j0}, m);
        if (hasR)
            wave_mm3<T, TW, TW, true, false, 2 / TW, RE>(acc, WOp<T>{Qr + i0, 1, m, m - i0},
                                             WOp<T>{Qr + j0, 1, m, m - j0}, m);
        cx<T>* Vo = W + s.oAo + oi * mm;
#pragma unroll
        for (int a = 0; a < TW; ++a)
#pragma unroll
            for (int b = 0; b < TW; ++b)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = i0 + 16 * a + MF<T>::row(kr, v), j = j0 + 16 * b + cc;
                    if (i < m && j <= i) {
                        const cx<T> x = TW == 1 ? xo[a][b][v] : cvt<T>(inA[s.oA + q * mm + i * m + j]);
                        cx<T> o{x.r - acc.re(a, b, v), x.i - acc.im(a, b, v)};
                        if (i == j)
                            o.i = T(0);
                        Vo[i * m + j] = o;
                    }
                }
    } else if (kind == 1) {
        wave_mm3<T, TW, TW, true, false, 2 / TW, RE>(acc, WOp<T>{Pr + i0, 1, m, m - i0},
                                         WOp<T>{Qr + j0, 1, m, m - j0}, m);
        cx<T>* Fo = W + s.oBo + oi * mm;
#pragma unroll
        for (int a = 0; a < TW; ++a)
#pragma unroll
            for (int b = 0; b < TW; ++b)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = i0 + 16 * a + MF<T>::row(kr, v), j = j0 + 16 * b + cc;
                    if (i < m && j < m)
                        Fo[i * m + j] = cx<T>{-acc.re(a, b, v), -acc.im(a, b, v)};
                }
    } else {
        const cx<T>* gl = W + s.og + tl * mk;
        const cx<T>* gr = W + s.og + tr * mk;
        if (hasL)
            wave_mm3<T, TW, TW, true, false, 2 / TW, RE>(acc, WOp<T>{Pl + i0, 1, m, m - i0},
                                             WOp<T>{gl + j0, 1, k, k - j0}, m);
        if (hasR)
            wave_mm3<T, TW, TW, true, false, 2 / TW, RE>(acc, WOp<T>{Qr + i0, 1, m, m - i0},
                                             WOp<T>{gr + j0, 1, k, k - j0}, m);
        cx<T>* vo = W + s.oyo + oi * mk;
#pragma unroll
        for (int a = 0; a < TW; ++a)
#pragma unroll
            for (int b = 0; b < TW; ++b)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = i0 + 16 * a + MF<T>::row(kr, v), c = j0 + 16 * b + cc;
                    if (i < m && c < k) {
                        const cx<T> x = TW == 1 ? xo[a][b][v] : cvt<T>(iny[s.oy + q * mk + i * k + c]);
                        vo[i * k + c] = cx<T>{x.r - acc.re(a, b, v), x.i - acc.im(a, b, v)};
                    }
                }
    }
}

// ------------------------------------------------------------ k_reduce_lds

// The matrix part of the reduced system (A' lower tiles, B') for blocks above
// 32 with the operand panels staged in LDS: one work-group of four waves per
// (kept block, 64 x 64 tile); wave (a, b) owns the 32 x 32 quarter at rows
// 32 a, columns 32 b of the tile.  For each 16-row panel of the contraction
// the work-group loads 16 x 64 of the left and of the right operand once
// (every element then feeds 32 output rows or columns instead of 16 in
// k_reduce_big) and the waves run their 3M products from LDS; the next panel
// is fetched into registers while the current one is consumed (two LDS
// buffers, one barrier per panel).  Items per kept block: the
// NT (NT + 1) / 2 lower tiles of A', then the NT^2 tiles of B' (NT =
// ceil(m / 64)).  The right-hand-side tiles y' run in k_reduce_big.
//
// FP64 MFMA bounds it: at m = 256 it is busy 67 % of the time for complex data and
// 48 to 55 % for real data, which keeps real parts only in LDS (complex elements
// there met bank conflicts) and leaves out the 16 x 16 tiles without output: N = 4096, m = 256 real 8.85 -> 7.37 ms per solve.  Complex data
// runs all four tiles of a quarter: leaving some out cost the loop its
// schedule (N = 4096, m = 256: 18.3 -> 20.2 ms with y'; with tests inside the
// loop N = 1023, m = 200 3.87 -> 4.25 ms).
template <class T, class EI = cx<T>, bool RE = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 8))) void k_reduce_lds(const Seg* __restrict__ segs, int nseg,
                                                    int64_t total, int ntile,
                                                    const EI* __restrict__ inA,
                                                    cx<T>* __restrict__ W,
                                                    const unsigned long long* __restrict__ flags)
{
    using EL = lds_el<T, RE>;
    // real panels: rows 32 banks apart, so that the two rows that half a wave
    // reads at a time do not meet
    constexpr int KP = 16, LD = RE ? (sizeof(T) == 8 ? 80 : 72) : 65;
    __shared__ typename EL::type sA[2][KP * LD], sB[2][KP * LD];
    const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63, kr = lane >> 4, cc = lane & 15;
    const int64_t li = xcd_item();
    // real data: the quarter of each wave turns with the item, so that the
    // lighter quarters at the edges of a block fall on every SIMD
    const int wq = RE ? __builtin_amdgcn_readfirstlane((wv + (int)li + (int)(li >> 5)) & 3) : wv;
    const int wa = wq >> 1, wb = wq & 1;
    const int64_t w = li / ntile;
    int u = (int)(li - w * ntile);
    if (w >= total)
        return;
    const Seg& s = segs[find_seg(segs, nseg, w)];
    const int64_t t = w - s.w0;
    const int q = s.k0 + (int)t * s.ks;
    const int m = s.m, d = s.d, n = s.n;
    const int l = q - d, r = q + d;
    const bool hasL = l >= 0, hasR = r < n;
    const int64_t tl = hasL ? (l - s.e0) / s.es : 0, tr = hasR ? (r - s.e0) / s.es : 0;
    const int64_t oi = s.out_by_pos ? q : t;
    const int64_t mm = (int64_t)m * m;
    if ((flags[s.sys] >> 40) <= (unsigned long long)s.level)
        return; // the level's elimination broke down: stop this system
    const int NT = (m + 63) >> 6, nV = NT * (NT + 1) / 2, nF = NT * NT;
    int kind, ti, tj;
    if (u < nV) {
        kind = 0;
        ti = tri_row(u);
        tj = u - ti * (ti + 1) / 2;
    } else if (u < nV + nF) {
        kind = 1;
        u -= nV;
        ti = u / NT;
        tj = u % NT;
        if (!hasR || r + d >= n)
            return;
    } else {
        return;
    }
    const cx<T>* Pl = W + s.oP + tl * mm;
    const cx<T>* Qr = W + s.oQ + tr * mm;
    const cx<T>* Pr = W + s.oP + tr * mm;
    const int i0 = 64 * ti, j0 = 64 * tj;
    // products: A' tiles sum P_l^H P_l (hasL) and Q_r^H Q_r (hasR); B' tiles
    // are P_r^H Q_r
    const int npr = kind == 0 ? (hasL ? 1 : 0) + (hasR ? 1 : 0) : 1;
    const int nkp = (m + KP - 1) / KP, npan = npr * nkp;
    // 16 x 16 tiles past the block's edge or above the diagonal of A' hold no
    // output (complex data: quarters above the diagonal only)
    const int ib = i0 + 32 * wa, jb = j0 + 32 * wb;
    auto on = [&](int a, int b) {
        return ib + 16 * a < m && jb + 16 * b < m && !(kind == 0 && jb + 16 * b > ib + 16 * a);
    };
    const bool on00 = on(0, 0), on01 = on(0, 1), on10 = on(1, 0), on11 = on(1, 1);
    const bool live = on00 || on01 || on10 || on11;
    const bool full = RE ? on00 && on01 && on10 && on11 : !(kind == 0 && ti == tj && wb > wa);
    // thread tid moves elements e = tid + 256 e4 of a 16 x 64 panel: row
    // e / 64, column e % 64
    cx<T> ra0, ra1, ra2, ra3, rb0, rb1, rb2, rb3;
#define CRS_PANEL_LOAD(pn)                                                                         \
    do {                                                                                           \
        const int pr_ = (pn) / nkp, t0_ = ((pn) - pr_ * nkp) * KP;                                  \
        const cx<T>* X_ = kind == 1 ? Pr : ((hasL && pr_ == 0) ? Pl : Qr);                          \
        const cx<T>* Y_ = kind == 1 ? Qr : X_;                                                      \
        const int row_ = tid >> 6, col_ = tid & 63;                                                 \
        const bool oa_ = i0 + col_ < m, ob_ = j0 + col_ < m;                                        \
        const cx<T>* xa_ = X_ + (int64_t)(t0_ + row_) * m + i0 + col_;                              \
        const cx<T>* yb_ = Y_ + (int64_t)(t0_ + row_) * m + j0 + col_;                              \
        const int64_t st_ = 4 * (int64_t)m;                                                         \
        ra0 = (t0_ + row_ < m && oa_) ? xa_[0] : czero<T>();                                        \
        ra1 = (t0_ + row_ + 4 < m && oa_) ? xa_[st_] : czero<T>();                                  \
        ra2 = (t0_ + row_ + 8 < m && oa_) ? xa_[2 * st_] : czero<T>();                              \
        ra3 = (t0_ + row_ + 12 < m && oa_) ? xa_[3 * st_] : czero<T>();                             \
        rb0 = (t0_ + row_ < m && ob_) ? yb_[0] : czero<T>();                                        \
        rb1 = (t0_ + row_ + 4 < m && ob_) ? yb_[st_] : czero<T>();                                  \
        rb2 = (t0_ + row_ + 8 < m && ob_) ? yb_[2 * st_] : czero<T>();                              \
        rb3 = (t0_ + row_ + 12 < m && ob_) ? yb_[3 * st_] : czero<T>();                             \
    } while (0)
#define CRS_PANEL_STORE(b)                                                                         \
    do {                                                                                           \
        const int o_ = (tid >> 6) * LD + (tid & 63);                                                \
        sA[b][o_] = EL::to(ra0);                                                                            \
        sA[b][o_ + 4 * LD] = EL::to(ra1);                                                                   \
        sA[b][o_ + 8 * LD] = EL::to(ra2);                                                                   \
        sA[b][o_ + 12 * LD] = EL::to(ra3);                                                                  \
        sB[b][o_] = EL::to(rb0);                                                                            \
        sB[b][o_ + 4 * LD] = EL::to(rb1);                                                                   \
        sB[b][o_ + 8 * LD] = EL::to(rb2);                                                                   \
        sB[b][o_ + 12 * LD] = EL::to(rb3);                                                                  \
    } while (0)
    Acc3<T, 2, 2, RE> acc;
    acc.zero();
    if (npan > 0) {
        CRS_PANEL_LOAD(0);
        CRS_PANEL_STORE(0);
    }
    __syncthreads();
    for (int pn = 0; pn < npan; ++pn) {
        const int b = pn & 1;
        if (pn + 1 < npan)
            CRS_PANEL_LOAD(pn + 1);
        auto operands = [&](int ks, cx<T>(&x)[2], cx<T>(&y)[2]) {
            const int row = 4 * ks + kr;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                x[i] = EL::from(sA[b][row * LD + 32 * wa + 16 * i + cc]);
                y[i] = EL::from(sB[b][row * LD + 32 * wb + 16 * i + cc]);
                x[i].i = -x[i].i; // conj: the left operand is X^H
            }
        };
        if (full) {
#pragma unroll
            for (int ks = 0; ks < KP / 4; ++ks) {
                cx<T> x[2], y[2];
                operands(ks, x, y);
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc.step(i, j, x[i].r, x[i].i, y[j].r, y[j].i);
            }
        } else if (RE && live) {
#pragma unroll
            for (int ks = 0; ks < KP / 4; ++ks) {
                cx<T> x[2], y[2];
                operands(ks, x, y);
                if (on00)
                    acc.step(0, 0, x[0].r, x[0].i, y[0].r, y[0].i);
                if (on01)
                    acc.step(0, 1, x[0].r, x[0].i, y[1].r, y[1].i);
                if (on10)
                    acc.step(1, 0, x[1].r, x[1].i, y[0].r, y[0].i);
                if (on11)
                    acc.step(1, 1, x[1].r, x[1].i, y[1].r, y[1].i);
            }
        }
        if (pn + 1 < npan)
            CRS_PANEL_STORE(b ^ 1);
        __syncthreads();
    }
#undef CRS_PANEL_LOAD
#undef CRS_PANEL_STORE
    if (kind == 0) {
        const EI* Aq = inA + s.oA + q * mm;
        cx<T>* Vo = W + s.oAo + oi * mm;
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = ib + 16 * a + MF<T>::row(kr, v), j = jb + 16 * b + cc;
                    if (i < m && j <= i) {
                        const cx<T> x = cvt<T>(Aq[(int64_t)i * m + j]);
                        cx<T> o{x.r - acc.re(a, b, v), x.i - acc.im(a, b, v)};
                        if (i == j)
                            o.i = T(0);
                        Vo[(int64_t)i * m + j] = o;
                    }
                }
    } else {
        cx<T>* Fo = W + s.oBo + oi * mm;
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = ib + 16 * a + MF<T>::row(kr, v), j = jb + 16 * b + cc;
                    if (i < m && j < m)
                        Fo[(int64_t)i * m + j] = cx<T>{-acc.re(a, b, v), -acc.im(a, b, v)};
                }
    }
}

// -------------------------------------------------------------- k_back_big

// One work-group per (eliminated block, 16-column strip of x_p), one wave per
// 16-row tile J of the block (blockDim = 64 x the largest tile count of the
// launch; waves beyond a block's S tiles only join the barriers):
//   phase A, all waves at once: w_J = g_J - Q_J x_{p-d} - P_J x_{p+d}, kept
//     in the MFMA accumulators;
//   phase B, bottom-up over the tiles I: wave I forms x_I = D_I^H w_I (the
//     accumulator is the right operand, see k_trsm_reg), stores it and
//     publishes it in LDS; every wave J < I then applies
//     w_J -= L_IJ^H x_I (its operand loaded one step ahead).
// The block's serial chain is S short steps instead of S full tile sweeps.
template <class T, bool RE = false>
__global__ __launch_bounds__(1024) void k_back_big(const Seg* __restrict__ segs, int nseg,
                                                   int64_t total, int nstrip,
                                                   const cx<T>* __restrict__ W,
                                                   cx<T>* __restrict__ X,
                                                   const unsigned long long* __restrict__ flags,
                                                   cx<double>* __restrict__ U, int upd)
{
    using v4 = typename MF<T>::v4;
    __shared__ cx<T> sx[256]; // x_I, row-major 16 x 16
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, kr = lane >> 4, cc = lane & 15;
    const int64_t li = xcd_item();
    const int64_t w = li / nstrip;
    const int u = (int)(li - w * nstrip);
    if (w >= total)
        return;
    const Seg& s = segs[find_seg(segs, nseg, w)];
    const int64_t t = w - s.w0;
    const int p = s.e0 + (int)t * s.es;
    const int m = s.m, k = s.k, d = s.d, S = (m + 15) >> 4;
    const int c0 = 16 * u;
    if (c0 >= k)
        return;
    const int nc = min(16, k - c0);
    const bool hasPrev = p - d >= 0, hasNext = p + d < s.n;
    const int64_t mm = (int64_t)m * m, mk = (int64_t)m * k;
    cx<T>* xp = X + s.ox + (s.xo + s.xs * p) * mk;
    cx<double>* up = upd ? U + s.oU + p * mk : nullptr;
    if (flags[s.sys] != kNoFail) {
        const T nan = T(NAN);
        for (int e = threadIdx.x; e < m * 16; e += blockDim.x)
            if ((e & 15) < nc) {
                const int64_t o = (e >> 4) * k + c0 + (e & 15);
                put_x<T>(xp, up, upd ? 1 : 0, o, cx<T>{nan, nan});
                if (upd && hasNext)
                    put_x<T>(xp, up + d * mk, 1, o, cx<T>{nan, nan});
            }
        return;
    }
    const cx<T>* xm = X + s.ox + (s.xo + s.xs * (p - d)) * mk;
    const cx<T>* xn = X + s.ox + (s.xo + s.xs * (p + d)) * mk;
    if (upd && hasNext) {
        // this strip's columns of the kept neighbour's correction (at most
        // four elements per thread: blockDim = 64 ceil(m / 16)), their loads
        // issued together before the stores
        cx<double>* uq = up + d * mk;
        cx<T> dv[4];
        cx<double> ov[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = threadIdx.x + u * blockDim.x;
            const bool ok = e < m * 16 && (e & 15) < nc;
            const int64_t o = ok ? (e >> 4) * k + c0 + (e & 15) : 0;
            dv[u] = xn[o];
            ov[u] = upd == 2 ? uq[o] : cx<double>{0.0, 0.0};
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = threadIdx.x + u * blockDim.x;
            if (e < m * 16 && (e & 15) < nc)
                uq[(e >> 4) * k + c0 + (e & 15)] =
                    cx<double>{ov[u].r + (double)dv[u].r, ov[u].i + (double)dv[u].i};
        }
    }
    const cx<T>* L = W + s.oL + t * mm;
    const cx<T>* P = W + s.oP + t * mm;
    const cx<T>* Q = W + s.oQ + t * mm;
    const cx<T>* Dg = W + s.oD + t * (int64_t)S * 256;
    const cx<T>* g = W + s.og + t * mk;
    const bool own = wv < S;
    const int r0 = 16 * wv;
    // D_J^H operand of this wave's own tile: (D^H)[cc][rr] = conj(D[rr][cc])
    cx<T> aD[4];
#pragma unroll
    for (int v = 0; v < 4; ++v)
        aD[v] = own ? Dg[wv * 256 + MF<T>::row(kr, v) * 16 + cc] : czero<T>();
    // phase A
    Acc3<T, 1, 1, RE> acc;
    acc.zero();
    if (own && hasPrev)
        wave_mm3<T, 1, 1, false, false, 4, RE>(acc, WOp<T>{Q + (int64_t)r0 * m, m, 1, m - r0},
                                               WOp<T>{xm + c0, 1, k, nc}, m);
    if (own && hasNext)
        wave_mm3<T, 1, 1, false, false, 4, RE>(acc, WOp<T>{P + (int64_t)r0 * m, m, 1, m - r0},
                                               WOp<T>{xn + c0, 1, k, nc}, m);
    v4 wr, wi;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int r = r0 + MF<T>::row(kr, v);
        const cx<T> gv = (own && r < m && cc < nc) ? g[r * k + c0 + cc] : czero<T>();
        wr[v] = gv.r - acc.re(0, 0, v);
        wi[v] = gv.i - acc.im(0, 0, v);
    }
    // operand of the update at step I: A(i, t) = conj(L[16 I + t][r0 + i]),
    // lane (cc, kr) holds t = 4 s + kr for the contraction steps s
    auto load_l = [&](int I, cx<T>(&a)[4]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int row = 16 * I + 4 * q + kr;
            a[q] = (own && wv < I && row < m) ? L[(int64_t)row * m + r0 + cc] : czero<T>();
        }
    };
    cx<T> an[4];
    load_l(S - 1, an);
    // phase B
    for (int I = S - 1; I >= 0; --I) {
        cx<T> a[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            a[q] = an[q];
        if (I > 0)
            load_l(I - 1, an);
        if (wv == I) {
            v4 xr = {0, 0, 0, 0}, xi = {0, 0, 0, 0};
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const cx<T> q = aD[v];
                xr = MF<T>::mma(q.r, wr[v], xr);
                if constexpr (!RE) {
                    xr = MF<T>::mma(q.i, wi[v], xr);
                    xi = MF<T>::mma(q.r, wi[v], xi);
                    xi = MF<T>::mma(-q.i, wr[v], xi);
                }
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int rr = MF<T>::row(kr, v), r = r0 + rr;
                sx[rr * 16 + cc] = cx<T>{xr[v], xi[v]};
                if (r < m && cc < nc)
                    put_x<T>(xp, up, upd, (int64_t)r * k + c0 + cc, cx<T>{xr[v], xi[v]});
            }
        }
        __syncthreads();
        if (wv < I) {
            // w_J -= conj(L_IJ)^T x_I: contraction step q pairs t = 4 q + kr
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const cx<T> b = sx[(4 * q + kr) * 16 + cc];
                const T ar = a[q].r, ai = -a[q].i; // conj(L)
                wr = MF<T>::mma(-ar, b.r, wr);
                if constexpr (!RE) {
                    wr = MF<T>::mma(ai, b.i, wr);
                    wi = MF<T>::mma(-ar, b.i, wi);
                    wi = MF<T>::mma(-ai, b.r, wi);
                }
            }
        }
        __syncthreads();
    }
}

// -------------------------------------------------------------- k_grad_big

// gA_j = -lam_j x_j^H and gB_j = -(lam_{j+1} x_j^H + x_{j+1} lam_j^H), one
// wave per (block row j, 32 x 32 tile); whole-system segments as in k_grad.
template <class T>
__global__ __launch_bounds__(64) void k_grad_big(const Seg* __restrict__ segs, int nseg,
                                                 int64_t total, int ntile,
                                                 const cx<T>* __restrict__ X,
                                                 const cx<T>* __restrict__ Lam,
                                                 cx<T>* __restrict__ gA, cx<T>* __restrict__ gB)
{
    using v4 = typename MF<T>::v4;
    const int lane = threadIdx.x, kr = lane >> 4, cc = lane & 15;
    const int64_t li = xcd_item();
    const int64_t w = li / ntile;
    const int u = (int)(li - w * ntile);
    if (w >= total)
        return;
    const Seg& s = segs[find_seg(segs, nseg, w)];
    const int j = (int)(w - s.w0);
    const int m = s.m, k = s.k, n = s.n, T32 = (m + 31) >> 5;
    if (u >= T32 * T32)
        return;
    const int i0 = 32 * (u / T32), j0 = 32 * (u % T32);
    const int64_t mm = (int64_t)m * m, mk = (int64_t)m * k;
    const cx<T>* l0 = Lam + s.oy + j * mk;
    const cx<T>* x0 = X + s.ox + j * mk;
    v4 cr[2][2], ci[2][2];
    zero_acc<T, 2, 2>(cr, ci);
    wave_mm<T, 2, 2, false, true, 2>(cr, ci, WOp<T>{l0 + (int64_t)i0 * k, k, 1, m - i0},
                                     WOp<T>{x0 + (int64_t)j0 * k, k, 1, m - j0}, k);
    cx<T>* ga = gA + s.oA + j * mm;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = i0 + 16 * a + MF<T>::row(kr, v), c = j0 + 16 * b + cc;
                if (i < m && c < m)
                    ga[i * m + c] = cx<T>{-cr[a][b][v], -ci[a][b][v]};
            }
    if (j + 1 >= n)
        return;
    zero_acc<T, 2, 2>(cr, ci);
    wave_mm<T, 2, 2, false, true, 2>(cr, ci, WOp<T>{l0 + mk + (int64_t)i0 * k, k, 1, m - i0},
                                     WOp<T>{x0 + (int64_t)j0 * k, k, 1, m - j0}, k);
    wave_mm<T, 2, 2, false, true, 2>(cr, ci, WOp<T>{x0 + mk + (int64_t)i0 * k, k, 1, m - i0},
                                     WOp<T>{l0 + (int64_t)j0 * k, k, 1, m - j0}, k);
    cx<T>* gb = gB + s.oB + j * mm;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = i0 + 16 * a + MF<T>::row(kr, v), c = j0 + 16 * b + cc;
                if (i < m && c < m)
                    gb[i * m + c] = cx<T>{-cr[a][b][v], -ci[a][b][v]};
            }
}

} // namespace crs
