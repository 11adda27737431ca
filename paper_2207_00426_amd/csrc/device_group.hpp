// Scan operators spread over a group of 16 lanes (gfx950).
//
// The levels of a scan above the finest hold few elements, so their time is a
// serial chain of operators, and one operator on one lane is ~2700 FP64
// instructions that a lone wave issues at one per ~8 cycles: about 10 us.  Here
// one element is worked on by a DPP row of 16 lanes, four elements to a wave:
// lane r of the lower half (lanes 0-7) holds row r of the upper blocks of the
// Tria matrices, lane 8 + r row r of the lower blocks; a reflecting row is
// broadcast over the 16 lanes with row_newbcast moves, every lane forms the
// reflector from its copy, and each lane applies it to its own row.  Small
// products have one row of the result per lane.  A combine's two last Trias
// ([A_j Tm, U_j] and [A_i^T Xi22, Z_i]) run side by side on the two halves.
// Lanes (l & 7) >= NX carry a copy of row NX - 1 and store nothing.
//
// Operands and results are elements in LDS, all components of one element
// contiguous in the component order of visit(); a call reads every operand
// before it writes, so the output may be an operand's storage.  The arithmetic
// is FP64 also for FP32 scans, whose elements are widened on their way into
// LDS: an FP32 row would be scaled before its reflection, which costs more
// than FP64's rate, and the long spans these levels combine are where FP32
// rounding is worst.
#pragma once

#include <type_traits>

#include "device_ops.hpp"

namespace pss {
namespace grp {

constexpr int kLanes = 16;

// value of x in lane L of this lane's group
template <int L>
__device__ __forceinline__ double bc(double x)
{
    return __longlong_as_double(
        __builtin_amdgcn_update_dpp(0LL, __double_as_longlong(x), 0x150 + L, 0xf, 0xf, true));
}
// lane L for the lower half, lane 8 + L for the upper half (bank mask 0xc:
// the second move writes lanes 8-15 only)
template <int L>
__device__ __forceinline__ double bc2(double x)
{
    const long long v = __double_as_longlong(x);
    const long long lo = __builtin_amdgcn_update_dpp(0LL, v, 0x150 + L, 0xf, 0xf, true);
    return __longlong_as_double(__builtin_amdgcn_update_dpp(lo, v, 0x150 + 8 + L, 0xf, 0xc, false));
}

// compile-time loop: f(integral_constant<int, i>) for i in [0, N)
template <int N, int I = 0, class Fn>
__device__ __forceinline__ void each(Fn &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        each<N, I + 1>(f);
    }
}

// orders one wave's LDS accesses across its lanes (LDS operations of a wave
// complete in order; this keeps the compiler from moving them)
__device__ __forceinline__ void lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <int NX>
struct Lane {
    int r;       // row
    bool hi;     // upper half
    bool stores; // holds a row of its own
    __device__ __forceinline__ Lane()
    {
        const int l = threadIdx.x & (kLanes - 1), q = l & 7;
        hi = l >= 8;
        stores = q < NX;
        r = q < NX ? q : NX - 1;
    }
};

// one sweep of pss::lq_rows over the group: row is this lane's, rho its
// logical index; row i of the matrix sits in lane i (Two: and, for the upper
// half's own matrix, in lane 8 + i).  inv[i] receives 1 / L[i][i].
template <int K, int Z0, bool Two, typename T, int C>
__device__ __forceinline__ void lq(T (&row)[C], int rho, T (&inv)[K])
{
    each<K>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        constexpr int jend = cmin(C, Z0 + i + 1);
        T x[C];
#pragma unroll
        for (int j = i; j < jend; ++j) {
            if constexpr (Two)
                x[j] = bc2<i>(row[j]);
            else
                x[j] = bc<i>(row[j]);
        }
        T sig = T(0);
#pragma unroll
        for (int j = i + 1; j < jend; ++j)
            sig = pfma(x[j], x[j], sig);
        const Reflector<T> h(x[i], sig);
        inv[i] = h.q;
        // every row takes the reflection: on a row that is already reduced it
        // reaches only columns right of that row's diagonal, which are stale
        h.row(row, x, i, jend);
        row[i] = rho == i ? h.d : row[i];
    });
}

// component offsets of the element types (the order of visit())
template <int NX>
struct FOff {
    static constexpr int A = 0, b = NX * NX, U = b + NX, eta = U + tri_size(NX), Z = eta + NX;
};
template <int NX>
struct SOff {
    static constexpr int E = 0, g = NX * NX, D = g + NX;
};
template <int NX>
struct MOff {
    static constexpr int m = 0, N = NX;
};

// L[t][r] for t >= r, else 0 (column r of a packed lower factor), and row r
template <int NX, typename T>
__device__ __forceinline__ void lower_col(const T *L, int r, T (&c)[NX])
{
#pragma unroll
    for (int t = 0; t < NX; ++t) {
        const T v = L[t * (t + 1) / 2 + (t < r ? t : r)];
        c[t] = t >= r ? v : T(0);
    }
}
template <int NX, typename T>
__device__ __forceinline__ void lower_row(const T *L, int r, T *c)
{
#pragma unroll
    for (int j = 0; j < NX; ++j) {
        const T v = L[r * (r + 1) / 2 + (j < r ? j : r)];
        c[j] = j <= r ? v : T(0);
    }
}

// q = eta_j - Z_j Z_j^T m and the upper Xi row [U^T Z_j, I] of row r, shared
// by the combine and the apply form.  Zj: all of Z_j; uc: column r of U.
template <int NX, typename T>
__device__ __forceinline__ void xi_front(const T *ej, const T *m, const T (&uc)[NX], int r,
                                         T (&q)[NX], T (&zt)[NX], T (&row)[2 * NX])
{
    using O = FOff<NX>;
    T Zj[NX][NX];
#pragma unroll
    for (int t = 0; t < NX; ++t)
#pragma unroll
        for (int a = 0; a <= t; ++a)
            Zj[t][a] = ej[O::Z + tri_idx(t, a)];
#pragma unroll
    for (int a = 0; a < NX; ++a) {
        T s = Zj[a][a] * m[a];
#pragma unroll
        for (int i = a + 1; i < NX; ++i)
            s = pfma(Zj[i][a], m[i], s);
        zt[a] = s;
    }
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        T s = Zj[i][0] * zt[0];
#pragma unroll
        for (int a = 1; a <= i; ++a)
            s = pfma(Zj[i][a], zt[a], s);
        q[i] = ej[O::eta + i] - s;
    }
#pragma unroll
    for (int a = 0; a < NX; ++a) {
        T s = uc[a] * Zj[a][a];
#pragma unroll
        for (int t = a + 1; t < NX; ++t)
            s = pfma(uc[t], Zj[t][a], s);
        row[a] = s;
        row[NX + a] = a == r ? T(1) : T(0);
    }
}

// Tm = U Xi11^{-T}: row r from row r of U; then all of Tm in every lane
template <int NX, typename T>
__device__ __forceinline__ void tm_rows(const T (&row)[2 * NX], const T (&inv)[NX],
                                        const T (&ur)[NX], T (&Tm)[NX], T (&TF)[NX][NX])
{
    T X11[NX][NX];
    each<NX>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
#pragma unroll
        for (int j = 0; j < i; ++j)
            X11[i][j] = bc<i>(row[j]);
    });
#pragma unroll
    for (int j = 0; j < NX; ++j) {
        T s = ur[j];
#pragma unroll
        for (int t = 0; t < j; ++t)
            s = pfma(-Tm[t], X11[j][t], s);
        Tm[j] = s * inv[j];
    }
    each<NX>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
#pragma unroll
        for (int j = 0; j < NX; ++j)
            TF[i][j] = bc<i>(Tm[j]);
    });
}

// Table 3 (filter_combine_v): o = e_i (x) e_j
template <typename T, int NX>
__device__ __forceinline__ void filter_combine(const T *ei, const T *ej, T *o,
                                               const Lane<NX> &ln)
{
    using O = FOff<NX>;
    const int r = ln.r;
    T q[NX], zt[NX], row[2 * NX], bi[NX], zr[NX];
    {
        T uc[NX];
        lower_col<NX>(ei + O::U, r, uc);
#pragma unroll
        for (int i = 0; i < NX; ++i)
            bi[i] = ei[O::b + i];
        xi_front<NX>(ej, bi, uc, r, q, zt, row);
    }
    lower_row<NX>(ej + O::Z, r, zr);
    // the upper half holds the lower Xi rows [Z_j, 0]
#pragma unroll
    for (int a = 0; a < NX; ++a) {
        row[a] = ln.hi ? zr[a] : row[a];
        row[NX + a] = ln.hi ? T(0) : row[NX + a];
    }
    T inv[NX];
    lq<NX, NX, false>(row, ln.hi ? NX : r, inv);
    T Tm[NX], TF[NX][NX], ur[NX];
    lower_row<NX>(ei + O::U, r, ur);
    tm_rows<NX>(row, inv, ur, Tm, TF);
    lds_order(); // what follows is read when it is needed, not before the sweep
    // tq = Tm^T q; v_r = b_i + Tm tq (filtered mean of the span's start)
    T tq[NX], v = ei[O::b + r];
#pragma unroll
    for (int a = 0; a < NX; ++a) {
        T s = TF[0][a] * q[0];
#pragma unroll
        for (int t = 1; t < NX; ++t)
            s = pfma(TF[t][a], q[t], s);
        tq[a] = s;
    }
#pragma unroll
    for (int a = 0; a < NX; ++a)
        v = pfma(Tm[a], tq[a], v);
    // upper half: gq = G^T q = q - Xi21 tq, row r
    T gq = ej[O::eta + r];
#pragma unroll
    for (int a = 0; a < NX; ++a) {
        gq = pfma(-zr[a], zt[a], gq);
        gq = pfma(-row[a], tq[a], gq);
    }
    T Aj[NX], Ac[NX]; // row r of A_j, column r of A_i
#pragma unroll
    for (int t = 0; t < NX; ++t) {
        Aj[t] = ej[O::A + r * NX + t];
        Ac[t] = ei[O::A + t * NX + r];
    }
    // lower half: A_j Tm (row r); upper half: A_i^T Xi22 (row r)
    T AT[NX], w2[2 * NX];
#pragma unroll
    for (int j = 0; j < NX; ++j) {
        T s = Aj[0] * TF[0][j];
#pragma unroll
        for (int t = 1; t < NX; ++t)
            s = pfma(Aj[t], TF[t][j], s);
        AT[j] = s;
        w2[j] = T(0);
    }
    T AG[NX]; // A_j G = A_j - A_j Tm Xi21^T
    T ob = ej[O::b + r], oe = ei[O::eta + r];
    each<NX>([&](auto ic) {
        constexpr int t = decltype(ic)::value;
#pragma unroll
        for (int c = 0; c < NX; ++c)
            w2[c] = pfma(Ac[t], bc<8 + t>(row[NX + c]), w2[c]);
        T s = Aj[t];
#pragma unroll
        for (int a = 0; a < NX; ++a)
            s = pfma(-AT[a], bc<8 + t>(row[a]), s);
        AG[t] = s;
        ob = pfma(Aj[t], bc<t>(v), ob);
        oe = pfma(Ac[t], bc<8 + t>(gq), oe);
    });
    // U = Tria([A_j Tm, U_j]) below, Z = Tria([A_i^T Xi22, Z_i]) above
    {
        const T *L = ln.hi ? ei + O::Z : ej + O::U;
#pragma unroll
        for (int j = 0; j < NX; ++j)
            w2[j] = ln.hi ? w2[j] : AT[j];
        lower_row<NX>(L, r, w2 + NX);
    }
    lds_order();
    T An[NX];
#pragma unroll
    for (int j = 0; j < NX; ++j)
        An[j] = T(0);
#pragma unroll
    for (int t = 0; t < NX; ++t)
#pragma unroll
        for (int j = 0; j < NX; ++j)
            An[j] = pfma(AG[t], ei[O::A + t * NX + j], An[j]);
    lq<NX, NX, true>(w2, r, inv);
    lds_order();
    if (ln.stores) {
        T *F = o + (ln.hi ? O::Z : O::U) + r * (r + 1) / 2;
#pragma unroll
        for (int j = 0; j < NX; ++j)
            if (j <= r)
                F[j] = w2[j];
        if (ln.hi) {
            o[O::eta + r] = oe;
        } else {
            o[O::b + r] = ob;
#pragma unroll
            for (int j = 0; j < NX; ++j)
                o[O::A + r * NX + j] = An[j];
        }
    }
    lds_order();
}

// Table 3 with a true prefix on the left (filter_apply_v): o = p (x) e_j, both
// marginals
template <typename T, int NX>
__device__ __forceinline__ void filter_apply(const T *p, const T *ej, T *o, const Lane<NX> &ln)
{
    using O = FOff<NX>;
    using M = MOff<NX>;
    const int r = ln.r;
    T q[NX], zt[NX], row[2 * NX], inv[NX], Tm[NX], TF[NX][NX];
    {
        T uc[NX], m[NX];
        lower_col<NX>(p + M::N, r, uc);
#pragma unroll
        for (int i = 0; i < NX; ++i)
            m[i] = p[M::m + i];
        xi_front<NX>(ej, m, uc, r, q, zt, row);
    }
    lq<NX, NX, false>(row, r, inv);
    T ur[NX];
    lower_row<NX>(p + M::N, r, ur);
    tm_rows<NX>(row, inv, ur, Tm, TF);
    T v = p[M::m + r];
#pragma unroll
    for (int a = 0; a < NX; ++a) {
        T s = TF[0][a] * q[0];
#pragma unroll
        for (int t = 1; t < NX; ++t)
            s = pfma(TF[t][a], q[t], s);
        v = pfma(Tm[a], s, v);
    }
    T w2[2 * NX], ob = ej[O::b + r];
#pragma unroll
    for (int j = 0; j < NX; ++j)
        w2[j] = T(0);
    each<NX>([&](auto ic) {
        constexpr int t = decltype(ic)::value;
        const T a = ej[O::A + r * NX + t];
#pragma unroll
        for (int j = 0; j < NX; ++j)
            w2[j] = pfma(a, TF[t][j], w2[j]);
        ob = pfma(a, bc<t>(v), ob);
    });
    lower_row<NX>(ej + O::U, r, w2 + NX);
    lq<NX, NX, false>(w2, r, inv);
    lds_order();
    if (ln.stores && !ln.hi) {
        o[M::m + r] = ob;
        T *F = o + M::N + r * (r + 1) / 2;
#pragma unroll
        for (int j = 0; j < NX; ++j)
            if (j <= r)
                F[j] = w2[j];
    }
    lds_order();
}

// Table 5 (smoother_combine_v): o = {E_i E_j, E_i g_j + g_i, Tria([E_i D_j, D_i])}
template <typename T, int NX>
__device__ __forceinline__ void smoother_combine(const T *ei, const T *ej, T *o,
                                                 const Lane<NX> &ln)
{
    using O = SOff<NX>;
    const int r = ln.r;
    T w[2 * NX], EE[NX], g = ei[O::g + r], inv[NX];
#pragma unroll
    for (int j = 0; j < NX; ++j)
        w[j] = EE[j] = T(0);
#pragma unroll
    for (int t = 0; t < NX; ++t) {
        const T a = ei[O::E + r * NX + t];
        g = pfma(a, ej[O::g + t], g);
#pragma unroll
        for (int j = 0; j < NX; ++j) {
            EE[j] = pfma(a, ej[O::E + t * NX + j], EE[j]);
            if (j <= t)
                w[j] = pfma(a, ej[O::D + tri_idx(t, j)], w[j]);
        }
    }
    lower_row<NX>(ei + O::D, r, w + NX);
    lq<NX, NX, false>(w, r, inv);
    lds_order();
    if (ln.stores && !ln.hi) {
        o[O::g + r] = g;
        T *F = o + O::D + r * (r + 1) / 2;
#pragma unroll
        for (int j = 0; j < NX; ++j) {
            o[O::E + r * NX + j] = EE[j];
            if (j <= r)
                F[j] = w[j];
        }
    }
    lds_order();
}

// Table 5 with a true suffix on the right (smoother_apply_v)
template <typename T, int NX>
__device__ __forceinline__ void smoother_apply(const T *ei, const T *s, T *o, const Lane<NX> &ln)
{
    using O = SOff<NX>;
    using M = MOff<NX>;
    const int r = ln.r;
    T w[2 * NX], m = ei[O::g + r], inv[NX];
#pragma unroll
    for (int j = 0; j < NX; ++j)
        w[j] = T(0);
#pragma unroll
    for (int t = 0; t < NX; ++t) {
        const T a = ei[O::E + r * NX + t];
        m = pfma(a, s[M::m + t], m);
#pragma unroll
        for (int j = 0; j <= t; ++j)
            w[j] = pfma(a, s[M::N + tri_idx(t, j)], w[j]);
    }
    lower_row<NX>(ei + O::D, r, w + NX);
    lq<NX, NX, false>(w, r, inv);
    lds_order();
    if (ln.stores && !ln.hi) {
        o[M::m + r] = m;
        T *F = o + M::N + r * (r + 1) / 2;
#pragma unroll
        for (int j = 0; j < NX; ++j)
            if (j <= r)
                F[j] = w[j];
    }
    lds_order();
}

// shared by the two forms of the adjoint map below: a = Phi^T m2 + u (row r)
// and row r (j <= r) of Phi^T S2 Phi + sym((Phi^T m2) u^T) + Gam, for the map
// t = {Phi, u, Gam} (stored as {E, g, D}) and (m2, S2 = packed symmetric)
template <typename T, int NX>
__device__ __forceinline__ void adj_rows(const T *t, const T *m2, const T *S2,
                                         const Lane<NX> &ln, T &a, T (&row)[NX])
{
    using O = SOff<NX>;
    const int r = ln.r;
    T P[NX][NX], af[NX], X[NX], ar = T(0), pc[NX];
#pragma unroll
    for (int q = 0; q < NX; ++q) {
        af[q] = X[q] = T(0);
#pragma unroll
        for (int j = 0; j < NX; ++j)
            P[q][j] = t[O::E + q * NX + j];
    }
#pragma unroll
    for (int q = 0; q < NX; ++q) {
        const T mq = m2[q], sq = S2[q < r ? r * (r + 1) / 2 + q : q * (q + 1) / 2 + r];
        pc[q] = t[O::E + q * NX + r];
        ar = pfma(pc[q], mq, ar);
#pragma unroll
        for (int j = 0; j < NX; ++j) {
            af[j] = pfma(P[q][j], mq, af[j]);
            X[j] = pfma(sq, P[q][j], X[j]); // row r of S2 Phi
        }
    }
    const T ur = t[O::g + r];
#pragma unroll
    for (int j = 0; j < NX; ++j) {
        T s = t[O::D + r * (r + 1) / 2 + (j < r ? j : r)];
        s = pfma(T(0.5) * ar, t[O::g + j], s);
        row[j] = pfma(T(0.5) * ur, af[j], s);
    }
    each<NX>([&](auto ic) {
        constexpr int q = decltype(ic)::value;
#pragma unroll
        for (int j = 0; j < NX; ++j)
            row[j] = pfma(pc[q], bc<q>(X[j]), row[j]);
    });
    a = ar + ur;
}

// adj_combine_v: o = t1 o t2, t2 applied first
template <typename T, int NX>
__device__ __forceinline__ void adj_combine(const T *t1, const T *t2, T *o, const Lane<NX> &ln)
{
    using O = SOff<NX>;
    const int r = ln.r;
    T a, row[NX], PP[NX];
    adj_rows<T, NX>(t1, t2 + O::g, t2 + O::D, ln, a, row);
#pragma unroll
    for (int j = 0; j < NX; ++j)
        PP[j] = T(0);
#pragma unroll
    for (int q = 0; q < NX; ++q) {
        const T p2 = t2[O::E + r * NX + q];
#pragma unroll
        for (int j = 0; j < NX; ++j)
            PP[j] = pfma(p2, t1[O::E + q * NX + j], PP[j]);
    }
    lds_order();
    if (ln.stores && !ln.hi) {
        o[O::g + r] = a;
        T *D = o + O::D + r * (r + 1) / 2;
#pragma unroll
        for (int j = 0; j < NX; ++j) {
            o[O::E + r * NX + j] = PP[j];
            if (j <= r)
                D[j] = row[j];
        }
    }
    lds_order();
}

// adj_apply_v: o = t(lam), lam = (m_bar, packed P_bar)
template <typename T, int NX>
__device__ __forceinline__ void adj_apply(const T *t, const T *lam, T *o, const Lane<NX> &ln)
{
    using M = MOff<NX>;
    const int r = ln.r;
    T a, row[NX];
    adj_rows<T, NX>(t, lam + M::m, lam + M::N, ln, a, row);
    lds_order();
    if (ln.stores && !ln.hi) {
        o[M::m + r] = a;
        T *D = o + M::N + r * (r + 1) / 2;
#pragma unroll
        for (int j = 0; j < NX; ++j)
            if (j <= r)
                D[j] = row[j];
    }
    lds_order();
}

} // namespace grp
} // namespace pss
