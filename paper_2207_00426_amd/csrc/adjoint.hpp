// Adjoint (reverse-mode) pass of the square-root filter's pseudo-log-
// likelihood: the VJP of the filter scan as a reverse associative scan of
// affine cotangent maps (device_adj.hpp) and the per-step VJP with respect to
// the linearisation Gamma_k (Section 5.2, eq. gradient, at a frozen nominal).
// In FP64 its finest level works on the tiles of steps.hpp, a thread on E
// consecutive steps:
//   k_filter_walk  filters from the marginal before the thread's first step;
//                  writes the log-likelihood terms, the filtering marginals,
//                  and the aggregate of its cotangent maps, each on request
//   k_adj_down     from the cotangent of the state after its last step back to
//                  its first: every step's cotangents and the prior's
// In FP32, whose marginals and linearisation are in the plain layout, it is a
// tile scan (AdjSrc): threads that read E numbers apart gain nothing from longer
// runs of steps, and its in-tile tree leaves the levels above 64 times fewer
// elements.  (Backward pass of 64 x 10^4 steps 340 us, of 300 x 600 222; with 2
// steps folded a thread and no tree 449 and 281.)
#pragma once

#include "device_adj.hpp"
#include "steps.hpp"

namespace pss {

// Reverse scan of the cotangent maps T_k, run as a forward scan over the
// time-reversed maps (scan position p holds T_{n-p}); a scan prefix covers
// later times and composes as "later map first".  Elements use the smoother
// element's storage (E <- Phi, g <- u, D <- Gam), prefixes the marginal's
// (m <- m_bar, N <- P_bar, both lower triangles of symmetric matrices).
template <typename T_, int NX_>
struct AdjScan {
    using T = T_;
    static constexpr int NX = NX_;
    using Elem = SElem<T, NX>;
    using Pre = Marg<T, NX>;
    static constexpr int NE = Sizes<NX>::selem;
    static constexpr int NP = Sizes<NX>::marg;
    static constexpr const char *name = "adjoint";
    PSS_INL static SSlotV<T, NX, int> slot(T *lds, int Tb, int s)
    {
        return SSlotV<T, NX, int>{lds + s, Tb};
    }
    PSS_INL static SRegV<T, NX> reg(Elem &e) { return SRegV<T, NX>{&e}; }
    template <int NZ = NX, class VA, class VB, class VO>
    PSS_INL static void combine_v(const VA &a, const VB &b, const VO &o)
    {
        adj_combine_v<T, NX>(b, a, o);
    }
    template <int NZ = NX, class VA>
    PSS_INL static void apply_v(const Pre &p, const VA &a, Pre &o)
    {
        adj_apply_v<T, NX>(a, p, o);
    }
    template <class VS, class VD>
    PSS_INL static void copy_v(const VS &src, const VD &dst)
    {
        selem_copy<T, NX>(src, dst);
    }
};

template <typename T, int NX>
struct GroupOp<AdjScan<T, NX>> {
    static constexpr bool value = NX >= 2;
    using Ref = SAosRef<T, NX>;
    static __device__ __forceinline__ void combine(const double *a, const double *b, double *o,
                                                   const grp::Lane<NX> &ln)
    {
        grp::adj_combine<double, NX>(b, a, o, ln);
    }
    static __device__ __forceinline__ void apply(const double *p, const double *a, double *o,
                                                 const grp::Lane<NX> &ln)
    {
        grp::adj_apply<double, NX>(a, p, o, ln);
    }
};

// theta contraction of the coordinated-turn model: dl/dtheta_j =
// sum_k tr(Lam_bar_k dQ/dtheta_j) + tr(Om_bar_k dR/dtheta_j) with
// dQ/dlog q1 = q1 Qv, dQ/dlog q2 = q2 Qw, dR/dlog sigma = 2 sigma^2 I.
template <typename T, int NX>
struct AdjTheta {
    T dQ1[NX][NX];
    T dQ2[NX][NX];
    T dR;
};

// output of the step VJP: per-step theta terms (terms[c * T_y + t], FP64)
template <typename T, int NX, int NY>
struct ThetaOut {
    static constexpr bool kGamma = false;
    AdjTheta<T, NX> th;
    double *terms; // at the steps' interleaved slots
    int64_t T_y;
};

// output of the step VJP: the cotangent of every input of the step in the
// library's representation (pss_gamma fields at step slot t, factors as
// packed lower triangles), scaled by the sequence's cotangent w_b
template <typename T, int NX, int NY>
struct GammaOut {
    static constexpr bool kGamma = true;
    GammaRef<T, NX, NY> bar; // stride 1, ld = T_y
    const double *w;         // [B] or null (ones)
    int ilv;                 // at interleaved slots instead of plain ones
};

// cotangents of one step, given the cotangent lam of its filtering marginal
// and the step's quantities q, Np = N^-, P22 P22^T = P_k, mp = m^-; t: the
// step's slot in the output
template <typename T, int NX, int NY>
PSS_INL void adj_emit(const ThetaOut<T, NX, NY> &out, int b, int64_t t, const T (&F)[NX][NX],
                      const T (&SL)[NX][NX], const T (&H)[NY][NX], const T (&SO)[NY][NY],
                      const Marg<T, NX> &f, const StepQ<T, NX, NY> &q, const T (&Np)[NX][NX],
                      const T (&P22)[NX][NX], const T (&mp)[NX], const Marg<T, NX> &lam)
{
    T Lb[NX][NX], Ob[NY][NY], cb[NX], db[NY];
    adj_gram_bars(H, q, lam, Lb, Ob, cb, db);
    double g1 = 0.0, g2 = 0.0, g3 = 0.0;
#pragma unroll
    for (int i = 0; i < NX; ++i)
#pragma unroll
        for (int j = 0; j < NX; ++j) {
            g1 += (double)(Lb[i][j] * out.th.dQ1[i][j]);
            g2 += (double)(Lb[i][j] * out.th.dQ2[i][j]);
        }
#pragma unroll
    for (int a = 0; a < NY; ++a)
        g3 += (double)(Ob[a][a] * out.th.dR);
    out.terms[t] = g1;
    out.terms[out.T_y + t] = g2;
    out.terms[2 * out.T_y + t] = g3;
}

template <typename T, int NX, int NY>
PSS_INL void adj_emit(const GammaOut<T, NX, NY> &out, int b, int64_t t, const T (&F)[NX][NX],
                      const T (&SL)[NX][NX], const T (&H)[NY][NX], const T (&SO)[NY][NY],
                      const Marg<T, NX> &f, const StepQ<T, NX, NY> &q, const T (&Np)[NX][NX],
                      const T (&P22)[NX][NX], const T (&mp)[NX], const Marg<T, NX> &lam)
{
    T Lb[NX][NX], Ob[NY][NY], cb[NX], db[NY];
    adj_gram_bars(H, q, lam, Lb, Ob, cb, db);
    const T w = out.w ? (T)out.w[b] : T(1);
    // Sl = (W v v^T W - W) / 2
    T Sl[NY][NY];
#pragma unroll
    for (int a = 0; a < NY; ++a)
#pragma unroll
        for (int b = 0; b <= a; ++b) {
            T s = T(0);
#pragma unroll
            for (int u = a; u < NY; ++u)
                s = pfma(q.Yi[u][a], q.Yi[u][b], s);
            Sl[a][b] = Sl[b][a] = T(0.5) * (q.Wv[a] * q.Wv[b] - s);
        }
    // factor cotangents of S_L and S_O: lower triangles of 2 G_bar S
    T SLb[NX][NX], SOb[NY][NY];
    mm_lower(Lb, SL, SLb);
    mm_lower(Ob, SO, SOb);
    // F_bar = c_bar m^T + 2 Lam_bar F N N^T
    T Fb[NX][NX];
    {
        T FN[NX][NX], X[NX][NX];
        mm_lower(F, f.N, FN);
        mm(Lb, FN, X);
#pragma unroll
        for (int i = 0; i < NX; ++i)
#pragma unroll
            for (int j = 0; j < NX; ++j) {
                T s = cb[i] * f.m[j];
#pragma unroll
                for (int u = 0; u <= j; ++u)
                    s = pfma(T(2) * X[i][u], f.N[j][u], s);
                Fb[i][j] = s;
            }
    }
    // H_bar = 2 Sl H P^- + W v (m^- + P_k m_bar)^T - (K^T m_bar) m_k^T
    //         - 2 K^T P_bar P_k,  P^- = Np Np^T, P_k = P22 P22^T,
    //         m_k = m^- + K v with v = Y w
    T Hb[NY][NX];
    {
        T Pm[NX][NX], Pk[NX][NX], Pb[NX][NX], kb[NY], mk[NX], pm[NX];
        sym_from_lower(Pm, [&](int i, int j) {
            T s = T(0);
            for (int u = 0; u <= j; ++u)
                s = pfma(Np[i][u], Np[j][u], s);
            return s;
        });
        sym_from_lower(Pk, [&](int i, int j) {
            T s = T(0);
            for (int u = 0; u < NX; ++u)
                s = pfma(P22[i][u], P22[j][u], s);
            return s;
        });
        sym_from_lower(Pb, [&](int i, int j) { return lam.N[i][j]; });
        mtv(q.K, lam.m, kb);
        // K v = Psi21 w (K = Psi21 Y^{-1}) -- recovered as K (Y w)
        T v[NY];
#pragma unroll
        for (int a = 0; a < NY; ++a) {
            // Y = Yi^{-1}: solve Yi v = w
            T s = q.w[a];
#pragma unroll
            for (int u = 0; u < a; ++u)
                s = pfma(-q.Yi[a][u], v[u], s);
            v[a] = s * prcp(q.Yi[a][a]);
        }
        mv(Pk, lam.m, pm);
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            T s = mp[i];
#pragma unroll
            for (int a = 0; a < NY; ++a)
                s = pfma(q.K[i][a], v[a], s);
            mk[i] = s;
        }
        T SH[NY][NX], KP[NY][NX];
        mm(Sl, H, SH);
#pragma unroll
        for (int a = 0; a < NY; ++a)
#pragma unroll
            for (int j = 0; j < NX; ++j) {
                T s = T(0);
#pragma unroll
                for (int u = 0; u < NX; ++u)
                    s = pfma(q.K[u][a], Pb[u][j], s);
                KP[a][j] = s;
            }
#pragma unroll
        for (int a = 0; a < NY; ++a)
#pragma unroll
            for (int j = 0; j < NX; ++j) {
                T s = q.Wv[a] * (mp[j] + pm[j]) - kb[a] * mk[j];
#pragma unroll
                for (int u = 0; u < NX; ++u) {
                    s = pfma(T(2) * SH[a][u], Pm[u][j], s);
                    s = pfma(T(-2) * KP[a][u], Pk[u][j], s);
                }
                Hb[a][j] = s;
            }
    }
    // scale by the sequence's cotangent and store
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        cb[i] *= w;
#pragma unroll
        for (int j = 0; j < NX; ++j) {
            Fb[i][j] *= w;
            SLb[i][j] *= T(2) * w;
        }
    }
#pragma unroll
    for (int a = 0; a < NY; ++a) {
        db[a] *= w;
#pragma unroll
        for (int j = 0; j < NX; ++j)
            Hb[a][j] *= w;
#pragma unroll
        for (int j = 0; j < NY; ++j)
            SOb[a][j] *= T(2) * w;
    }
    out.bar.store_trans(t, Fb, cb, SLb);
    out.bar.store_obs(t, Hb, db, SOb);
}

// cotangent of the prior (m0, P0) from lambda_0, per sequence: m0_bar [NX][B],
// N0_bar [P][B] = lower triangle of 2 P0_bar N0, scaled by w_b; m0_bar null:
// not wanted
template <typename T, int NX>
struct AdjPrior {
    T *m0_bar;
    T *N0_bar;
    const T *N0; // packed prior factor
    const double *w;
    int B;
    PSS_INL void put(int b, const Marg<T, NX> &lam) const
    {
        if (!m0_bar)
            return;
        const T s = w ? (T)w[b] : T(1);
        T Pb[NX][NX], L[NX][NX];
        sym_from_lower(Pb, [&](int i, int j) { return lam.N[i][j]; });
#pragma unroll
        for (int i = 0; i < NX; ++i)
#pragma unroll
            for (int j = 0; j < NX; ++j)
                L[i][j] = (j <= i) ? N0[tri_idx(i, j)] : T(0);
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            m0_bar[(int64_t)i * B + b] = s * lam.m[i];
#pragma unroll
            for (int j = 0; j <= i; ++j) {
                T a = T(0);
#pragma unroll
                for (int u = j; u < NX; ++u)
                    a = pfma(Pb[i][u], L[u][j], a);
                N0_bar[(int64_t)tri_idx(i, j) * B + b] = T(2) * s * a;
            }
        }
    }
};

// The thread's start is its level-1 prefix (pre), or with `have` the stored
// marginal of its first state.  marg (m null: not written) receives the
// filtering marginal of state k at the interleaved slot of step k + 1; ell
// (nullable) the log-likelihood terms at the interleaved slots.  ADJ: the maps
// T_k folded into an element of the adjoint scan's level 1 (scanned backwards).
template <typename T, int NX, int NY, bool ADJ, class AggRef, class PreRef>
__global__ __launch_bounds__(256) void k_filter_walk(StepGeom g, GammaRef<T, NX, NY> gam,
                                                     const T *y, int64_t T_y,
                                                     StepPrior<T, NX> prior, PreRef pre,
                                                     MargRef<T, NX> have, MargRef<T, NX> marg,
                                                     double *ell, AggRef agg,
                                                     const int64_t *next_off, int nT, int nE)
{
    const TileInfo ti = tile_info(g);
    if ((int)threadIdx.x >= ti.nvalid)
        return;
    const int64_t p0 = ti.start + (int64_t)threadIdx.x * ti.E;
    int64_t pe = p0 + ti.E;
    if (pe > ti.start + ti.tcnt)
        pe = ti.start + ti.tcnt;
    const int64_t v = ti.start / ti.E + threadIdx.x, cnt1 = next_off[ti.b + 1] - next_off[ti.b];
    Marg<T, NX> f;
    if (p0 == 0) {
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            f.m[i] = prior.m0[i];
#pragma unroll
            for (int j = 0; j <= i; ++j)
                f.N[i][j] = prior.N0[tri_idx(i, j)];
        }
    } else if (have.m) {
        have.load(ilv_slot(ti, p0), f);
    } else {
        pre.load(next_off[ti.b] + v, f);
    }
    SElem<T, NX> a;
    for (int64_t p = p0; p < pe; ++p) {
        const int64_t u = ilv_slot(ti, p), ug = gam.stride ? u : 0;
        if (marg.m)
            marg.store(u, f);
        T F[NX][NX], M[NX][2 * NX], mp[NX];
#pragma unroll
        for (int i = 0; i < NX; ++i)
#pragma unroll
            for (int j = 0; j < NX; ++j)
                F[i][j] = gam.F[(i * NX + j) * gam.ld + ug];
        mv(F, f.m, mp);
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            mp[i] += gam.c[i * gam.ld + ug];
#pragma unroll
            for (int j = 0; j < NX; ++j) {
                T s = F[i][j] * f.N[j][j];
#pragma unroll
                for (int t = j + 1; t < NX; ++t)
                    s = pfma(F[i][t], f.N[t][j], s);
                M[i][j] = s;
                M[i][NX + j] = j <= i ? gam.SL[tri_idx(i, j <= i ? j : i) * gam.ld + ug] : T(0);
            }
        }
        lq_rows<NX, NX>(M);
        T H[NY][NX], d[NY], SO[NY][NY];
        gam.load_obs(ug, H, d, SO);
        T Q[NY + NX][NX + NY], w[NY][1];
        step_update(H, M, SO, Q);
#pragma unroll
        for (int q = 0; q < NY; ++q) {
            T s = y[q * T_y + ti.off + p] - d[q];
#pragma unroll
            for (int j = 0; j < NX; ++j)
                s = pfma(-H[q][j], mp[j], s);
            w[q][0] = s;
        }
        step_solve<T, NY, 1>(Q, w);
        if (ell) {
            double l = -0.5 * NY * 1.8378770664093454835606594728112; // log(2 pi)
#pragma unroll
            for (int q = 0; q < NY; ++q)
                l -= (double)plog(Q[q][q]) + 0.5 * (double)w[q][0] * (double)w[q][0];
            ell[u] = l;
        }
        if constexpr (ADJ) {
            // T_k = {Phi = F - P21 G, u = G^T w, Gam = (u u^T - G^T G) / 2},
            // G = Y^{-1} H F
            T G[NY][NX];
            mm(H, F, G);
            step_solve<T, NY, NX>(Q, G);
            SElem<T, NX> e;
#pragma unroll
            for (int i = 0; i < NX; ++i) {
                T uu = T(0);
#pragma unroll
                for (int q = 0; q < NY; ++q)
                    uu = pfma(G[q][i], w[q][0], uu);
                e.g[i] = uu;
#pragma unroll
                for (int j = 0; j < NX; ++j) {
                    T s = F[i][j];
#pragma unroll
                    for (int q = 0; q < NY; ++q)
                        s = pfma(-Q[NY + i][q], G[q][j], s);
                    e.E[i][j] = s;
                }
            }
#pragma unroll
            for (int i = 0; i < NX; ++i)
#pragma unroll
                for (int j = 0; j <= i; ++j) {
                    T s = e.g[i] * e.g[j];
#pragma unroll
                    for (int q = 0; q < NY; ++q)
                        s = pfma(-G[q][i], G[q][j], s);
                    e.D[i][j] = T(0.5) * s;
                }
            if (p == p0)
                a = e;
            else
                adj_combine_v<T, NX>(SRegV<T, NX>{&a}, SRegV<T, NX>{&e}, SRegV<T, NX>{&a});
        }
        // the factor is made triangular at every step, stored or not: a
        // gradient that starts from stored marginals repeats this arithmetic
        T P22[NX][NX];
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            f.m[i] = mp[i];
#pragma unroll
            for (int q = 0; q < NY; ++q)
                f.m[i] = pfma(Q[NY + i][q], w[q][0], f.m[i]);
#pragma unroll
            for (int j = 0; j < NX; ++j)
                P22[i][j] = Q[NY + i][NY + j];
        }
        tria_rect(P22, f.N);
    }
    if constexpr (ADJ)
        selem_copy<T, NX>(SRegV<T, NX>{&a},
                          view_of(agg, agg_slot(next_off, ti.b, cnt1 - 1 - v, nT, nE)));
}

// FP32: element p of sequence b at the finest level is the map of step k = n - p,
// built from the filtering marginal of state k - 1 and Gamma at step slot y_off[b]
// + k - 1; down_apply also emits the step's cotangents with the suffix lambda_k
template <typename T, int NX, int NY, class Out>
struct AdjSrc {
    static constexpr bool lazy_up = false, lazy_down = false, fused_down = true;
    static constexpr int leaf_nz = 0;
    GammaRef<T, NX, NY> gam;
    MargRef<T, NX> filt;
    const T *y;
    int64_t T_y;
    Out out;

    PSS_INL int64_t load(const TileInfo &ti, int64_t p, T (&F)[NX][NX], T (&c)[NX],
                         T (&SL)[NX][NX], T (&H)[NY][NX], T (&d)[NY], T (&SO)[NY][NY],
                         T (&yy)[NY], Marg<T, NX> &f) const
    {
        const int64_t t = ti.off + ti.cnt - 1 - p; // step slot of step n - p
        gam.load_trans(t, F, c, SL);
        gam.load_obs(t, H, d, SO);
#pragma unroll
        for (int a = 0; a < NY; ++a)
            yy[a] = y[a * T_y + t];
        filt.load(t + ti.b, f);
        return t;
    }
    PSS_INL void up(const TileInfo &ti, int64_t p, SElem<T, NX> &e) const
    {
        T F[NX][NX], c[NX], SL[NX][NX], H[NY][NX], d[NY], SO[NY][NY], yy[NY];
        Marg<T, NX> f;
        load(ti, p, F, c, SL, H, d, SO, yy, f);
        StepQ<T, NX, NY> q;
        T Np[NX][NX], P22[NX][NX], mp[NX];
        adj_step(F, c, SL, H, d, SO, yy, f, q, Np, P22, mp);
        adj_element(F, q, e);
    }
    PSS_INL void down_apply(const TileInfo &ti, int64_t p, const Marg<T, NX> &lam,
                            Marg<T, NX> &o) const
    {
        T F[NX][NX], c[NX], SL[NX][NX], H[NY][NX], d[NY], SO[NY][NY], yy[NY];
        Marg<T, NX> f;
        const int64_t t = load(ti, p, F, c, SL, H, d, SO, yy, f);
        StepQ<T, NX, NY> q;
        T Np[NX][NX], P22[NX][NX], mp[NX];
        adj_step(F, c, SL, H, d, SO, yy, f, q, Np, P22, mp);
        {
            SElem<T, NX> e;
            adj_element(F, q, e);
            adj_apply_v<T, NX>(SRegV<T, NX>{&e}, lam, o);
        }
        adj_emit(out, ti.b, t, F, SL, H, SO, f, q, Np, P22, mp, lam);
    }
};

// its sink: the inclusive suffix at the last scan position is lambda_0
template <typename T, int NX>
struct AdjDst {
    static constexpr bool stageable = false, stage_excl = false;
    AdjPrior<T, NX> prior;
    PSS_INL void put(const TileInfo &ti, int64_t p, const Marg<T, NX> &excl,
                     const Marg<T, NX> &incl) const
    {
        if (p == ti.cnt - 1)
            prior.put(ti.b, incl);
    }
};

template <typename T, int NX, int NY, class Out, class PreRef>
__global__ __launch_bounds__(256) void k_adj_down(StepGeom g, GammaRef<T, NX, NY> gam,
                                                  const T *y, int64_t T_y, MargRef<T, NX> marg,
                                                  PreRef pre, Out out, AdjPrior<T, NX> prior,
                                                  const int64_t *next_off)
{
    const TileInfo ti = tile_info(g);
    if ((int)threadIdx.x >= ti.nvalid)
        return;
    const int64_t p0 = ti.start + (int64_t)threadIdx.x * ti.E;
    int64_t pe = p0 + ti.E;
    if (pe > ti.start + ti.tcnt)
        pe = ti.start + ti.tcnt;
    const int64_t v = ti.start / ti.E + threadIdx.x, cnt1 = next_off[ti.b + 1] - next_off[ti.b];
    Marg<T, NX> lam;
    pre.load(next_off[ti.b] + cnt1 - 1 - v, lam);
    for (int64_t p = pe - 1; p >= p0; --p) {
        const int64_t u = ilv_slot(ti, p), ug = gam.stride ? u : 0;
        T F[NX][NX], c[NX], SL[NX][NX], H[NY][NX], d[NY], SO[NY][NY], yy[NY];
        gam.load_trans(ug, F, c, SL);
        gam.load_obs(ug, H, d, SO);
#pragma unroll
        for (int a = 0; a < NY; ++a)
            yy[a] = y[a * T_y + ti.off + p];
        Marg<T, NX> f, o;
        marg.load(u, f); // state p, before the step
        StepQ<T, NX, NY> q;
        T Np[NX][NX], P22[NX][NX], mp[NX];
        adj_step(F, c, SL, H, d, SO, yy, f, q, Np, P22, mp);
        {
            SElem<T, NX> e;
            adj_element(F, q, e);
            adj_apply_v<T, NX>(SRegV<T, NX>{&e}, lam, o);
        }
        int64_t at = u;
        if constexpr (Out::kGamma)
            at = out.ilv ? u : ti.off + p;
        adj_emit(out, ti.b, at, F, SL, H, SO, f, q, Np, P22, mp, lam);
        lam = o;
    }
    if (p0 == 0)
        prior.put(ti.b, lam);
}

// cotangents at interleaved slots to plain ones, one thread per step
template <typename T, int NX, int NY>
__global__ __launch_bounds__(256) void k_gamma_plain(const int64_t *y_off, int B, int64_t T_y,
                                                     GammaRef<T, NX, NY> src,
                                                     GammaRef<T, NX, NY> dst, StepTiles tiles)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= T_y)
        return;
    const int b = find_seq(y_off, B, t, 0);
    const int64_t i = step_slot(y_off, b, t - y_off[b], tiles);
    T F[NX][NX], c[NX], S[NX][NX], H[NY][NX], d[NY], O[NY][NY];
    src.load_trans(i, F, c, S);
    src.load_obs(i, H, d, O);
    dst.store_trans(t, F, c, S);
    dst.store_obs(t, H, d, O);
}

} // namespace pss
