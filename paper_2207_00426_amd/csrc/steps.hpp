// Finest level of the smoothing pass, built from Kalman steps.
//
// A thread owns E consecutive steps of one sequence and works on them one
// after the other, from the linearisation itself:
//   k_step_fold    the aggregate of its steps (a filter element of level 1):
//                  the conditional filter started from a known state, its
//                  transfer matrix A and the information (eta, Z) its
//                  measurements hold about that state
//   k_step_walk    from the filtering marginal before its first step (the scan
//                  above): filters, writes the smoother element of every state
//                  (Table 4) and folds them into the thread's smoother aggregate
//   k_step_smooth  from the smoothing marginal after its last step: Table 5's
//                  apply form, back to its first state
// so no filter element is ever stored, and the filtering marginals only on
// request.  A step costs about half the flops of building an element and
// combining it (Lemma 1 and Table 3 hold for any split of the steps).  Between
// two steps the factor N of a marginal is any square root of P, NX x NX and
// dense: the next step's Tria([F N, S_L]) depends on its Gram matrix alone, so
// the update's own Tria stops after its NY measurement rows.  A stored factor
// is triangular as everywhere.
//
// The linearisation, the stash of smoother elements and the nominal between
// passes are tile-interleaved (ilv): a wave's accesses are whole lines.
//
// Measured at 10^6 FP64 coordinated-turn steps, per pass: fold 0.137 ms for 0.56
// GB (4.1 TB/s, one wave a SIMD), walk 0.193 ms for 0.92 GB, smooth 0.12 ms for
// 0.54 GB (both bound by their bytes; a large copy reaches 4.9 TB/s); they replace
// element build (0.224), filter up and down (0.202, 0.139) and smoother up and down
// (0.334, 0.191 ms).  Holding fold and walk to 256 registers (two waves a SIMD)
// gained nothing: 0.161 and 0.221 ms.  Reading the next step's linearisation while
// this one computes (448 and 466 registers) took the walk to 0.182 ms there, but
// made short sequences slower: 8 steps of fold 34 -> 36 us, of walk 45 -> 48.
#pragma once

#include "kernels.hpp"
#include "scan_group.hpp"

namespace pss {

// marginals of every state: plain (state k of sequence b at y_off[b] + b + k)
// or tile-interleaved (state k < n at the slot of step k, state n at T_y + b)
template <typename T, int NX>
struct NomRef {
    MargRef<T, NX> r;
    int64_t T_y;
    int ilv;
    PSS_INL int64_t slot(const int64_t *y_off, const TileInfo &ti, int64_t k) const
    {
        if (!ilv)
            return ti.off + ti.b + k;
        return k < ti.cnt ? ilv_slot(ti, k) : T_y + ti.b;
    }
};

// tiles of the finest level: T threads of E steps each, fewer for a short
// sequence
struct StepTiles {
    int T, E;
    ShortRule few;
    PSS_INL int elems(int64_t n) const { return few.elems(n, E); }
};

// k / TS of a step index, in 32 bits wherever k fits (a 64-bit division takes
// some forty instructions more)
PSS_INL int64_t tile_of(int64_t k, int64_t TS)
{
    if (((k | TS) >> 32) == 0)
        return (int64_t)((uint32_t)k / (uint32_t)TS);
    return k / TS;
}

// stored slot of step k of sequence b
PSS_INL int64_t step_slot(const int64_t *y_off, int b, int64_t k, const StepTiles &tl)
{
    const int64_t cnt = y_off[b + 1] - y_off[b];
    const int E = tl.elems(cnt);
    const int64_t TS = (int64_t)tl.T * E, start = tile_of(k, TS) * TS;
    const int tcnt = (int)(cnt - start < TS ? cnt - start : TS);
    return y_off[b] + start + ilv((int)(k - start), tcnt, E);
}
// its inverse: the step stored at slot i
PSS_INL int64_t slot_step(const int64_t *y_off, int b, int64_t i, const StepTiles &tl)
{
    const int64_t q = i - y_off[b], cnt = y_off[b + 1] - y_off[b];
    const int E = tl.elems(cnt);
    const int64_t TS = (int64_t)tl.T * E, start = tile_of(q, TS) * TS;
    const int tcnt = (int)(cnt - start < TS ? cnt - start : TS);
    return start + ilv_inv((int)(q - start), tcnt, E);
}

// place of thread v's aggregate among the level-1 elements of its sequence
PSS_INL int64_t agg_slot(const int64_t *next_off, int b, int64_t v, int nT, int nE)
{
    const int64_t off = next_off[b], cnt = next_off[b + 1] - off;
    const int64_t TS = (int64_t)nT * nE, start = tile_of(v, TS) * TS;
    const int tcnt = (int)((cnt - start) < TS ? (cnt - start) : TS);
    return off + start + ilv((int)(v - start), tcnt, nE);
}

// The steps' arithmetic is FP64 for FP32 storage too: a step then needs no
// scaling of its rows, which cost FP32 more than its faster rate gave back, and
// the only rounding to FP32 is of what is stored.
using StepT = double;

template <typename T, int NX, typename W>
PSS_INL void marg_cast(const Marg<T, NX> &a, Marg<W, NX> &o)
{
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        o.m[i] = W(a.m[i]);
#pragma unroll
        for (int j = 0; j <= i; ++j)
            o.N[i][j] = W(a.N[i][j]);
    }
}

template <typename T, int NX, int NY, typename W>
PSS_INL void load_obs_w(const GammaRef<T, NX, NY> &gam, int64_t u, W (&H)[NY][NX], W (&d)[NY],
                        W (&SO)[NY][NY])
{
#pragma unroll
    for (int a = 0; a < NY; ++a) {
#pragma unroll
        for (int j = 0; j < NX; ++j)
            H[a][j] = W(gam.H[(a * NX + j) * gam.ld + u]);
        d[a] = W(gam.d[a * gam.ld + u]);
#pragma unroll
        for (int j = 0; j <= a; ++j)
            SO[a][j] = W(gam.SO[tri_idx(a, j) * gam.ld + u]);
    }
}

// where the filter starts: the prior (m0, N0), its mean relative to r_0 in
// deviation coordinates
template <typename T, int NX>
struct StepPrior {
    const T *m0, *N0;
    const T *dev_m; // nominal means, component i of state 0 of sequence b at
    int64_t dev_ld; // dev_m[i * dev_ld + s0]; null: absolute coordinates
    PSS_INL T mean(int i, int64_t s0) const
    {
        using W = typename BranchPrec<T>::type;
        return dev_m ? T(W(m0[i]) - W(dev_m[i * dev_ld + s0])) : m0[i];
    }
};

template <typename T, int NX, int NY, class AggRef>
__global__ __launch_bounds__(256) void k_step_fold(StepGeom g, GammaRef<T, NX, NY> gam,
                                                   const T *y, int64_t T_y,
                                                   StepPrior<T, NX> prior, NomRef<T, NX> nom,
                                                   AggRef agg, const int64_t *next_off, int nT,
                                                   int nE)
{
    using W = StepT;
    const TileInfo ti = tile_info(g);
    if ((int)threadIdx.x >= ti.nvalid)
        return;
    const int64_t p0 = ti.start + (int64_t)threadIdx.x * ti.E;
    int64_t pe = p0 + ti.E;
    if (pe > ti.start + ti.tcnt)
        pe = ti.start + ti.tcnt;
    FElem<W, NX> e; // U dense between steps
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        e.b[i] = e.eta[i] = W(0);
#pragma unroll
        for (int j = 0; j < NX; ++j) {
            e.A[i][j] = (i == j) ? W(1) : W(0);
            e.U[i][j] = e.Z[i][j] = W(0);
        }
    }
    if (p0 == 0) { // the sequence's first thread: a true prefix (A = 0)
        const int64_t s0 = nom.slot(g.y_off, ti, 0);
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            e.b[i] = prior.mean(i, s0);
            e.A[i][i] = W(0);
#pragma unroll
            for (int j = 0; j <= i; ++j)
                e.U[i][j] = prior.N0[tri_idx(i, j)];
        }
    }
    for (int64_t p = p0; p < pe; ++p) {
        const int64_t u = gam.stride ? ilv_slot(ti, p) : 0;
        W M[NX][2 * NX];
        {
            W F[NX][NX];
#pragma unroll
            for (int i = 0; i < NX; ++i)
#pragma unroll
                for (int j = 0; j < NX; ++j)
                    F[i][j] = W(gam.F[(i * NX + j) * gam.ld + u]);
            W FA[NX][NX], Fb[NX];
            mm(F, e.A, FA);
            mv(F, e.b, Fb);
#pragma unroll
            for (int i = 0; i < NX; ++i) {
                e.b[i] = Fb[i] + W(gam.c[i * gam.ld + u]);
#pragma unroll
                for (int j = 0; j < NX; ++j)
                    e.A[i][j] = FA[i][j];
            }
#pragma unroll
            for (int i = 0; i < NX; ++i)
#pragma unroll
                for (int j = 0; j < NX; ++j) {
                    W s = F[i][0] * e.U[0][j];
#pragma unroll
                    for (int t = 1; t < NX; ++t)
                        s = pfma(F[i][t], e.U[t][j], s);
                    M[i][j] = s;
                    M[i][NX + j] =
                        j <= i ? W(gam.SL[tri_idx(i, j <= i ? j : i) * gam.ld + u]) : W(0);
                }
        }
        lq_rows<NX, NX>(M);
        W H[NY][NX], d[NY], SO[NY][NY];
        load_obs_w(gam, u, H, d, SO);
        W Q[NY + NX][NX + NY];
        step_update(H, M, SO, Q);
        // G = Y^{-1} H A, w = Y^{-1} (y - H b - d)
        W G[NY][NX], w[NY][1];
        mm(H, e.A, G);
#pragma unroll
        for (int a = 0; a < NY; ++a) {
            W s = W(y[a * T_y + ti.off + p]) - d[a];
#pragma unroll
            for (int j = 0; j < NX; ++j)
                s = pfma(-H[a][j], e.b[j], s);
            w[a][0] = s;
        }
        step_solve<W, NY, NX>(Q, G);
        step_solve<W, NY, 1>(Q, w);
        W Gt[NX][NY];
#pragma unroll
        for (int i = 0; i < NX; ++i)
#pragma unroll
            for (int a = 0; a < NY; ++a) {
                Gt[i][a] = G[a][i];
                e.eta[i] = pfma(G[a][i], w[a][0], e.eta[i]);
                e.b[i] = pfma(Q[NY + i][a], w[a][0], e.b[i]);
            }
#pragma unroll
        for (int i = 0; i < NX; ++i)
#pragma unroll
            for (int j = 0; j < NX; ++j) {
                W s = e.A[i][j];
#pragma unroll
                for (int a = 0; a < NY; ++a)
                    s = pfma(-Q[NY + i][a], G[a][j], s);
                e.A[i][j] = s;
                e.U[i][j] = Q[NY + i][NY + j];
            }
        W Zn[NX][NX];
        tria_cols_lower(Gt, e.Z, Zn);
#pragma unroll
        for (int i = 0; i < NX; ++i)
#pragma unroll
            for (int j = 0; j <= i; ++j)
                e.Z[i][j] = Zn[i][j];
    }
    {
        W Un[NX][NX];
        tria_rect(e.U, Un);
#pragma unroll
        for (int i = 0; i < NX; ++i)
#pragma unroll
            for (int j = 0; j <= i; ++j)
                e.U[i][j] = Un[i][j];
    }
    const int64_t v = ti.start / ti.E + threadIdx.x;
    felem_copy<W, NX>(FRegV<W, NX>{&e}, view_of(agg, agg_slot(next_off, ti.b, v, nT, nE)));
}

// filtering marginals on request: state k of sequence b at plain slot
// y_off[b] + b + k of (m, N); m null: not taken
template <typename T, int NX, int NY, class AggRef, class PreRef>
__global__ __launch_bounds__(256) void k_step_walk(StepGeom g, GammaRef<T, NX, NY> gam,
                                                   const T *y, int64_t T_y,
                                                   StepPrior<T, NX> prior, NomRef<T, NX> nom,
                                                   PreRef pre, SElemRef<T, NX> stash,
                                                   AggRef agg, MargAos<T, NX> last,
                                                   MargRef<T, NX> filt, const int64_t *next_off,
                                                   int nT, int nE)
{
    using W = StepT;
    const TileInfo ti = tile_info(g);
    if ((int)threadIdx.x >= ti.nvalid)
        return;
    const int64_t p0 = ti.start + (int64_t)threadIdx.x * ti.E;
    int64_t pe = p0 + ti.E;
    if (pe > ti.start + ti.tcnt)
        pe = ti.start + ti.tcnt;
    const int64_t v = ti.start / ti.E + threadIdx.x, cnt1 = next_off[ti.b + 1] - next_off[ti.b];
    W m[NX], N[NX][NX]; // N dense between steps
    {
        Marg<T, NX> f;
        if (p0 == 0) {
            const int64_t s0 = nom.slot(g.y_off, ti, 0);
#pragma unroll
            for (int i = 0; i < NX; ++i) {
                f.m[i] = prior.mean(i, s0);
#pragma unroll
                for (int j = 0; j <= i; ++j)
                    f.N[i][j] = prior.N0[tri_idx(i, j)];
            }
            if (filt.m)
                filt.store(ti.off + ti.b, f);
        } else {
            pre.load(next_off[ti.b] + v, f);
        }
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            m[i] = W(f.m[i]);
#pragma unroll
            for (int j = 0; j < NX; ++j)
                N[i][j] = j <= i ? W(f.N[i][j]) : W(0);
        }
    }
    SElem<W, NX> a; // the thread's smoother aggregate
    for (int64_t p = p0; p < pe; ++p) {
        const int64_t u = ilv_slot(ti, p), ug = gam.stride ? u : 0;
        // [[F N, S_L], [N, 0]], upper rows reduced: N^- = M11, E = M21 M11^{-1},
        // D D^T = M22 M22^T (Table 4)
        W M[2 * NX][2 * NX], mp[NX];
        {
            W F[NX][NX];
#pragma unroll
            for (int i = 0; i < NX; ++i)
#pragma unroll
                for (int j = 0; j < NX; ++j)
                    F[i][j] = W(gam.F[(i * NX + j) * gam.ld + ug]);
            mv(F, m, mp);
#pragma unroll
            for (int i = 0; i < NX; ++i) {
                mp[i] += W(gam.c[i * gam.ld + ug]);
#pragma unroll
                for (int j = 0; j < NX; ++j) {
                    W s = F[i][0] * N[0][j];
#pragma unroll
                    for (int t = 1; t < NX; ++t)
                        s = pfma(F[i][t], N[t][j], s);
                    M[i][j] = s;
                    M[i][NX + j] =
                        j <= i ? W(gam.SL[tri_idx(i, j <= i ? j : i) * gam.ld + ug]) : W(0);
                    M[NX + i][j] = N[i][j];
                    M[NX + i][NX + j] = W(0);
                }
            }
        }
        lq_rows<NX, NX>(M);
        {
            SElem<W, NX> e;
            {
                W P11[NX][NX], P21[NX][NX], P22[NX][NX];
#pragma unroll
                for (int i = 0; i < NX; ++i)
#pragma unroll
                    for (int j = 0; j < NX; ++j) {
                        P11[i][j] = M[i][j];
                        P21[i][j] = M[NX + i][j];
                        P22[i][j] = M[NX + i][NX + j];
                    }
                rsolve_lower(P21, P11, e.E);
                tria_rect(P22, e.D);
            }
#pragma unroll
            for (int i = 0; i < NX; ++i) {
                W s = m[i];
#pragma unroll
                for (int j = 0; j < NX; ++j)
                    s = pfma(-e.E[i][j], mp[j], s);
                e.g[i] = s;
            }
            selem_copy<W, NX>(SRegV<W, NX>{&e}, view_of(stash, u));
            if (p == p0)
                a = e;
            else
                smoother_combine_v<W, NX>(SRegV<W, NX>{&a}, SRegV<W, NX>{&e}, SRegV<W, NX>{&a});
        }
        W H[NY][NX], d[NY], SO[NY][NY];
        load_obs_w(gam, ug, H, d, SO);
        W Q[NY + NX][NX + NY], w[NY][1];
        step_update(H, M, SO, Q);
#pragma unroll
        for (int q = 0; q < NY; ++q) {
            W s = W(y[q * T_y + ti.off + p]) - d[q];
#pragma unroll
            for (int j = 0; j < NX; ++j)
                s = pfma(-H[q][j], mp[j], s);
            w[q][0] = s;
        }
        step_solve<W, NY, 1>(Q, w);
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            m[i] = mp[i];
#pragma unroll
            for (int q = 0; q < NY; ++q)
                m[i] = pfma(Q[NY + i][q], w[q][0], m[i]);
#pragma unroll
            for (int j = 0; j < NX; ++j)
                N[i][j] = Q[NY + i][NY + j];
        }
        if (filt.m) {
            Marg<W, NX> f;
            Marg<T, NX> o;
            tria_rect(N, f.N);
#pragma unroll
            for (int i = 0; i < NX; ++i)
                f.m[i] = m[i];
            marg_cast(f, o);
            filt.store(ti.off + ti.b + p + 1, o);
        }
    }
    if (v == cnt1 - 1) {
        // the sequence's end: the filtering marginal of state n is the
        // smoother's start (its element {0, m, N}), folded in here
        Marg<W, NX> f, o;
        tria_rect(N, f.N);
#pragma unroll
        for (int i = 0; i < NX; ++i)
            f.m[i] = m[i];
        T *q = last.p + (int64_t)ti.b * Sizes<NX>::marg;
        visit(f, [&](int c, W &x) { q[c] = T(x); });
        smoother_apply(a, f, o);
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            a.g[i] = o.m[i];
#pragma unroll
            for (int j = 0; j < NX; ++j) {
                a.E[i][j] = W(0);
                if (j <= i)
                    a.D[i][j] = o.N[i][j];
            }
        }
    }
    // the smoother scans backwards: its element cnt1 - 1 - v
    selem_copy<W, NX>(SRegV<W, NX>{&a},
                      view_of(agg, agg_slot(next_off, ti.b, cnt1 - 1 - v, nT, nE)));
}

template <typename T, int NX, class PreRef>
__global__ __launch_bounds__(256) void k_step_smooth(StepGeom g, SElemRef<T, NX> stash,
                                                     PreRef pre, MargAos<T, NX> last,
                                                     NomRef<T, NX> dev, NomRef<T, NX> out,
                                                     const int64_t *next_off)
{
    using W = StepT;
    const TileInfo ti = tile_info(g);
    if ((int)threadIdx.x >= ti.nvalid)
        return;
    const int64_t p0 = ti.start + (int64_t)threadIdx.x * ti.E;
    int64_t pe = p0 + ti.E;
    if (pe > ti.start + ti.tcnt)
        pe = ti.start + ti.tcnt;
    const int64_t v = ti.start / ti.E + threadIdx.x, cnt1 = next_off[ti.b + 1] - next_off[ti.b];
    Marg<W, NX> s;
    // deviation coordinates: the stored mean is r_k plus the deviation
    auto put = [&](int64_t k, const Marg<W, NX> &x) {
        const int64_t at = out.slot(g.y_off, ti, k);
        Marg<T, NX> o;
        marg_cast(x, o);
        if (dev.r.m) {
            const int64_t rk = dev.slot(g.y_off, ti, k);
#pragma unroll
            for (int i = 0; i < NX; ++i)
                o.m[i] = T(x.m[i] + W(dev.r.m[i * dev.r.ld + rk]));
        }
        out.r.store(at, o);
    };
    Marg<T, NX> s0;
    if (v == cnt1 - 1) {
        last.load(ti.b, s0);
        marg_cast(s0, s);
        put(ti.cnt, s);
    } else {
        pre.load(next_off[ti.b] + cnt1 - 1 - v, s0);
        marg_cast(s0, s);
    }
    for (int64_t p = pe - 1; p >= p0; --p) {
        const auto e = view_of(stash, ilv_slot(ti, p));
        Marg<W, NX> o;
        smoother_apply_v<W, NX>(e, s, o);
        s = o;
        put(p, s);
    }
}

// interleaved marginals to plain ones, one thread per state
template <typename T, int NX>
__global__ __launch_bounds__(256) void k_nominal_plain(const int64_t *y_off, int B, int64_t T_y,
                                                       int64_t T_x, MargRef<T, NX> src,
                                                       MargRef<T, NX> dst, StepTiles tiles)
{
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= T_x)
        return;
    const int b = find_seq(y_off, B, s, 1);
    const int64_t k = s - y_off[b] - b, n = y_off[b + 1] - y_off[b];
    Marg<T, NX> x;
    src.load(k < n ? step_slot(y_off, b, k, tiles) : T_y + b, x);
    dst.store(s, x);
}

// a caller's per-step linearisation into interleaved slots, one thread per slot
template <typename T, int NX, int NY>
__global__ __launch_bounds__(256) void k_gamma_ilv(const int64_t *y_off, int B, int64_t T_y,
                                                   GammaRef<T, NX, NY> src,
                                                   GammaRef<T, NX, NY> dst, StepTiles tiles)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= T_y)
        return;
    const int b = find_seq(y_off, B, i, 0);
    const int64_t t = y_off[b] + slot_step(y_off, b, i, tiles);
    T F[NX][NX], c[NX], S[NX][NX], H[NY][NX], d[NY], O[NY][NY];
    src.load_trans(t, F, c, S);
    src.load_obs(t, H, d, O);
    dst.store_trans(i, F, c, S);
    dst.store_obs(i, H, d, O);
}

// Linearisation of every step into its interleaved slot, two threads per stored
// slot in blocks of their own: the transition at state k (blockIdx.y = 0) and
// the measurement at state k + 1 (1).  They share nothing but the index, and one
// after the other they made a chain of some 4000 instructions, all there is to a
// short sequence's launch.  A block takes 256 steps that follow each other, so
// that it reads a plain nominal's lines once, and its lanes follow the slots: a
// run of 256 / E lanes stores whole lines.  FP64 cubature: 100 steps 8.7 us (in
// one chain 12), 10^6 steps 182 us (one thread per slot 198, per step 255).
// Lin: trans(marginal, F, c, S_L) and obs(marginal, y, H, d, S_O).
template <class Lin>
__global__ __launch_bounds__(256) void k_step_lin(const int64_t *y_off, int B, int64_t T_y,
                                                  Lin lin, NomRef<typename Lin::T, Lin::NX> nom,
                                                  const typename Lin::T *y,
                                                  GammaRef<typename Lin::T, Lin::NX, Lin::NY> out,
                                                  StepTiles tiles, int dev)
{
    using T = typename Lin::T;
    constexpr int NX = Lin::NX, NY = Lin::NY;
    const int64_t base = (int64_t)blockIdx.x * 256;
    int64_t i = base + threadIdx.x;
    int b = find_seq(y_off, B, base, 0); // the block's first; the threads go on from it
    if (base + 256 <= T_y) { // the steps E apart side by side
        const int E = tiles.elems(y_off[b + 1] - y_off[b]);
        if ((E & (E - 1)) == 0 && E <= 16) {
            const int run = 256 / E;
            i = base + (threadIdx.x & (run - 1)) * E + threadIdx.x / run;
        }
    }
    if (i >= T_y)
        return;
    while (y_off[b + 1] <= i)
        ++b;
    const int64_t n = y_off[b + 1] - y_off[b], k = i - y_off[b];
    const int64_t u = step_slot(y_off, b, k, tiles);
    // state k: in tile order it has the step's slot
    const int64_t s0 = nom.ilv ? u : i + b;
    const int64_t s1 = !nom.ilv ? s0 + 1
                       : k + 1 < n ? step_slot(y_off, b, k + 1, tiles)
                                   : T_y + b;
    Marg<T, NX> mg;
    if (blockIdx.y == 0) {
        nom.r.load(s0, mg);
        T F[NX][NX], c[NX], S[NX][NX];
        lin.trans(mg, F, c, S);
        if (dev) {
            T rk[NX];
#pragma unroll
            for (int q = 0; q < NX; ++q)
                rk[q] = nom.r.m[q * nom.r.ld + s1];
            dev_trans_offset(F, mg.m, rk, c);
        }
        out.store_trans(u, F, c, S);
    } else {
        nom.r.load(s1, mg);
        T yy[NY], H[NY][NX], d[NY], S[NY][NY];
#pragma unroll
        for (int a = 0; a < NY; ++a)
            yy[a] = y[a * T_y + i];
        lin.obs(mg, yy, H, d, S);
        if (dev)
            dev_obs_offset(H, mg.m, d);
        out.store_obs(u, H, d, S);
    }
}

template <typename T_, bool TAYLOR>
struct LinCT {
    using T = T_;
    static constexpr int NX = 5, NY = 2;
    CTParams<T> P;
    PSS_INL void trans(const Marg<T, 5> &mg, T (&F)[5][5], T (&c)[5], T (&S)[5][5]) const
    {
        if constexpr (TAYLOR)
            ct_taylor_transition(P, mg, F, c, S);
        else
            ct_slr_transition<T, true>(P, mg, F, c, S);
    }
    PSS_INL void obs(const Marg<T, 5> &mg, const T (&y)[2], T (&H)[2][5], T (&d)[2],
                     T (&S)[2][2]) const
    {
        if constexpr (TAYLOR)
            ct_taylor_bearings(P, mg, y, H, d, S);
        else
            ct_slr_bearings(P, mg, y, H, d, S);
    }
};

template <typename T_>
struct LinCTRule {
    using T = T_;
    static constexpr int NX = 5, NY = 2;
    CTParams<T> P;
    RuleSpec<T> R;
    PSS_INL void trans(const Marg<T, 5> &mg, T (&F)[5][5], T (&c)[5], T (&S)[5][5]) const
    {
        ct_rule_transition(R, P, mg, F, c, S);
    }
    PSS_INL void obs(const Marg<T, 5> &mg, const T (&y)[2], T (&H)[2][5], T (&d)[2],
                     T (&S)[2][2]) const
    {
        ct_rule_bearings(R, P, mg, y, H, d, S);
    }
};

template <typename T_>
struct LinRicker {
    using T = T_;
    static constexpr int NX = 1, NY = 1;
    RickerParams<T> P;
    RuleSpec<T> R;
    int taylor;
    PSS_INL void trans(const Marg<T, 1> &mg, T (&F)[1][1], T (&c)[1], T (&S)[1][1]) const
    {
        if (taylor) {
            T H[1][1], d[1], O[1][1];
            ricker_taylor(P, mg, mg, true, false, F, c, S, H, d, O);
        } else {
            ricker_rule_transition(R, P, mg, F, c, S);
        }
    }
    PSS_INL void obs(const Marg<T, 1> &mg, const T (&y)[1], T (&H)[1][1], T (&d)[1],
                     T (&S)[1][1]) const
    {
        if (taylor) {
            T F[1][1], c[1], O[1][1];
            ricker_taylor(P, mg, mg, false, true, F, c, O, H, d, S);
        } else {
            ricker_rule_poisson(R, P, mg, H, d, S);
        }
    }
};

} // namespace pss
