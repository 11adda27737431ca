// Host-side launch logic: workspace layout, scan level planning and the
// per-(dtype, nx, ny) implementations behind the C ABI.
#pragma once

#include <algorithm>
#include <type_traits>

#include "adjoint.hpp"
#include "common.hpp"
#include "kernels.hpp"
#include "scan_group.hpp"
#include "steps.hpp"

namespace pss {

template <typename T>
inline const T *cptr(const void *p) { return static_cast<const T *>(p); }
template <typename T>
inline T *mptr(void *p) { return static_cast<T *>(p); }

// default launch shapes (overridable through pss_problem).  One 64-lane wave per
// tile at the finest level; where it scans stored elements, the filter folds 4 of
// them per thread, the smoother 2 (its operator is cheaper, and with 2 its level-0
// reads and stash writes stay closer to whole cache lines).  The filter's finest
// level is flat: its per-thread aggregates are the next level's elements, so no
// in-tile tree runs there (a tree step keeps the whole wave busy for one operator
// while half of its lanes or fewer have work).  The smoother's operator is cheap
// next to its element construction, so its finest level keeps the tree and saves a
// level.  Above it, Tup x E1 and Tup x Eup only set how many elements a tile has:
// its block splits them over 32 groups of 16 lanes (scan_group.hpp), 8 elements a
// group in a full tile of 256.  One element per lane, T threads of E, is left for a
// scalar state, the covariance form and FP32 log-likelihoods.
template <typename T, int NX>
struct Defaults {
    static constexpr int T0 = 64;
    static constexpr int E0_filter = 4;
    static constexpr int E0_smoother = 2;
    // Kalman steps per thread (steps.hpp): 8 balance the level above, which
    // costs most per element, against the thread's serial steps; a short
    // sequence leaves the chip idle and only the serial steps and the rounds
    // above them count.  The rule looks at the sequence alone, so that its
    // result does not depend on its batch.  us per call at 2, 4 and 8 steps, 2
    // FP64 passes: one sequence of 100 158, 181, 249; of 256 206, 198, 264; of 512
    // 285, 241, 282; of 768 325, 281, 315; of 1003 327, 324, 327; of 10^6 3556,
    // -, 2095; 60 of 768 398, 327, 375.  One FP32 pass of 300 of 600 steps 735,
    // 525, 540, of 1000 1070, 788, 647.  A scalar state has cheap operators and
    // folds 2 (2 passes of 10^4 Ricker steps: 112 us, with 8 129).
    static constexpr int E0_step = NX == 1 ? 2 : 8;
    static constexpr int64_t n_half = NX == 1 ? 0 : 768;
    static constexpr int64_t n_quarter = NX == 1 ? 0 : 256;
    static constexpr int Tup = 64;
    static constexpr int E1_filter = 4;
    static constexpr int E1_smoother = 2;
    static constexpr int Eup_filter = 2;
    static constexpr int Eup_smoother = 2;
    static constexpr bool flat_filter = true;
    static constexpr bool flat_smoother = false;
};

// marginals of a call up to this size are written in the caller's layout by
// the last smoothing pass itself
constexpr size_t kDirectBytes = size_t(16) << 20;

template <typename T, int NX, int NY>
struct Core {
    using FS = FilterScan<T, NX>;
    using SS = SmootherScan<T, NX>;
    static constexpr int P = tri_size(NX);
    static constexpr int PY = tri_size(NY);
    static constexpr bool kFlatF = Defaults<T, NX>::flat_filter;
    static constexpr bool kFlatS = Defaults<T, NX>::flat_smoother;
    // log-likelihoods from Kalman steps; FP32 keeps the scan over elements
    // (see FilterScanLane)
    static constexpr bool kStepsLL = sizeof(T) == 8;

    // ------------------------------------------------------------------
    static void shapes(const Ctx &c, bool smoother, int &T0, int &E0, int &Tup, int &E1,
                       int &Eup)
    {
        T0 = c.p->scan_threads > 0 ? c.p->scan_threads : Defaults<T, NX>::T0;
        E0 = c.p->scan_elems > 0 ? c.p->scan_elems
                                 : (smoother ? Defaults<T, NX>::E0_smoother
                                             : Defaults<T, NX>::E0_filter);
        Tup = Defaults<T, NX>::Tup;
        E1 = smoother ? Defaults<T, NX>::E1_smoother : Defaults<T, NX>::E1_filter;
        Eup = smoother ? Defaults<T, NX>::Eup_smoother : Defaults<T, NX>::Eup_filter;
        if (Tup > T0)
            Tup = T0;
    }

    // workspace of one scan; with base == nullptr only sizes
    template <class Op>
    struct ScanWs {
        int64_t *tile_off[kMaxLevels];
        int64_t *elem_off[kMaxLevels]; // element offsets of level l >= 1
        T *agg[kMaxLevels];  // elements of level l >= 1
        T *pre[kMaxLevels];  // exclusive prefixes of level l >= 1
        T *tree[kMaxLevels]; // LDS tree of a tree level l < L-1
    };

    template <class Op>
    static ScanWs<Op> carve_scan(Carver &cv, const Ctx &c, const ScanShape &sh)
    {
        ScanWs<Op> w{};
        for (int l = 0; l < sh.L; ++l)
            w.tile_off[l] = cv.template take<int64_t>(c.B + 1);
        for (int l = 1; l < sh.L; ++l) {
            w.elem_off[l] = cv.template take<int64_t>(c.B + 1);
            w.agg[l] = cv.template take<T>((size_t)Op::NE * sh.nelem[l]);
            w.pre[l] = cv.template take<T>((size_t)Op::NP * sh.nelem[l]);
        }
        for (int l = 0; l + 1 < sh.L; ++l)
            if (!sh.flat[l])
                w.tree[l] = cv.template take<T>((size_t)Op::NE * sh.ntiles[l] * sh.T[l]);
        return w;
    }

    static FElemRef<T, NX> felem_ref(T *base, int64_t ld)
    {
        FElemRef<T, NX> r;
        r.ld = ld;
        r.A = base;
        r.b = r.A + (int64_t)NX * NX * ld;
        r.U = r.b + (int64_t)NX * ld;
        r.eta = r.U + (int64_t)P * ld;
        r.Z = r.eta + (int64_t)NX * ld;
        return r;
    }
    static SElemRef<T, NX> selem_ref(T *base, int64_t ld)
    {
        SElemRef<T, NX> r;
        r.ld = ld;
        r.E = base;
        r.g = r.E + (int64_t)NX * NX * ld;
        r.D = r.g + (int64_t)NX * ld;
        return r;
    }
    static MargRef<T, NX> marg_ref(T *base, int64_t ld)
    {
        MargRef<T, NX> r;
        r.ld = ld;
        r.m = base;
        r.N = base + (int64_t)NX * ld;
        return r;
    }
    static MargRef<T, NX> marg_ref2(const void *m, const void *N, int64_t ld)
    {
        MargRef<T, NX> r;
        r.ld = ld;
        r.m = const_cast<T *>(cptr<T>(m));
        r.N = const_cast<T *>(cptr<T>(N));
        return r;
    }
    static GammaRef<T, NX, NY> gamma_ref(const pss_gamma *g, int64_t T_y)
    {
        GammaRef<T, NX, NY> r;
        r.F = mptr<T>(g->F);
        r.c = mptr<T>(g->c);
        r.SL = mptr<T>(g->SL);
        r.H = mptr<T>(g->H);
        r.d = mptr<T>(g->d);
        r.SO = mptr<T>(g->SO);
        r.stride = g->stride;
        r.ld = g->stride ? T_y : 1;
        return r;
    }
    // a linearisation buffer carved from the workspace (stride 1)
    static pss_gamma carve_gamma(Carver &cv, int64_t T_y)
    {
        pss_gamma g;
        g.F = cv.template take<T>((size_t)NX * NX * T_y);
        g.c = cv.template take<T>((size_t)NX * T_y);
        g.SL = cv.template take<T>((size_t)P * T_y);
        g.H = cv.template take<T>((size_t)NY * NX * T_y);
        g.d = cv.template take<T>((size_t)NY * T_y);
        g.SO = cv.template take<T>((size_t)PY * T_y);
        g.stride = 1;
        return g;
    }

    // one in space of exactly its size (component arrays back to back)
    static pss_gamma carve_gamma_packed(T *p, int64_t T_y)
    {
        pss_gamma g;
        g.F = p;
        g.c = p += (int64_t)NX * NX * T_y;
        g.SL = p += (int64_t)NX * T_y;
        g.H = p += (int64_t)P * T_y;
        g.d = p += (int64_t)NY * NX * T_y;
        g.SO = p += (int64_t)NY * T_y;
        g.stride = 1;
        return g;
    }

    template <class Op>
    static size_t lds_bytes(int Tb, int E, bool stage)
    {
        return scan_lds(Op::NE, Op::NP, Tb, E, sizeof(T), stage);
    }

    template <class K>
    static int prep_lds(K kernel, size_t bytes)
    {
        return hip_check(hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize,
                                             (int)bytes),
                         "hipFuncSetAttribute");
    }

    // references to a level's elements and prefixes: one element per 16-lane
    // group above the finest level where the scan has group operators (stored
    // whole), else one per lane
    template <class Op, class AggRef>
    static auto agg_of(const ScanShape &sh, const ScanWs<Op> &w, int l,
                       AggRef (*agg_ref)(T *, int64_t))
    {
        if constexpr (GroupOp<Op>::value)
            return typename GroupOp<Op>::Ref{w.agg[l]};
        else
            return agg_ref(w.agg[l], sh.nelem[l]);
    }
    template <class Op>
    static auto pre_of(const ScanShape &sh, const ScanWs<Op> &w, int l)
    {
        if constexpr (GroupOp<Op>::value)
            return MargAos<T, NX>{w.pre[l]};
        else
            return marg_ref(w.pre[l], sh.nelem[l]);
    }
    // elements per thread that the finest level's aggregates are interleaved
    // for (whole elements need no interleaving)
    template <class Op>
    static int agg_ilv(const ScanShape &sh) { return GroupOp<Op>::value ? 1 : sh.E[1]; }

    template <class Op>
    static LevelGeom level_geom(const Ctx &c, const ScanShape &sh, const ScanWs<Op> &w, int l,
                                int extra)
    {
        LevelGeom g;
        g.y_off = c.p->y_off;
        g.elem_off = l > 0 ? w.elem_off[l] : nullptr;
        g.tile_off = w.tile_off[l];
        g.level = l;
        g.extra = extra;
        g.B = c.B;
        g.E = sh.E[l];
        g.stage = scan_stage(Op::NE, Op::NP, sh.T[l], sh.E[l], sizeof(T));
        return g;
    }
    // the finest level's, where it runs Kalman steps
    template <class Op>
    static StepGeom step_geom(const Ctx &c, const ScanShape &sh, const ScanWs<Op> &w)
    {
        StepGeom g;
        static_cast<LevelGeom &>(g) = level_geom(c, sh, w, 0, 0);
        g.few = sh.few;
        return g;
    }

    // multi-level scan driver: the finest level's kernels come from the caller
    // (up0 writes the elements of level 1, down0 reads their prefixes, top0 is
    // the whole scan where level 0 is the top), the levels above run here.
    // Flat: level 0 may be flat (then it is, see plan_scan).
    // stop > 0 (and < sh.L): run only the levels below `stop`, whose
    // exclusive prefixes w.pre[stop] the caller provides (a checkpoint):
    // the up-sweeps that rebuild those levels' trees and elements, then their
    // down-sweeps; the levels from `stop` up are not run.
    template <class Op, bool Flat, class AggRef, class Start, class Up0, class Top0, class Down0>
    static int run_levels(const Ctx &c, const ScanShape &sh, const ScanWs<Op> &w, int extra,
                          const Start &start, AggRef (*agg_ref)(T *, int64_t), int stop,
                          const Up0 &up0, const Top0 &top0, const Down0 &down0)
    {
        const int top = (stop > 0 && stop < sh.L) ? stop : sh.L;
        const bool partial = top < sh.L;
        int rc = PSS_OK;
        constexpr bool Grp = GroupOp<Op>::value;
        using LvSrc = RefSrc<Op, AggRef>;
        using LvSrcI = RefSrc<Op, AggRef, true>;
        using LvDst = PreDst<Op, MargRef<T, NX>>;
        auto ggeom = [&](int l) {
            return GroupGeom{w.elem_off[l], w.tile_off[l], c.B, sh.T[l] * sh.E[l]};
        };
        // calls launch(src) with the element source of level l >= 1
        auto with_src = [&](int l, auto &&launch) -> int {
            if constexpr (Flat) {
                if (l == 1 && sh.flat[0])
                    return launch(LvSrcI{agg_ref(w.agg[l], sh.nelem[l])});
            }
            return launch(LvSrc{agg_ref(w.agg[l], sh.nelem[l])});
        };
        // up-sweeps of the lower levels (below a checkpoint: all levels
        // under it; a flat level right under it needs no up-sweep, its
        // down-sweep reads the stored prefixes per thread)
        for (int l = 0; l + 1 < sh.L && l < top; ++l) {
            if (partial && l == top - 1 && sh.flat[l])
                continue;
            if (l == 0) {
                if ((rc = up0()))
                    return rc;
                continue;
            }
            const LevelGeom g = level_geom(c, sh, w, l, extra);
            const int64_t tree_ld = sh.ntiles[l] * sh.T[l];
            const size_t lb = lds_bytes<Op>(sh.T[l], sh.E[l], g.stage);
            const dim3 grid((unsigned)sh.ntiles[l]);
            KTime kt(c.s, Op::name, "up", l);
            if constexpr (Grp) {
                static_assert(kGroups <= 64, "the saved prefixes use the tree's space");
                hipLaunchKernelGGL((k_group_up<Op>), grid, dim3(kGroupThreads), 0, c.s, ggeom(l),
                                   w.agg[l], w.agg[l + 1], w.tree[l]);
            } else {
                rc = with_src(l, [&](auto s) -> int {
                    auto k = k_scan_up<Op, decltype(s), AggRef>;
                    if (int r = prep_lds(k, lb))
                        return r;
                    hipLaunchKernelGGL(k, grid, dim3(sh.T[l]), lb, c.s, g, s,
                                       agg_ref(w.agg[l + 1], sh.nelem[l + 1]), w.tree[l],
                                       tree_ld);
                    return 0;
                });
                if (rc)
                    return rc;
            }
            if ((rc = hip_check(hipGetLastError(), "scan up launch")))
                return rc;
        }
        // top level
        if (!partial && sh.L == 1) {
            if ((rc = top0()))
                return rc;
        } else if (!partial) {
            const int l = sh.L - 1;
            const LevelGeom g = level_geom(c, sh, w, l, extra);
            const size_t lb = lds_bytes<Op>(sh.T[l], sh.E[l], g.stage);
            const dim3 grid((unsigned)sh.ntiles[l]);
            KTime kt(c.s, Op::name, "top", l);
            if constexpr (Grp) {
                hipLaunchKernelGGL((k_group_top<Op, Start>), grid, dim3(kGroupThreads), 0, c.s,
                                   ggeom(l), w.agg[l], w.pre[l], start);
            } else {
                LvDst d{marg_ref(w.pre[l], sh.nelem[l])};
                rc = with_src(l, [&](auto s) -> int {
                    auto k = k_scan_top<Op, decltype(s), LvDst, Start>;
                    if (int r = prep_lds(k, lb))
                        return r;
                    hipLaunchKernelGGL(k, grid, dim3(sh.T[l]), lb, c.s, g, s, d, start);
                    return 0;
                });
                if (rc)
                    return rc;
            }
            if ((rc = hip_check(hipGetLastError(), "scan top launch")))
                return rc;
        }
        // down-sweeps of the lower levels
        for (int l = top - (partial ? 1 : 2); l >= 0; --l) {
            if (l == 0) {
                if ((rc = down0()))
                    return rc;
                continue;
            }
            const LevelGeom g = level_geom(c, sh, w, l, extra);
            const int64_t tree_ld = sh.ntiles[l] * sh.T[l];
            const size_t lb = lds_bytes<Op>(sh.T[l], sh.E[l], g.stage);
            const dim3 grid((unsigned)sh.ntiles[l]);
            KTime kt(c.s, Op::name, "down", l);
            if constexpr (Grp) {
                hipLaunchKernelGGL((k_group_down<Op>), grid, dim3(kGroupThreads), 0, c.s,
                                   ggeom(l), w.agg[l], w.tree[l], w.pre[l + 1], w.pre[l]);
            } else {
                LvDst d{marg_ref(w.pre[l], sh.nelem[l])};
                MargRef<T, NX> pin = marg_ref(w.pre[l + 1], sh.nelem[l + 1]);
                rc = with_src(l, [&](auto s) -> int {
                    auto k = k_scan_down<Op, decltype(s), LvDst, MargRef<T, NX>>;
                    if (int r = prep_lds(k, lb))
                        return r;
                    hipLaunchKernelGGL(k, grid, dim3(sh.T[l]), lb, c.s, g, s, d, w.tree[l],
                                       tree_ld, pin);
                    return 0;
                });
                if (rc)
                    return rc;
            }
            if ((rc = hip_check(hipGetLastError(), "scan down launch")))
                return rc;
        }
        return PSS_OK;
    }

    // a scan whose finest level folds and applies given elements (Src0, Dst0);
    // Top0: it may be the top (a plan without never_top)
    template <class Op, bool Flat, bool Top0 = true, class Src0, class Dst0, class AggRef,
              class Start>
    static int run_scan(const Ctx &c, const ScanShape &sh, const ScanWs<Op> &w, int extra,
                        const Src0 &src0, const Dst0 &dst0, const Start &start,
                        AggRef (*agg_ref)(T *, int64_t), int stop = 0)
    {
        int rc = launch_plan(c, sh, extra, w.tile_off, w.elem_off);
        if (rc)
            return rc;
        const LevelGeom g = level_geom(c, sh, w, 0, extra);
        const int64_t tree_ld = sh.ntiles[0] * sh.T[0];
        const size_t lb = lds_bytes<Op>(sh.T[0], sh.E[0], g.stage);
        const dim3 grid((unsigned)sh.ntiles[0]), block(sh.T[0]);
        auto up0 = [&]() -> int {
            KTime kt(c.s, Op::name, "up", 0);
            const auto agg = agg_of(sh, w, 1, agg_ref);
            using Agg = std::decay_t<decltype(agg)>;
            if constexpr (Flat) {
                if (sh.flat[0]) {
                    auto k = k_scan_up_flat<Op, Src0, Agg>;
                    if (int r = prep_lds(k, lb))
                        return r;
                    hipLaunchKernelGGL(k, grid, block, lb, c.s, g, src0, agg, w.elem_off[1],
                                       sh.T[1], agg_ilv<Op>(sh));
                    return hip_check(hipGetLastError(), "scan up launch");
                }
            }
            auto k = k_scan_up<Op, Src0, Agg>;
            if (int r = prep_lds(k, lb))
                return r;
            hipLaunchKernelGGL(k, grid, block, lb, c.s, g, src0, agg, w.tree[0], tree_ld);
            return hip_check(hipGetLastError(), "scan up launch");
        };
        auto top0 = [&]() -> int {
            if constexpr (Top0) {
                KTime kt(c.s, Op::name, "top", 0);
                auto k = k_scan_top<Op, Src0, Dst0, Start>;
                if (int r = prep_lds(k, lb))
                    return r;
                hipLaunchKernelGGL(k, grid, block, lb, c.s, g, src0, dst0, start);
                return hip_check(hipGetLastError(), "scan top launch");
            }
            return PSS_OK;
        };
        auto down0 = [&]() -> int {
            KTime kt(c.s, Op::name, "down", 0);
            const auto pin = pre_of(sh, w, 1);
            using Pre = std::decay_t<decltype(pin)>;
            if constexpr (Flat) {
                if (sh.flat[0]) {
                    auto k = k_scan_down_flat<Op, Src0, Dst0, Pre>;
                    if (int r = prep_lds(k, lb))
                        return r;
                    hipLaunchKernelGGL(k, grid, block, lb, c.s, g, src0, dst0, w.elem_off[1],
                                       pin);
                    return hip_check(hipGetLastError(), "scan down launch");
                }
            }
            auto k = k_scan_down<Op, Src0, Dst0, Pre>;
            if (int r = prep_lds(k, lb))
                return r;
            hipLaunchKernelGGL(k, grid, block, lb, c.s, g, src0, dst0, w.tree[0], tree_ld, pin);
            return hip_check(hipGetLastError(), "scan down launch");
        };
        return run_levels<Op, Flat>(c, sh, w, extra, start, agg_ref, stop, up0, top0, down0);
    }

    // ------------------------------------------------------------------
    // filter scan (elements read from `el`)
    static ScanShape filter_shape(const Ctx &c)
    {
        int T0, E0, Tup, E1, Eup;
        shapes(c, false, T0, E0, Tup, E1, Eup);
        return plan_scan(c, 0, T0, E0, Tup, E1, Eup, kFlatF);
    }
    static ScanShape smoother_shape(const Ctx &c)
    {
        int T0, E0, Tup, E1, Eup;
        shapes(c, true, T0, E0, Tup, E1, Eup);
        return plan_scan(c, 1, T0, E0, Tup, E1, Eup, kFlatS);
    }

    static size_t fscan_bytes(const Ctx &c)
    {
        Carver cv{nullptr};
        carve_scan<FS>(cv, c, filter_shape(c));
        return cv.used;
    }
    static size_t sscan_bytes(const Ctx &c)
    {
        Carver cv{nullptr};
        carve_scan<SS>(cv, c, smoother_shape(c));
        cv.template take<T>((size_t)Sizes<NX>::selem * c.T_x); // element stash
        return cv.used;
    }

    // ilv: the elements are stored tile-interleaved for this scan's level 0
    // (as written by felem(..., true)); the library's own passes use that
    // cov: the standard (covariance-form) scan of the same storage layout
    static int fscan(const Ctx &c, const pss_felem *el, void *mf, void *Nf, void *ws,
                     bool ilv = false, bool cov = false)
    {
        const ScanShape sh = filter_shape(c);
        Carver cv{static_cast<char *>(ws)};
        auto w = carve_scan<FS>(cv, c, sh);
        FElemRef<T, NX> er;
        er.A = mptr<T>(el->A);
        er.b = mptr<T>(el->b);
        er.U = mptr<T>(el->U);
        er.eta = mptr<T>(el->eta);
        er.Z = mptr<T>(el->Z);
        er.ld = c.T_y;
        FiltDst<T, NX> dst{marg_ref2(mf, Nf, c.T_x), c.p->y_off};
        dst.dev_m = cptr<T>(c.dev_m);
        StartPre<T, NX> st{cptr<T>(c.p->m0), cptr<T>(c.p->N0)};
        // finest-level elements: Z = Tria([Z_k, 0]) with Z_k of ny columns
        constexpr int LZ = NY < NX ? NY : NX;
        if (cov) {
            using FSC = FilterScanCov<T, NX>;
            StartPreCov<T, NX> stc{cptr<T>(c.p->m0), cptr<T>(c.p->N0)};
            Carver cc{static_cast<char *>(ws)};
            auto wc = carve_scan<FSC>(cc, c, sh);
            if (ilv) {
                RefSrc<FSC, FElemRef<T, NX>, true> src{er};
                return run_scan<FSC, kFlatF>(c, sh, wc, 0, src, dst, stc, &felem_ref);
            }
            RefSrc<FSC, FElemRef<T, NX>> src{er};
            return run_scan<FSC, kFlatF>(c, sh, wc, 0, src, dst, stc, &felem_ref);
        }
        if (ilv) {
            RefSrc<FS, FElemRef<T, NX>, true, LZ> src{er};
            return run_scan<FS, kFlatF>(c, sh, w, 0, src, dst, st, &felem_ref);
        }
        RefSrc<FS, FElemRef<T, NX>, false, LZ> src{er};
        return run_scan<FS, kFlatF>(c, sh, w, 0, src, dst, st, &felem_ref);
    }

    // the filter scan of a log-likelihood over stored (interleaved) elements,
    // one element per lane at every level.  ck_pre: the exclusive prefixes of
    // level ck_level (1 <= ck_level < levels) -- written there by a full scan,
    // or, with resume, read from there and only the levels below re-run
    static int fscan_lane(const Ctx &c, const pss_felem *el, void *mf, void *Nf, void *ws,
                          int ck_level, T *ck_pre, bool resume)
    {
        using FL = FilterScanLane<T, NX>;
        const ScanShape sh = filter_shape(c);
        Carver cv{static_cast<char *>(ws)};
        auto w = carve_scan<FL>(cv, c, sh);
        const bool ck = ck_pre && ck_level >= 1 && ck_level < sh.L;
        if (ck)
            w.pre[ck_level] = ck_pre;
        FElemRef<T, NX> er;
        er.A = mptr<T>(el->A);
        er.b = mptr<T>(el->b);
        er.U = mptr<T>(el->U);
        er.eta = mptr<T>(el->eta);
        er.Z = mptr<T>(el->Z);
        er.ld = c.T_y;
        FiltDst<T, NX> dst{marg_ref2(mf, Nf, c.T_x), c.p->y_off};
        StartPre<T, NX> st{cptr<T>(c.p->m0), cptr<T>(c.p->N0)};
        constexpr int LZ = NY < NX ? NY : NX;
        RefSrc<FL, FElemRef<T, NX>, true, LZ> src{er};
        return run_scan<FL, kFlatF>(c, sh, w, 0, src, dst, st, &felem_ref,
                                    ck && resume ? ck_level : 0);
    }

    static int sscan(const Ctx &c, const pss_gamma *g, const void *mf, const void *Nf, void *ms,
                     void *Ns, void *ws, bool cov = false)
    {
        const ScanShape sh = smoother_shape(c);
        Carver cv{static_cast<char *>(ws)};
        auto w = carve_scan<SS>(cv, c, sh);
        T *stash = cv.template take<T>((size_t)Sizes<NX>::selem * c.T_x);
        SmoothDst<T, NX> dst{marg_ref2(ms, Ns, c.T_x)};
        dst.dev_m = cptr<T>(c.dev_m);
        StartPre<T, NX> st{nullptr, nullptr};
        if (cov) {
            using SSC = SmootherScanCov<T, NX>;
            Carver cc{static_cast<char *>(ws)};
            auto wc = carve_scan<SSC>(cc, c, sh);
            SmootherSrc<T, NX, NY, true> src{gamma_ref(g, c.T_y), marg_ref2(mf, Nf, c.T_x),
                                             selem_ref(stash, c.T_x), c.p->y_off};
            return run_scan<SSC, kFlatS>(c, sh, wc, 1, src, dst, st, &selem_ref);
        }
        SmootherSrc<T, NX, NY> src{gamma_ref(g, c.T_y), marg_ref2(mf, Nf, c.T_x),
                                   selem_ref(stash, c.T_x), c.p->y_off};
        return run_scan<SS, kFlatS>(c, sh, w, 1, src, dst, st, &selem_ref);
    }

    static int felem(const Ctx &c, const pss_gamma *g, const void *y, const pss_felem *out,
                     bool ilv = false, bool cov = false)
    {
        int ilv_T = 0, ilv_E = 0;
        if (ilv) {
            const ScanShape sh = filter_shape(c);
            ilv_T = sh.T[0];
            ilv_E = sh.E[0];
        }
        FElemRef<T, NX> er;
        er.A = mptr<T>(out->A);
        er.b = mptr<T>(out->b);
        er.U = mptr<T>(out->U);
        er.eta = mptr<T>(out->eta);
        er.Z = mptr<T>(out->Z);
        er.ld = c.T_y;
        // a block covers a whole level-0 tile (64 x 4): the strided reads of
        // its tile-interleaved elements meet the same cache lines in one L2
        const int tb = 256;
        KTime kt(c.s, cov ? "filter_elements_cov" : "filter_elements", "", 0);
        const dim3 grid((unsigned)((c.T_y + tb - 1) / tb));
        if (cov)
            hipLaunchKernelGGL((k_filter_elements<T, NX, NY, true>), grid, dim3(tb), 0, c.s,
                               c.p->y_off, c.B, c.T_y, gamma_ref(g, c.T_y), cptr<T>(y),
                               cptr<T>(c.p->m0), cptr<T>(c.p->N0), er, ilv_T, ilv_E,
                               cptr<T>(c.dev_m), c.T_x);
        else
            hipLaunchKernelGGL((k_filter_elements<T, NX, NY>), grid, dim3(tb), 0, c.s,
                               c.p->y_off, c.B, c.T_y, gamma_ref(g, c.T_y), cptr<T>(y),
                               cptr<T>(c.p->m0), cptr<T>(c.p->N0), er, ilv_T, ilv_E,
                               cptr<T>(c.dev_m), c.T_x);
        return hip_check(hipGetLastError(), "filter elements launch");
    }

    // ------------------------------------------------------------------
    // model-specific pieces
    static int slr(const Ctx &c, const void *m, const void *N, const void *y,
                   const pss_gamma *out);
    // the CT model with cubature or Taylor linearisation in FP32: slr and
    // the (tile-interleaved) filter elements in one kernel; returns 1,
    // launching nothing, for every other case.  (In FP64 the fused kernel's
    // register footprint made it slower than the two kernels it replaces:
    // 0.47 ms against 0.17 + 0.23 ms at n = 10^6; in FP32 0.16 against
    // 0.08 + 0.13 ms.)
    static int slr_felem(const Ctx &c, const void *m, const void *N, const void *y,
                         const pss_gamma *g, const pss_felem *el, bool cov, bool store_obs);
    static int grad_terms(const Ctx &c, const pss_gamma *g, const void *y, const void *mf,
                          const void *Nf, const void *ms, const void *Ns, double *gterms);

    // ------------------------------------------------------------------
    // composite operations
    static size_t felem_bytes(const Ctx &c)
    {
        return align256((size_t)Sizes<NX>::felem * c.T_y * sizeof(T));
    }
    static size_t marg_bytes(const Ctx &c)
    {
        return align256((size_t)Sizes<NX>::marg * c.T_x * sizeof(T));
    }
    static size_t gamma_bytes(const Ctx &c)
    {
        Carver cv{nullptr};
        carve_gamma(cv, c.T_y);
        return cv.used;
    }
    // nonlinear models are linearised on every pass; a linear one is given
    static bool nonlinear(const Ctx &c) { return c.p->model != PSS_MODEL_LINEAR; }

    // scan and sum space of the log-likelihood calls (shared in time); the
    // covariance form scans stored elements
    static size_t grad_scans(const Ctx &c, int nc)
    {
        size_t adj;
        if (kStepsLL) {
            adj = scan_bytes(c, grad_shape(c));
        } else {
            Carver cv{nullptr};
            carve_scan<AdjScan<T, NX>>(cv, c, adj_shape(c));
            adj = cv.used;
        }
        return std::max({fscan_bytes(c), adj, seq_sum_bytes(c, nc)});
    }

    // (each part walks the sequences: only what the operation needs)
    static size_t ws_size(const Ctx &c, int op)
    {
        auto scans = [&]() { return std::max(fscan_bytes(c), sscan_bytes(c)); };
        auto fwd = [&]() {
            return gamma_bytes(c) + felem_bytes(c) + marg_bytes(c) +
                   align256(c.T_y * sizeof(double));
        };
        switch (op) {
        case PSS_OP_SLR:
        case PSS_OP_FILTER_ELEMENTS:
            return 0;
        case PSS_OP_FILTER_SCAN:
            return fscan_bytes(c);
        case PSS_OP_SMOOTHER_SCAN:
            return sscan_bytes(c);
        case PSS_OP_IPLS: {
            // stored elements, which the covariance form uses; the steps' stash
            // is smaller by about a marginal per step, and the size a caller
            // asks for stays one for both
            const size_t el = felem_bytes(c) + scans();
            return gamma_bytes(c) + marg_bytes(c) +
                   (c.p->form == PSS_FORM_COV
                        ? el
                        : std::max(el, align256(step_stash(c) * sizeof(T)) +
                                           scan_bytes(c, step_shape(c))));
        }
        case PSS_OP_LOGLIK:
            return fwd() + grad_scans(c, 1);
        case PSS_OP_LOGLIK_GRAD:
            return fwd() + grad_scans(c, 3) + align256(3 * c.T_y * sizeof(double)) +
                   align256(3 * c.B * sizeof(double));
        case PSS_OP_LOGLIK_VJP:
            return fwd() + grad_scans(c, 1);
        case PSS_OP_SCORE_FISHER:
            return gamma_bytes(c) + felem_bytes(c) + marg_bytes(c) +
                   align256(c.T_y * sizeof(double)) + std::max(scans(), seq_sum_bytes(c, 3)) +
                   marg_bytes(c) + align256(3 * c.T_y * sizeof(double)) +
                   align256(3 * c.B * sizeof(double));
        case PSS_OP_SEQUENTIAL:
            return gamma_bytes(c) + marg_bytes(c);
        default:
            return 0;
        }
    }

    // ------------------------------------------------------------------
    // checkpoints of the log-likelihood's filter pass (pss_ckpt): the
    // per-sequence log-likelihoods, then what the level keeps -- level 0
    // every filtering marginal, level l in [1, levels) the exclusive
    // prefixes of the filter scan's level-l elements, higher levels nothing
    struct CkView {
        int level = 0;
        double *ll = nullptr;
        T *marg = nullptr; // level 0: [Sizes::marg][T_x]
        T *pre = nullptr;  // level l: [Sizes::marg][nelem_l]
    };
    static size_t ckpt_bytes(const Ctx &c, int level)
    {
        Carver cv{nullptr};
        cv.template take<double>((size_t)c.B);
        if (level == 0) {
            cv.template take<T>((size_t)Sizes<NX>::marg * c.T_x);
        } else {
            const ScanShape sh = filter_shape(c);
            int64_t n = level < sh.L ? sh.nelem[level] : 0;
            if constexpr (kStepsLL) { // what fills it (no more, by its longer runs)
                const ScanShape gs = grad_shape(c);
                n = std::max(n, level < gs.L ? gs.nelem[level] : 0);
            }
            if (n > 0)
                cv.template take<T>((size_t)Sizes<NX>::marg * n);
        }
        return cv.used;
    }
    static CkView ckpt_view(const Ctx &c, const pss_ckpt *ck)
    {
        CkView v;
        if (!ck)
            return v;
        v.level = ck->level;
        Carver cv{static_cast<char *>(ck->buf)};
        v.ll = cv.template take<double>((size_t)c.B);
        if (ck->level == 0)
            v.marg = cv.template take<T>((size_t)Sizes<NX>::marg * c.T_x);
        else if (ck->level < (kStepsLL ? grad_shape(c).L : filter_shape(c).L))
            v.pre = cv.template take<T>(0);
        return v;
    }
    // the filter scan's level count for this problem (checkpoint levels
    // from it up keep nothing but the log-likelihoods)
    static int filter_levels(const Ctx &c) { return filter_shape(c).L; }

    // tiles of the finest level when it runs Kalman steps (steps.hpp)
    static ScanShape step_shape(const Ctx &c)
    {
        int T0, E0, Tup, E1, Eup;
        shapes(c, false, T0, E0, Tup, E1, Eup);
        if (c.p->scan_elems > 0)
            return plan_scan(c, 0, T0, E0, Tup, E1, Eup, true);
        using D = Defaults<T, NX>;
        return plan_scan(c, 0, T0, D::E0_step, Tup, E1, Eup, true,
                         ShortRule{D::n_half, D::n_quarter});
    }
    static size_t step_stash(const Ctx &c)
    {
        return (size_t)Sizes<NX>::selem * c.T_y + (size_t)Sizes<NX>::marg * c.B;
    }
    static StepTiles step_tiles(const ScanShape &sh)
    {
        return StepTiles{sh.T[0], sh.E[0], sh.few};
    }

    // the same for the FP64 log-likelihood calls: at least 4 steps a thread, so
    // that a checkpoint of level 1 holds a prefix per 4 states at most.  Their
    // walks are longer per step and their scans above cheaper, so 8 steps pay
    // only on long sequences (us per gradient at 4 and 8 steps: 1 x 1500 210 and
    // 220, 8 x 6000 of a linear model 253 and 313, 1 x 10^4 227 and 274, 64 x
    // 10^4 889 and 806).
    static ScanShape grad_shape(const Ctx &c)
    {
        int T0, E0, Tup, E1, Eup;
        shapes(c, false, T0, E0, Tup, E1, Eup);
        if (c.p->scan_elems > 0)
            return plan_scan(c, 0, T0, E0, Tup, E1, Eup, true);
        using D = Defaults<T, NX>;
        return plan_scan(c, 0, T0, std::max(4, D::E0_step), Tup, E1, Eup, true,
                         ShortRule{NX == 1 ? 0 : 8192, 0});
    }
    // FP32's adjoint scan, tiles of a wave with 2 steps a thread (their reads are
    // 2 numbers apart; at 4 the passes take half as long again)
    static ScanShape adj_shape(const Ctx &c)
    {
        const int T0 = c.p->scan_threads > 0 ? c.p->scan_threads : Defaults<T, NX>::T0;
        const int Tup = std::min(T0, (int)Defaults<T, NX>::Tup);
        return plan_scan(c, 0, T0, 2, Tup, 2, 2, false, {}, true);
    }
    static size_t scan_bytes(const Ctx &c, const ScanShape &sh)
    {
        Carver cv{nullptr};
        carve_scan<FS>(cv, c, sh);
        return cv.used;
    }
    template <class Op>
    static ScanWs<Op> share_ws(const ScanShape &sh, const ScanWs<FS> &w)
    {
        static_assert(Op::NE <= FS::NE && Op::NP <= FS::NP, "shares the filter scan's space");
        ScanWs<Op> o{};
        for (int l = 0; l < sh.L; ++l) {
            o.tile_off[l] = w.tile_off[l];
            o.elem_off[l] = w.elem_off[l];
            o.agg[l] = w.agg[l];
            o.pre[l] = w.pre[l];
            o.tree[l] = w.tree[l];
        }
        return o;
    }

    // linearisation of every step into its interleaved slot
    static int step_lin(const Ctx &c, const NomRef<T, NX> &nom, const void *y,
                        const pss_gamma *out, const ScanShape &sh);

    // Algorithm 3 in covariance form: the scans over stored elements
    static int ipls_cov(const Ctx &c, const pss_gamma *gin, const void *y, int n_iter,
                        void *m_nom, void *N_nom, void *mf_out, void *Nf_out, void *ws)
    {
        Carver cv{static_cast<char *>(ws)};
        pss_gamma gw = carve_gamma(cv, c.T_y);
        T *fel = cv.template take<T>((size_t)Sizes<NX>::felem * c.T_y);
        T *mfb = cv.template take<T>((size_t)Sizes<NX>::marg * c.T_x);
        void *scan_ws = cv.base + cv.used;
        const pss_gamma *g = nonlinear(c) ? &gw : gin;
        Ctx cs = c;
        if (sizeof(T) == 4 && c.p->model == PSS_MODEL_CT_BEARINGS && !mf_out)
            cs.dev_m = m_nom;
        FElemRef<T, NX> fr = felem_ref(fel, c.T_y);
        pss_felem el{fr.A, fr.b, fr.U, fr.eta, fr.Z};
        void *mf = mf_out ? mf_out : (void *)mfb;
        void *Nf = mf_out ? Nf_out : (void *)(mfb + (size_t)NX * c.T_x);
        int rc = PSS_OK;
        for (int it = 0; it < n_iter && rc == PSS_OK; ++it) {
            const int fused =
                nonlinear(c) ? slr_felem(cs, m_nom, N_nom, y, &gw, &el, true, false) : 1;
            if (fused < 0) {
                rc = fused;
                break;
            }
            if (fused) {
                if (nonlinear(c) && (rc = slr(cs, m_nom, N_nom, y, &gw)))
                    break;
                if ((rc = felem(cs, g, y, &el, true, true)))
                    break;
            }
            if ((rc = fscan(cs, &el, mf, Nf, scan_ws, true, true)))
                break;
            rc = sscan(cs, g, mf, Nf, m_nom, N_nom, scan_ws, true);
        }
        return rc;
    }

    // Algorithm 3 in square-root form: the finest level runs Kalman steps
    static int ipls(const Ctx &c, const pss_gamma *gin, const void *y, int n_iter, void *m_nom,
                    void *N_nom, void *mf_out, void *Nf_out, void *ws)
    {
        if (c.p->form == PSS_FORM_COV)
            return ipls_cov(c, gin, y, n_iter, m_nom, N_nom, mf_out, Nf_out, ws);
        const ScanShape sh = step_shape(c);
        Carver cv{static_cast<char *>(ws)};
        pss_gamma gw = carve_gamma(cv, c.T_y);
        // the smoother elements, then one marginal per sequence
        T *fel = cv.template take<T>(step_stash(c));
        T *mid = cv.template take<T>((size_t)Sizes<NX>::marg * c.T_x);
        const auto w = carve_scan<FS>(cv, c, sh);
        const SElemRef<T, NX> stash = selem_ref(fel, c.T_y);
        const MargAos<T, NX> last{fel + (size_t)Sizes<NX>::selem * c.T_y};
        // the smoother's upper levels take over the filter's space
        const auto ws_s = share_ws<SS>(sh, w);
        int rc = launch_plan(c, sh, 0, w.tile_off, w.elem_off);
        if (rc)
            return rc;
        const StepTiles tiles = step_tiles(sh);
        GammaRef<T, NX, NY> gam = gamma_ref(&gw, c.T_y);
        if (!nonlinear(c) && (rc = step_given(c, gin, gw, tiles, gam)))
            return rc;
        const NomRef<T, NX> plain{marg_ref2(m_nom, N_nom, c.T_x), c.T_y, 0};
        const NomRef<T, NX> inner{marg_ref(mid, c.T_x), c.T_y, 1};
        // The last pass writes the caller's layout itself while the lines it
        // fills piecemeal stay in the caches (each thread fills E consecutive
        // states of every component); a longer one writes interleaved and a
        // copy follows.  10^6 FP64 states: 0.32 ms in place, 0.12 + 0.07 ms with
        // the copy; 4 * 10^5 FP32 states 0.083 against 0.031 + 0.020 ms.
        const bool direct = (size_t)c.T_x * Sizes<NX>::marg * sizeof(T) <= kDirectBytes;
        // FP32: the CT model's passes run in deviation coordinates relative
        // to the nominal means (see Ctx), unless the caller takes the
        // filtering marginals (those are absolute).  On the 10^6-step track
        // this cut the late passes' mean error about 5x; FP64 loses nothing
        // measurable in absolute coordinates and keeps them.
        const bool dev = sizeof(T) == 4 && c.p->model == PSS_MODEL_CT_BEARINGS && !mf_out;
        const MargRef<T, NX> filt = marg_ref2(mf_out, Nf_out, c.T_x);
        for (int it = 0; it < n_iter; ++it) {
            const bool fin = it + 1 == n_iter;
            const NomRef<T, NX> in = it == 0 ? plain : inner, out = fin && direct ? plain : inner;
            Ctx cs = c;
            cs.dev_m = dev ? in.r.m : nullptr;
            if (nonlinear(c) && (rc = step_lin(cs, in, y, &gw, sh)))
                return rc;
            NomRef<T, NX> rdev = in;
            if (!dev)
                rdev.r.m = nullptr;
            MargRef<T, NX> fo = filt;
            if (!fin)
                fo.m = nullptr;
            if ((rc = step_pass(cs, sh, w, ws_s, gam, y, in, rdev, out, stash, last, fo)))
                return rc;
        }
        if (!direct && n_iter > 0) {
            KTime kt(c.s, "nominal_plain", "", 0);
            hipLaunchKernelGGL((k_nominal_plain<T, NX>), dim3((unsigned)((c.T_x + 255) / 256)),
                               dim3(256), 0, c.s, c.p->y_off, c.B, c.T_y, c.T_x, inner.r, plain.r,
                               tiles);
            rc = hip_check(hipGetLastError(), "nominal layout launch");
        }
        return rc;
    }

    // ------------------------------------------------------------------
    // Algorithm 3 over tiles of T threads of E elements whose prefixes are
    // chained one tile after the other, everything in the type's own precision
    // and in absolute coordinates: FP32 bearings tracks of pss_ipls_batched.
    // Their results carry rounding of up to some 1e-5 (a bearings track is
    // ill-conditioned in FP32), so another bracketing, deviation coordinates or
    // FP64 steps move them by as much (measured up to 3.5e-5), and callers
    // compare them with stored ones: operators, coordinates and brackets stay
    // what they are.
    static ScanShape chain_shape(const Ctx &c, int extra, int T0, int E0)
    {
        ScanShape sh = plan_scan(c, extra, T0, E0, T0, E0, E0, false);
        sh.L = 1; // the chain takes the place of the levels above
        return sh;
    }
    template <class Op>
    static ScanWs<Op> carve_chain(Carver &cv, const Ctx &c, const ScanShape &sh)
    {
        ScanWs<Op> w{};
        w.tile_off[0] = cv.template take<int64_t>(c.B + 1);
        w.agg[1] = cv.template take<T>((size_t)Op::NE * sh.ntiles[0]);
        w.pre[1] = cv.template take<T>((size_t)Op::NP * sh.ntiles[0]);
        return w;
    }
    // everything but the chains' trees, which share one space
    struct TilesWs {
        ScanShape sh_f, sh_s;
        pss_gamma gam; // transition part only
        T *fel, *mf, *stash;
        ScanWs<FS> f;
        ScanWs<SS> s;
    };
    static TilesWs carve_tiles(Carver &cv, const Ctx &c, const TileChain &tc)
    {
        TilesWs w{};
        w.sh_f = chain_shape(c, 0, tc.T, tc.E_f);
        w.sh_s = chain_shape(c, 1, tc.T, tc.E_s);
        w.gam.F = cv.template take<T>((size_t)NX * NX * c.T_y);
        w.gam.c = cv.template take<T>((size_t)NX * c.T_y);
        w.gam.SL = cv.template take<T>((size_t)P * c.T_y);
        w.gam.stride = 1;
        w.fel = cv.template take<T>((size_t)Sizes<NX>::felem * c.T_y);
        w.mf = cv.template take<T>((size_t)Sizes<NX>::marg * c.T_x);
        w.stash = cv.template take<T>((size_t)Sizes<NX>::selem * c.T_x);
        w.f = carve_chain<FS>(cv, c, w.sh_f);
        w.s = carve_chain<SS>(cv, c, w.sh_s);
        const size_t nt = std::max((size_t)FS::NE * w.sh_f.ntiles[0],
                                   (size_t)SS::NE * w.sh_s.ntiles[0]);
        w.f.tree[0] = w.s.tree[0] = cv.template take<T>(nt * tc.T);
        return w;
    }
    static size_t tiles_bytes(const Ctx &c, const TileChain &tc)
    {
        Carver cv{nullptr};
        carve_tiles(cv, c, tc);
        return cv.used;
    }
    template <class Op, class Src, class Dst, class AggRef, class Start>
    static int run_chain(const Ctx &c, const ScanShape &sh, const ScanWs<Op> &w, int extra,
                         const Src &src, const Dst &dst, const Start &start,
                         AggRef (*agg_ref)(T *, int64_t))
    {
        using Pre = MargRef<T, NX>;
        const LevelGeom g = level_geom(c, sh, w, 0, extra);
        const int64_t nt = sh.ntiles[0], tree_ld = nt * sh.T[0];
        const size_t lb = lds_bytes<Op>(sh.T[0], sh.E[0], g.stage);
        const dim3 grid((unsigned)nt), block(sh.T[0]);
        const AggRef agg = agg_ref(w.agg[1], nt);
        const Pre pre = marg_ref(w.pre[1], nt);
        int rc;
        {
            KTime kt(c.s, Op::name, "up", 0);
            auto k = k_scan_up<Op, Src, AggRef>;
            if ((rc = prep_lds(k, lb)))
                return rc;
            hipLaunchKernelGGL(k, grid, block, lb, c.s, g, src, agg, w.tree[0], tree_ld);
            if ((rc = hip_check(hipGetLastError(), "scan up launch")))
                return rc;
        }
        {
            KTime kt(c.s, Op::name, "chain", 0);
            hipLaunchKernelGGL((k_scan_chain<Op, AggRef, Start>), dim3((unsigned)((c.B + 63) / 64)),
                               dim3(64), 0, c.s, w.tile_off[0], c.B, agg, pre, start);
            if ((rc = hip_check(hipGetLastError(), "scan chain launch")))
                return rc;
        }
        KTime kt(c.s, Op::name, "down", 0);
        auto k = k_scan_down<Op, Src, Dst, Pre>;
        if ((rc = prep_lds(k, lb)))
            return rc;
        hipLaunchKernelGGL(k, grid, block, lb, c.s, g, src, dst, w.tree[0], tree_ld, pre);
        return hip_check(hipGetLastError(), "scan down launch");
    }
    static int ipls_tiles(const Ctx &c, const TileChain &tc, const void *y, int n_iter,
                          void *m_nom, void *N_nom, void *ws)
    {
        // its linearisation and elements are one kernel (slr_felem), FP32 CT only
        if constexpr (NX == 5 && NY == 2 && std::is_same_v<T, float>) {
            Carver cv{static_cast<char *>(ws)};
            const TilesWs w = carve_tiles(cv, c, tc);
            pss_problem p = *c.p; // the elements are interleaved for these tiles
            p.scan_threads = tc.T;
            p.scan_elems = tc.E_f;
            Ctx cs = c;
            cs.p = &p;
            int rc = launch_plan(cs, w.sh_f, 0, w.f.tile_off);
            if (!rc)
                rc = launch_plan(cs, w.sh_s, 1, w.s.tile_off);
            FElemRef<T, NX> fr = felem_ref(w.fel, c.T_y);
            const pss_felem el{fr.A, fr.b, fr.U, fr.eta, fr.Z};
            const MargRef<T, NX> mf = marg_ref(w.mf, c.T_x);
            constexpr int LZ = NY < NX ? NY : NX;
            const RefSrc<FS, FElemRef<T, NX>, true, LZ> fsrc{fr};
            const FiltDst<T, NX> fdst{mf, c.p->y_off};
            const SmootherSrc<T, NX, NY> ssrc{gamma_ref(&w.gam, c.T_y), mf,
                                              selem_ref(w.stash, c.T_x), c.p->y_off};
            const SmoothDst<T, NX> sdst{marg_ref2(m_nom, N_nom, c.T_x)};
            const StartPre<T, NX> st{cptr<T>(c.p->m0), cptr<T>(c.p->N0)}, none{nullptr, nullptr};
            for (int it = 0; it < n_iter && rc == PSS_OK; ++it) {
                if ((rc = slr_felem(cs, m_nom, N_nom, y, &w.gam, &el, false, false)))
                    break;
                if ((rc = run_chain(cs, w.sh_f, w.f, 0, fsrc, fdst, st, &felem_ref)))
                    break;
                rc = run_chain(cs, w.sh_s, w.s, 1, ssrc, sdst, none, &selem_ref);
            }
            return rc;
        } else {
            set_error("chained tiles are built for FP32 bearings tracks only");
            return PSS_EUNSUPPORTED;
        }
    }

    // a linear model's given linearisation: shared by all steps as it is, per
    // step into interleaved slots
    static int step_given(const Ctx &c, const pss_gamma *gin, const pss_gamma &gw,
                          const StepTiles &tiles, GammaRef<T, NX, NY> &gam)
    {
        if (gin->stride == 0) {
            gam = gamma_ref(gin, c.T_y);
            return PSS_OK;
        }
        hipLaunchKernelGGL((k_gamma_ilv<T, NX, NY>), dim3((unsigned)((c.T_y + 255) / 256)),
                           dim3(256), 0, c.s, c.p->y_off, c.B, c.T_y, gamma_ref(gin, c.T_y),
                           gamma_ref(&gw, c.T_y), tiles);
        return hip_check(hipGetLastError(), "linearisation layout launch");
    }

    // fold of the finest level into the filter scan's level 1
    static int step_fold(const Ctx &c, const ScanShape &sh, const ScanWs<FS> &w,
                         const GammaRef<T, NX, NY> &gam, const void *y,
                         const StepPrior<T, NX> &prior, const NomRef<T, NX> &nom)
    {
        KTime kt(c.s, "step_fold", "", 0);
        const auto agg = agg_of(sh, w, 1, &felem_ref);
        using Agg = std::decay_t<decltype(agg)>;
        hipLaunchKernelGGL((k_step_fold<T, NX, NY, Agg>), dim3((unsigned)sh.ntiles[0]),
                           dim3(sh.T[0]), 0, c.s, step_geom(c, sh, w), gam, cptr<T>(y),
                           c.T_y, prior, nom, agg, w.elem_off[1], sh.T[1], agg_ilv<FS>(sh));
        return hip_check(hipGetLastError(), "step fold launch");
    }

    // one filter and smoother pass over interleaved linearisation slots
    static int step_pass(const Ctx &c, const ScanShape &sh, const ScanWs<FS> &w,
                         const ScanWs<SS> &ws_s, const GammaRef<T, NX, NY> &gam, const void *y,
                         const NomRef<T, NX> &nom, const NomRef<T, NX> &dev,
                         const NomRef<T, NX> &out, const SElemRef<T, NX> &stash,
                         const MargAos<T, NX> &last, const MargRef<T, NX> &filt)
    {
        const StepGeom g = step_geom(c, sh, w);
        const dim3 grid((unsigned)sh.ntiles[0]), block(sh.T[0]);
        const StepPrior<T, NX> prior{cptr<T>(c.p->m0), cptr<T>(c.p->N0), cptr<T>(c.dev_m),
                                     nom.r.ld};
        const StartPre<T, NX> st{cptr<T>(c.p->m0), cptr<T>(c.p->N0)}, none{nullptr, nullptr};
        auto no_top = [&]() -> int { return PSS_OK; }; // a flat level 0 is never the top
        int rc = run_levels<FS, true>(
            c, sh, w, 0, st, &felem_ref, 0,
            [&]() -> int { return step_fold(c, sh, w, gam, y, prior, nom); },
            no_top,
            [&]() -> int {
                KTime kt(c.s, "step_walk", "", 0);
                const auto pre = pre_of(sh, w, 1);
                const auto agg = agg_of(sh, ws_s, 1, &selem_ref);
                using Pre = std::decay_t<decltype(pre)>;
                using Agg = std::decay_t<decltype(agg)>;
                hipLaunchKernelGGL((k_step_walk<T, NX, NY, Agg, Pre>), grid, block, 0, c.s, g,
                                   gam, cptr<T>(y), c.T_y, prior, nom, pre, stash, agg, last,
                                   filt, w.elem_off[1], sh.T[1], agg_ilv<SS>(sh));
                return hip_check(hipGetLastError(), "step walk launch");
            });
        if (rc)
            return rc;
        return run_levels<SS, true>(
            c, sh, ws_s, 0, none, &selem_ref, 0, no_top, no_top, [&]() -> int {
                KTime kt(c.s, "step_smooth", "", 0);
                const auto pre = pre_of(sh, ws_s, 1);
                using Pre = std::decay_t<decltype(pre)>;
                hipLaunchKernelGGL((k_step_smooth<T, NX, Pre>), grid, block, 0, c.s, g, stash,
                                   pre, last, dev, out, w.elem_off[1]);
                return hip_check(hipGetLastError(), "step smooth launch");
            });
    }

    // linearisation (nonlinear models) and level-0 filter elements
    // (tile-interleaved) at the nominal; the transition and measurement
    // parts of Gamma are both stored
    static int lin_elements(const Ctx &c, const pss_gamma *gin, const void *m_nom,
                            const void *N_nom, const void *y, const pss_gamma &gw,
                            const pss_felem *el)
    {
        int rc;
        const bool cov = c.p->form == PSS_FORM_COV;
        const int fused = nonlinear(c) ? slr_felem(c, m_nom, N_nom, y, &gw, el, cov, true) : 1;
        if (fused < 0)
            return fused;
        if (fused) {
            if (nonlinear(c) && (rc = slr(c, m_nom, N_nom, y, &gw)))
                return rc;
            if ((rc = felem(c, nonlinear(c) ? &gw : gin, y, el, true, cov)))
                return rc;
        }
        return PSS_OK;
    }

    // Filter pass over stored elements: the covariance form's and FP32's
    // log-likelihood, and the score by Fisher's identity; returns the carved
    // state.  With a checkpoint (FP32) the filtering marginals go to it (level
    // 0) or the scan's level-`level` prefixes do.
    static int loglik_core(const Ctx &c, const pss_gamma *gin, const void *m_nom,
                           const void *N_nom, const void *y, double *ll, Carver &cv,
                           pss_gamma &gw, T *&mfb, void *&scan_ws, const CkView &ck = CkView{})
    {
        gw = carve_gamma(cv, c.T_y);
        T *fel = cv.template take<T>((size_t)Sizes<NX>::felem * c.T_y);
        mfb = cv.template take<T>((size_t)Sizes<NX>::marg * c.T_x);
        double *ell = cv.template take<double>((size_t)c.T_y);
        scan_ws = cv.base + cv.used;
        if (!nonlinear(c))
            gw = *gin;
        const pss_gamma *g = &gw;
        if (ck.marg)
            mfb = ck.marg;
        FElemRef<T, NX> fr = felem_ref(fel, c.T_y);
        pss_felem el{fr.A, fr.b, fr.U, fr.eta, fr.Z};
        int rc;
        const bool cov = c.p->form == PSS_FORM_COV;
        if ((rc = lin_elements(c, gin, m_nom, N_nom, y, gw, &el)))
            return rc;
        T *Nfb = mfb + (size_t)NX * c.T_x;
        if constexpr (kStepsLL)
            rc = fscan(c, &el, mfb, Nfb, scan_ws, true, cov);
        else if (cov)
            rc = fscan(c, &el, mfb, Nfb, scan_ws, true, true);
        else
            rc = fscan_lane(c, &el, mfb, Nfb, scan_ws, ck.level, ck.pre, false);
        if (rc)
            return rc;
        const int tb = 128;
        {
            KTime kt(c.s, "loglik_terms", "", 0);
            const dim3 grid((unsigned)((c.T_y + tb - 1) / tb));
            if (cov)
                hipLaunchKernelGGL((k_loglik_terms_cov<T, NX, NY>), grid, dim3(tb), 0, c.s,
                                   c.p->y_off, c.B, c.T_y, c.T_x, gamma_ref(g, c.T_y), cptr<T>(y),
                                   marg_ref(mfb, c.T_x), ell);
            else
                hipLaunchKernelGGL((k_loglik_terms<T, NX, NY>), grid, dim3(tb), 0, c.s,
                                   c.p->y_off, c.B, c.T_y, c.T_x, gamma_ref(g, c.T_y), cptr<T>(y),
                                   marg_ref(mfb, c.T_x), ell);
            if ((rc = hip_check(hipGetLastError(), "loglik launch")))
                return rc;
        }
        return launch_seq_sum(c, 1, ell, c.T_y, ll, scan_ws);
    }

    // state of a log-likelihood or gradient call in square-root form, whose
    // finest level runs Kalman steps
    struct GradState {
        ScanShape sh;
        ScanWs<FS> w;
        pss_gamma gw;
        GammaRef<T, NX, NY> gam;
        T *fel;              // the filter elements' space, not used by the scans
        MargRef<T, NX> marg; // filtering marginals, state k at the slot of step k + 1
        double *ell;
        void *sums;
    };
    static int grad_state(const Ctx &c, const pss_gamma *gin, const void *m_nom,
                          const void *N_nom, const void *y, void *ws, GradState &s)
    {
        Carver cv{static_cast<char *>(ws)};
        s.gw = carve_gamma(cv, c.T_y);
        s.fel = cv.template take<T>((size_t)Sizes<NX>::felem * c.T_y);
        s.marg = marg_ref(cv.template take<T>((size_t)Sizes<NX>::marg * c.T_x), c.T_x);
        s.ell = cv.template take<double>((size_t)c.T_y);
        s.sums = cv.base + cv.used; // after the scans, in their space
        s.sh = grad_shape(c);
        s.w = carve_scan<FS>(cv, c, s.sh);
        s.gam = gamma_ref(&s.gw, c.T_y);
        int rc = launch_plan(c, s.sh, 0, s.w.tile_off, s.w.elem_off);
        if (rc)
            return rc;
        if (!nonlinear(c))
            return step_given(c, gin, s.gw, step_tiles(s.sh), s.gam);
        return step_lin(c, NomRef<T, NX>{marg_ref2(m_nom, N_nom, c.T_x), c.T_y, 0}, y, &s.gw,
                        s.sh);
    }

    // the walk over the finest level (k_filter_walk); have: from stored
    // marginals instead of the scan's prefixes
    template <bool ADJ>
    static int filter_walk(const Ctx &c, const GradState &s, const void *y,
                           const MargRef<T, NX> &have, const MargRef<T, NX> &out, double *ell)
    {
        using AS = AdjScan<T, NX>;
        KTime kt(c.s, "filter_walk", "", 0);
        const auto wa = share_ws<AS>(s.sh, s.w);
        const auto pre = pre_of(s.sh, s.w, 1);
        const auto agg = agg_of(s.sh, wa, 1, &selem_ref);
        using Pre = std::decay_t<decltype(pre)>;
        using Agg = std::decay_t<decltype(agg)>;
        const StepPrior<T, NX> prior{cptr<T>(c.p->m0), cptr<T>(c.p->N0), nullptr, 0};
        hipLaunchKernelGGL((k_filter_walk<T, NX, NY, ADJ, Agg, Pre>),
                           dim3((unsigned)s.sh.ntiles[0]), dim3(s.sh.T[0]), 0, c.s,
                           step_geom(c, s.sh, s.w), s.gam, cptr<T>(y), c.T_y, prior, pre,
                           have, out, ell, agg, s.w.elem_off[1], s.sh.T[1], agg_ilv<AS>(s.sh));
        return hip_check(hipGetLastError(), "filter walk launch");
    }

    // forward filter pass; stop: only the levels under a checkpoint's
    template <bool ADJ>
    static int grad_filter(const Ctx &c, const GradState &s, const void *y,
                           const MargRef<T, NX> &out, double *ell, int stop = 0)
    {
        const StepPrior<T, NX> prior{cptr<T>(c.p->m0), cptr<T>(c.p->N0), nullptr, 0};
        const StartPre<T, NX> st{cptr<T>(c.p->m0), cptr<T>(c.p->N0)};
        const MargRef<T, NX> none{nullptr, nullptr, 0};
        return run_levels<FS, true>(
            c, s.sh, s.w, 0, st, &felem_ref, stop,
            [&]() -> int {
                return step_fold(c, s.sh, s.w, s.gam, y, prior, NomRef<T, NX>{none, c.T_y, 0});
            },
            []() -> int { return PSS_OK; },
            [&]() -> int { return filter_walk<ADJ>(c, s, y, none, out, ell); });
    }

    static int copy_ll(const Ctx &c, double *dst, const double *src)
    {
        return hip_check(hipMemcpyAsync(dst, src, (size_t)c.B * sizeof(double),
                                        hipMemcpyDeviceToDevice, c.s),
                         "checkpoint log-likelihood copy");
    }

    static int loglik(const Ctx &c, const pss_gamma *gin, const void *m_nom, const void *N_nom,
                      const void *y, double *ll, const pss_ckpt *ckpt, void *ws)
    {
        const CkView ck = ckpt_view(c, ckpt);
        int rc;
        if (c.p->form == PSS_FORM_COV || !kStepsLL) {
            Carver cv{static_cast<char *>(ws)};
            pss_gamma gw;
            T *mfb;
            void *scan_ws;
            rc = loglik_core(c, gin, m_nom, N_nom, y, ll, cv, gw, mfb, scan_ws, ck);
            return rc || !ckpt ? rc : copy_ll(c, ck.ll, ll);
        }
        GradState s;
        if ((rc = grad_state(c, gin, m_nom, N_nom, y, ws, s)))
            return rc;
        MargRef<T, NX> out{nullptr, nullptr, 0};
        if (ck.marg)
            out = marg_ref(ck.marg, c.T_x);
        if (ck.pre)
            s.w.pre[ck.level] = ck.pre;
        if ((rc = grad_filter<false>(c, s, y, out, s.ell)))
            return rc;
        if ((rc = launch_seq_sum(c, 1, s.ell, c.T_y, ll, s.sums)))
            return rc;
        return ckpt ? copy_ll(c, ck.ll, ll) : PSS_OK;
    }

    // forward half of a gradient: the filtering marginals (FP64: and the maps'
    // level-1 aggregates) from a checkpoint (re-running what it does not hold) or
    // a full filter pass
    static int grad_forward(const Ctx &c, const pss_gamma *gin, const void *m_nom,
                            const void *N_nom, const void *y, const pss_ckpt *ckpt, double *ll,
                            void *ws, GradState &s)
    {
        const CkView ck = ckpt_view(c, ckpt);
        int rc;
        if constexpr (kStepsLL) {
            if ((rc = grad_state(c, gin, m_nom, N_nom, y, ws, s)))
                return rc;
            if (ck.marg) {
                s.marg = marg_ref(ck.marg, c.T_x);
                const MargRef<T, NX> none{nullptr, nullptr, 0};
                return filter_walk<true>(c, s, y, s.marg, none, nullptr);
            }
            if (ck.pre)
                s.w.pre[ck.level] = ck.pre;
            return grad_filter<true>(c, s, y, s.marg, ckpt ? nullptr : s.ell,
                                     ck.pre ? ck.level : 0);
        } else {
            // over stored elements, as FP32's log-likelihood
            Carver cv{static_cast<char *>(ws)};
            T *mf;
            if (!ckpt) {
                rc = loglik_core(c, gin, m_nom, N_nom, y, ll, cv, s.gw, mf, s.sums);
                s.fel = nullptr;
            } else {
                s.gw = carve_gamma(cv, c.T_y);
                s.fel = cv.template take<T>((size_t)Sizes<NX>::felem * c.T_y);
                mf = cv.template take<T>((size_t)Sizes<NX>::marg * c.T_x);
                cv.template take<double>((size_t)c.T_y);
                s.sums = cv.base + cv.used;
                if (!nonlinear(c))
                    s.gw = *gin;
                if (ck.marg) { // only the linearisation is redone
                    mf = ck.marg;
                    rc = nonlinear(c) ? slr(c, m_nom, N_nom, y, &s.gw) : PSS_OK;
                } else {
                    FElemRef<T, NX> fr = felem_ref(s.fel, c.T_y);
                    pss_felem el{fr.A, fr.b, fr.U, fr.eta, fr.Z};
                    if ((rc = lin_elements(c, gin, m_nom, N_nom, y, s.gw, &el)))
                        return rc;
                    rc = fscan_lane(c, &el, mf, mf + (size_t)NX * c.T_x, s.sums, ck.level,
                                    ck.pre, true);
                }
            }
            if (rc)
                return rc;
            s.gam = gamma_ref(&s.gw, c.T_y);
            s.marg = marg_ref(mf, c.T_x);
            return PSS_OK;
        }
    }

    // the gradient's reverse pass: the scan of the maps, the cotangents of
    // every step; ll last (its sums use the scans' space)
    template <class Out>
    static int grad_core(const Ctx &c, const pss_gamma *gin, const void *m_nom,
                         const void *N_nom, const void *y, const pss_ckpt *ckpt, GradState &s,
                         const Out &out, const AdjPrior<T, NX> &prior, double *ll, void *ws)
    {
        using AS = AdjScan<T, NX>;
        const CkView ck = ckpt_view(c, ckpt);
        int rc = grad_forward(c, gin, m_nom, N_nom, y, ckpt, ll, ws, s);
        if (rc)
            return rc;
        Carver cv{static_cast<char *>(s.sums)};
        const StartPre<T, NX> st{nullptr, nullptr};
        if constexpr (kStepsLL) {
            const auto wa = share_ws<AS>(s.sh, carve_scan<FS>(cv, c, s.sh));
            auto nothing = []() -> int { return PSS_OK; };
            rc = run_levels<AS, true>(
                c, s.sh, wa, 0, st, &selem_ref, 0, nothing, nothing, [&]() -> int {
                    KTime kt(c.s, "adjoint_down", "", 0);
                    const auto pre = pre_of(s.sh, wa, 1);
                    using Pre = std::decay_t<decltype(pre)>;
                    hipLaunchKernelGGL((k_adj_down<T, NX, NY, Out, Pre>),
                                       dim3((unsigned)s.sh.ntiles[0]), dim3(s.sh.T[0]), 0, c.s,
                                       step_geom(c, s.sh, wa), s.gam, cptr<T>(y), c.T_y,
                                       s.marg, pre, out, prior, wa.elem_off[1]);
                    return hip_check(hipGetLastError(), "adjoint down launch");
                });
        } else {
            const ScanShape sh = adj_shape(c);
            const auto wa = carve_scan<AS>(cv, c, sh);
            const AdjSrc<T, NX, NY, Out> src{s.gam, s.marg, cptr<T>(y), c.T_y, out};
            rc = run_scan<AS, false, false>(c, sh, wa, 0, src, AdjDst<T, NX>{prior}, st,
                                            &selem_ref);
        }
        if (rc)
            return rc;
        if (ckpt)
            return copy_ll(c, ll, ck.ll);
        return kStepsLL ? launch_seq_sum(c, 1, s.ell, c.T_y, ll, s.sums) : PSS_OK;
    }

    // gradient with respect to theta (coordinated-turn model) by the
    // reverse-mode adjoint: the cotangent scan from the filtering marginals,
    // the step VJP contracted with dQ/dtheta and dR/dtheta, fixed-order
    // per-sequence sums
    static int loglik_grad(const Ctx &c, const void *m_nom, const void *N_nom, const void *y,
                           const double *ll_bar, const pss_ckpt *ckpt, double *ll, double *grad,
                           double *theta_bar, void *ws)
    {
        if constexpr (NX == 5 && NY == 2) {
            Carver tail{static_cast<char *>(ws) + gamma_bytes(c) + felem_bytes(c) +
                        marg_bytes(c) + align256(c.T_y * sizeof(double)) + grad_scans(c, 3)};
            double *gterms = tail.template take<double>((size_t)3 * c.T_y);
            double *gseq = tail.template take<double>((size_t)3 * c.B);
            GradState s;
            int rc;
            const CTHost h = ct_host(c.p);
            ThetaOut<T, NX, NY> out;
            for (int i = 0; i < 5; ++i)
                for (int j = 0; j < 5; ++j) {
                    double a1 = 0.0, a2 = 0.0;
                    for (int q = 0; q < 5; ++q) {
                        a1 += h.L1[i][q] * h.L1[j][q];
                        a2 += h.L2[i][q] * h.L2[j][q];
                    }
                    out.th.dQ1[i][j] = (T)a1;
                    out.th.dQ2[i][j] = (T)a2;
                }
            out.th.dR = (T)(2.0 * h.sigma * h.sigma);
            out.terms = gterms;
            out.T_y = c.T_y;
            const AdjPrior<T, NX> prior{nullptr, nullptr, nullptr, nullptr, c.B};
            if ((rc = grad_core(c, nullptr, m_nom, N_nom, y, ckpt, s, out, prior, ll, ws)))
                return rc;
            double *gout = grad ? grad : gseq;
            if ((rc = launch_seq_sum(c, 3, gterms, c.T_y, gout, s.sums)))
                return rc;
            if (theta_bar)
                rc = launch_weighted_grad(c, gout, ll_bar, theta_bar);
            return rc;
        } else {
            set_error("the theta gradient needs the coordinated-turn model");
            return PSS_EUNSUPPORTED;
        }
    }

    // VJP of the log-likelihood with respect to the linearisation (every
    // step's Gamma in the library's representation) and the prior
    static int loglik_vjp(const Ctx &c, const pss_gamma *gin, const void *m_nom,
                          const void *N_nom, const void *y, const double *ll_bar,
                          const pss_ckpt *ckpt, double *ll, const pss_gamma *gbar, void *m0_bar,
                          void *N0_bar, void *ws)
    {
        GradState s;
        // as the smoothed marginals: long outputs are written interleaved (into
        // the filter elements' space, where that holds them) and copied
        constexpr int NG = NX * NX + NX + P + NY * NX + NY + PY;
        const bool direct = !kStepsLL || NG > Sizes<NX>::felem ||
                            (size_t)NG * c.T_y * sizeof(T) <= kDirectBytes;
        pss_gamma gi{};
        if (!direct) {
            Carver cv{static_cast<char *>(ws)};
            carve_gamma(cv, c.T_y);
            gi = carve_gamma_packed(
                cv.template take<T>((size_t)Sizes<NX>::felem * c.T_y), c.T_y);
        }
        GammaOut<T, NX, NY> out;
        out.bar = gamma_ref(direct ? gbar : &gi, c.T_y);
        out.w = ll_bar;
        out.ilv = direct ? 0 : 1;
        const AdjPrior<T, NX> prior{mptr<T>(m0_bar), mptr<T>(N0_bar), cptr<T>(c.p->N0), ll_bar,
                                    c.B};
        int rc = grad_core(c, gin, m_nom, N_nom, y, ckpt, s, out, prior, ll, ws);
        if (rc || direct)
            return rc;
        hipLaunchKernelGGL((k_gamma_plain<T, NX, NY>), dim3((unsigned)((c.T_y + 255) / 256)),
                           dim3(256), 0, c.s, c.p->y_off, c.B, c.T_y, out.bar,
                           gamma_ref(gbar, c.T_y), step_tiles(s.sh));
        return hip_check(hipGetLastError(), "cotangent layout launch");
    }

    // the frozen-nominal score by Fisher's identity from the parallel
    // smoother (a cross-check of the adjoint)
    static int score_fisher(const Ctx &c, const void *m_nom, const void *N_nom, const void *y,
                            const double *ll_bar, double *ll, double *grad, double *theta_bar,
                            void *ws)
    {
        // layout: [gamma | felem | mf | ell | scan ws ...] then the score part
        // after the largest scan workspace
        Carver cv{static_cast<char *>(ws)};
        pss_gamma gw;
        T *mfb;
        void *scan_ws;
        const size_t scans = std::max(std::max(fscan_bytes(c), sscan_bytes(c)),
                                      seq_sum_bytes(c, 3));
        Carver tail{static_cast<char *>(ws) + gamma_bytes(c) + felem_bytes(c) + marg_bytes(c) +
                    align256(c.T_y * sizeof(double)) + scans};
        T *msb = tail.template take<T>((size_t)Sizes<NX>::marg * c.T_x);
        double *gterms = tail.template take<double>((size_t)3 * c.T_y);
        double *gseq = tail.template take<double>((size_t)3 * c.B);
        int rc = loglik_core(c, nullptr, m_nom, N_nom, y, ll, cv, gw, mfb, scan_ws);
        if (rc)
            return rc;
        T *mf = mfb, *Nf = mfb + (size_t)NX * c.T_x;
        T *ms = msb, *Ns = msb + (size_t)NX * c.T_x;
        if ((rc = sscan(c, &gw, mf, Nf, ms, Ns, scan_ws)))
            return rc;
        if ((rc = grad_terms(c, &gw, y, mf, Nf, ms, Ns, gterms)))
            return rc;
        double *gout = grad ? grad : gseq;
        // per-sequence sums land component-major [3][B]
        if ((rc = launch_seq_sum(c, 3, gterms, c.T_y, gout, scan_ws)))
            return rc;
        if (theta_bar)
            rc = launch_weighted_grad(c, gout, ll_bar, theta_bar);
        return rc;
    }

    static int sequential(const Ctx &c, const pss_gamma *gin, const void *y, int n_iter,
                          void *m_nom, void *N_nom, void *mf_out, void *Nf_out, void *ws)
    {
        Carver cv{static_cast<char *>(ws)};
        pss_gamma gw = carve_gamma(cv, c.T_y);
        T *mfb = cv.template take<T>((size_t)Sizes<NX>::marg * c.T_x);
        const pss_gamma *g = nonlinear(c) ? &gw : gin;
        void *mf = mf_out ? mf_out : (void *)mfb;
        void *Nf = mf_out ? Nf_out : (void *)(mfb + (size_t)NX * c.T_x);
        int rc = PSS_OK;
        for (int it = 0; it < n_iter && rc == PSS_OK; ++it) {
            if (nonlinear(c) && (rc = slr(c, m_nom, N_nom, y, &gw)))
                break;
            const int tb = 64;
            const dim3 grid((unsigned)((c.B + tb - 1) / tb));
            KTime kt(c.s, "sequential", "", 0);
            if (c.p->form == PSS_FORM_COV)
                hipLaunchKernelGGL((k_sequential_cov<T, NX, NY>), grid, dim3(tb), 0, c.s,
                                   c.p->y_off, c.B, c.T_y, gamma_ref(g, c.T_y), cptr<T>(y),
                                   cptr<T>(c.p->m0), cptr<T>(c.p->N0), marg_ref2(mf, Nf, c.T_x),
                                   marg_ref2(m_nom, N_nom, c.T_x));
            else if constexpr (NX == 1) // scalar state: one thread per sequence
                hipLaunchKernelGGL((k_sequential_1t<T, NX, NY>), grid, dim3(tb), 0, c.s,
                                   c.p->y_off, c.B, c.T_y, gamma_ref(g, c.T_y), cptr<T>(y),
                                   cptr<T>(c.p->m0), cptr<T>(c.p->N0), marg_ref2(mf, Nf, c.T_x),
                                   marg_ref2(m_nom, N_nom, c.T_x));
            else // one wavefront per sequence
                hipLaunchKernelGGL((k_sequential<T, NX, NY>), dim3((unsigned)c.B), dim3(64), 0, c.s,
                                   c.p->y_off, c.B, c.T_y, gamma_ref(g, c.T_y), cptr<T>(y),
                                   cptr<T>(c.p->m0), cptr<T>(c.p->N0), marg_ref2(mf, Nf, c.T_x),
                                   marg_ref2(m_nom, N_nom, c.T_x));
            rc = hip_check(hipGetLastError(), "sequential launch");
        }
        return rc;
    }
};

template <typename T>
static bool rule_spec(const pss_problem *p, int nx, RuleSpec<T> &R)
{
    RuleHost h;
    if (!rule_host(p, nx, h))
        return false;
    R.kind = h.kind;
    R.np = h.np;
    R.p = h.p;
    R.w0 = (T)h.w0;
    R.wi = (T)h.wi;
    R.spread = (T)h.spread;
    for (int q = 0; q < kMaxGH; ++q) {
        R.gx[q] = (T)h.gx[q];
        R.gw[q] = (T)h.gw[q];
    }
    return true;
}

// device-side CT constants in the kernel's precision
template <typename T>
CTParams<T> ct_params(const CTHost &h)
{
    CTParams<T> P;
    P.dt = (T)h.dt;
    P.s1x = (T)h.s1x;
    P.s1y = (T)h.s1y;
    P.s2x = (T)h.s2x;
    P.s2y = (T)h.s2y;
    P.sigma = (T)h.sigma;
    for (int i = 0; i < 5; ++i)
        for (int j = 0; j < 5; ++j)
            P.LQ[i][j] = (T)h.LQ[i][j];
    return P;
}

template <typename T, int NX, int NY>
int Core<T, NX, NY>::slr_felem(const Ctx &c, const void *m, const void *N, const void *y,
                               const pss_gamma *g, const pss_felem *el, bool cov,
                               bool store_obs)
{
    if constexpr (NX == 5 && NY == 2 && std::is_same_v<T, float>) {
        const int lin = c.p->linearization;
        if (c.p->model == PSS_MODEL_CT_BEARINGS &&
            (lin == PSS_LIN_CUBATURE || lin == PSS_LIN_TAYLOR)) {
            const CTParams<T> P = ct_params<T>(ct_host(c.p));
            const ScanShape sh = filter_shape(c);
            FElemRef<T, NX> er;
            er.A = mptr<T>(el->A);
            er.b = mptr<T>(el->b);
            er.U = mptr<T>(el->U);
            er.eta = mptr<T>(el->eta);
            er.Z = mptr<T>(el->Z);
            er.ld = c.T_y;
            const int tb = 256; // one level-0 filter tile per block, as felem
            const dim3 grid((unsigned)((c.T_y + tb - 1) / tb));
            const int taylor = lin == PSS_LIN_TAYLOR ? 1 : 0;
            KTime kt(c.s, "slr_felem", "", 0);
            if (cov)
                hipLaunchKernelGGL((k_slr_felem_ct<T, true>), grid, dim3(tb), 0, c.s, c.p->y_off,
                                   c.B, c.T_y, P, marg_ref2(m, N, c.T_x), cptr<T>(y),
                                   cptr<T>(c.p->m0), cptr<T>(c.p->N0), gamma_ref(g, c.T_y),
                                   store_obs ? 1 : 0, er, sh.T[0], sh.E[0], taylor, 1,
                                   c.dev_m ? 1 : 0);
            else
                hipLaunchKernelGGL((k_slr_felem_ct<T, false>), grid, dim3(tb), 0, c.s,
                                   c.p->y_off, c.B, c.T_y, P, marg_ref2(m, N, c.T_x), cptr<T>(y),
                                   cptr<T>(c.p->m0), cptr<T>(c.p->N0), gamma_ref(g, c.T_y),
                                   store_obs ? 1 : 0, er, sh.T[0], sh.E[0], taylor, 0,
                                   c.dev_m ? 1 : 0);
            return hip_check(hipGetLastError(), "slr + filter elements launch");
        }
    }
    return 1;
}

template <typename T, int NX, int NY>
int Core<T, NX, NY>::step_lin(const Ctx &c, const NomRef<T, NX> &nom, const void *y,
                              const pss_gamma *out, const ScanShape &sh)
{
    const dim3 grid((unsigned)((c.T_y + 255) / 256), 2), block(256);
    const int lin = c.p->linearization, dev = c.dev_m ? 1 : 0;
    const StepTiles tiles = step_tiles(sh);
    auto run = [&](const auto &l) -> int {
        using Lin = std::decay_t<decltype(l)>;
        KTime kt(c.s, "slr", "", 0);
        hipLaunchKernelGGL((k_step_lin<Lin>), grid, block, 0, c.s, c.p->y_off, c.B, c.T_y, l, nom,
                           cptr<T>(y), gamma_ref(out, c.T_y), tiles, dev);
        return hip_check(hipGetLastError(), "slr launch");
    };
    if constexpr (NX == 5 && NY == 2) {
        if (c.p->model == PSS_MODEL_CT_BEARINGS) {
            const CTParams<T> P = ct_params<T>(ct_host(c.p));
            if (lin == PSS_LIN_CUBATURE)
                return run(LinCT<T, false>{P});
            if (lin == PSS_LIN_TAYLOR)
                return run(LinCT<T, true>{P});
            LinCTRule<T> l{P, {}};
            if (!rule_spec(c.p, NX, l.R))
                return PSS_EINVAL;
            return run(l);
        }
    }
    if constexpr (NX == 1 && NY == 1) {
        if (c.p->model == PSS_MODEL_RICKER_POISSON) {
            const RickerHost h = ricker_host(c.p);
            LinRicker<T> l{};
            l.P.loga = (T)h.loga;
            l.P.b = (T)h.b;
            l.P.sqQ = (T)h.sqQ;
            l.taylor = lin == PSS_LIN_TAYLOR ? 1 : 0;
            if (!l.taylor && !rule_spec(c.p, NX, l.R))
                return PSS_EINVAL;
            return run(l);
        }
    }
    (void)y;
    set_error("no linearisation is built for this model and dimension pair");
    return PSS_EUNSUPPORTED;
}

template <typename T, int NX, int NY>
int Core<T, NX, NY>::slr(const Ctx &c, const void *m, const void *N, const void *y,
                         const pss_gamma *out)
{
    const int tb = 128;
    const dim3 grid((unsigned)((c.T_x + tb - 1) / tb));
    const int lin = c.p->linearization;
    const int cov = c.p->form == PSS_FORM_COV ? 1 : 0;
    if constexpr (NX == 5 && NY == 2) {
        if (c.p->model == PSS_MODEL_CT_BEARINGS) {
            const CTParams<T> P = ct_params<T>(ct_host(c.p));
            if (lin == PSS_LIN_CUBATURE || lin == PSS_LIN_TAYLOR) {
                KTime kt(c.s, "slr", "", 0);
                hipLaunchKernelGGL((k_slr_ct<T>), grid, dim3(tb), 0, c.s, c.p->y_off, c.B, c.T_x,
                                   c.T_y, P, marg_ref2(m, N, c.T_x), cptr<T>(y),
                                   gamma_ref(out, c.T_y), lin == PSS_LIN_TAYLOR ? 1 : 0, cov,
                                   c.dev_m ? 1 : 0);
            } else {
                RuleSpec<T> R;
                if (!rule_spec(c.p, NX, R))
                    return PSS_EINVAL;
                KTime kt(c.s, "slr", "", 0);
                hipLaunchKernelGGL((k_slr_ct_rule<T>), grid, dim3(tb), 0, c.s, c.p->y_off, c.B,
                                   c.T_x, c.T_y, P, marg_ref2(m, N, c.T_x), cptr<T>(y),
                                   gamma_ref(out, c.T_y), R, cov, c.dev_m ? 1 : 0);
            }
            return hip_check(hipGetLastError(), "slr launch");
        }
    }
    if constexpr (NX == 1 && NY == 1) {
        if (c.p->model == PSS_MODEL_RICKER_POISSON) {
            const RickerHost h = ricker_host(c.p);
            RickerParams<T> P;
            P.loga = (T)h.loga;
            P.b = (T)h.b;
            P.sqQ = (T)h.sqQ;
            RuleSpec<T> R{};
            if (lin != PSS_LIN_TAYLOR && !rule_spec(c.p, NX, R))
                return PSS_EINVAL;
            KTime kt(c.s, "slr", "", 0);
            hipLaunchKernelGGL((k_slr_ricker<T>), grid, dim3(tb), 0, c.s, c.p->y_off, c.B, c.T_x, P,
                               marg_ref2(m, N, c.T_x), gamma_ref(out, c.T_y),
                               lin == PSS_LIN_TAYLOR ? 1 : 0, R, cov);
            return hip_check(hipGetLastError(), "slr launch");
        }
    }
    (void)y;
    set_error("no linearisation is built for this model and dimension pair");
    return PSS_EUNSUPPORTED;
}

template <typename T, int NX, int NY>
int Core<T, NX, NY>::grad_terms(const Ctx &c, const pss_gamma *g, const void *y, const void *mf,
                                const void *Nf, const void *ms, const void *Ns, double *gterms)
{
    if constexpr (NX == 5 && NY == 2) {
        const CTHost h = ct_host(c.p);
        CTGradParams<T> gp;
        for (int i = 0; i < 5; ++i)
            for (int j = 0; j < 5; ++j) {
                gp.L1[i][j] = (T)h.L1[i][j];
                gp.L2[i][j] = (T)h.L2[i][j];
            }
        gp.sig2 = (T)(h.sigma * h.sigma);
        const int tb = 128;
        KTime kt(c.s, "grad_terms", "", 0);
        hipLaunchKernelGGL((k_grad_ct<T>), dim3((unsigned)((c.T_y + tb - 1) / tb)), dim3(tb), 0,
                           c.s, c.p->y_off, c.B, c.T_y, gamma_ref(g, c.T_y), cptr<T>(y),
                           marg_ref2(mf, Nf, c.T_x), marg_ref2(ms, Ns, c.T_x), gp, gterms);
        return hip_check(hipGetLastError(), "grad launch");
    } else {
        set_error("the gradient needs the coordinated-turn model");
        return PSS_EUNSUPPORTED;
    }
}

// forwarding definitions of the public per-dimension interface
template <typename T, int NX, int NY>
size_t Impl<T, NX, NY>::ws_size(const Ctx &c, int op) { return Core<T, NX, NY>::ws_size(c, op); }
template <typename T, int NX, int NY>
int Impl<T, NX, NY>::slr(const Ctx &c, const void *m, const void *N, const void *y,
                         const pss_gamma *out)
{
    return Core<T, NX, NY>::slr(c, m, N, y, out);
}
template <typename T, int NX, int NY>
int Impl<T, NX, NY>::felem(const Ctx &c, const pss_gamma *g, const void *y, const pss_felem *out)
{
    return Core<T, NX, NY>::felem(c, g, y, out);
}
template <typename T, int NX, int NY>
int Impl<T, NX, NY>::fscan(const Ctx &c, const pss_felem *el, void *mf, void *Nf, void *ws)
{
    return Core<T, NX, NY>::fscan(c, el, mf, Nf, ws);
}
template <typename T, int NX, int NY>
int Impl<T, NX, NY>::sscan(const Ctx &c, const pss_gamma *g, const void *mf, const void *Nf,
                           void *ms, void *Ns, void *ws)
{
    return Core<T, NX, NY>::sscan(c, g, mf, Nf, ms, Ns, ws);
}
template <typename T, int NX, int NY>
int Impl<T, NX, NY>::ipls(const Ctx &c, const pss_gamma *g, const void *y, int n_iter,
                          void *m_nom, void *N_nom, void *mf_out, void *Nf_out, void *ws)
{
    return Core<T, NX, NY>::ipls(c, g, y, n_iter, m_nom, N_nom, mf_out, Nf_out, ws);
}
template <typename T, int NX, int NY>
size_t Impl<T, NX, NY>::tiles_bytes(const Ctx &c, const TileChain &tc)
{
    return Core<T, NX, NY>::tiles_bytes(c, tc);
}
template <typename T, int NX, int NY>
int Impl<T, NX, NY>::ipls_tiles(const Ctx &c, const TileChain &tc, const void *y, int n_iter,
                                void *m_nom, void *N_nom, void *ws)
{
    return Core<T, NX, NY>::ipls_tiles(c, tc, y, n_iter, m_nom, N_nom, ws);
}
template <typename T, int NX, int NY>
int Impl<T, NX, NY>::loglik(const Ctx &c, const pss_gamma *g, const void *m_nom,
                            const void *N_nom, const void *y, double *ll, const pss_ckpt *ckpt,
                            void *ws)
{
    return Core<T, NX, NY>::loglik(c, g, m_nom, N_nom, y, ll, ckpt, ws);
}
template <typename T, int NX, int NY>
int Impl<T, NX, NY>::loglik_grad(const Ctx &c, const void *m_nom, const void *N_nom,
                                 const void *y, const double *ll_bar, const pss_ckpt *ckpt,
                                 double *ll, double *grad, double *theta_bar, void *ws)
{
    return Core<T, NX, NY>::loglik_grad(c, m_nom, N_nom, y, ll_bar, ckpt, ll, grad, theta_bar,
                                        ws);
}
template <typename T, int NX, int NY>
int Impl<T, NX, NY>::loglik_vjp(const Ctx &c, const pss_gamma *g, const void *m_nom,
                                const void *N_nom, const void *y, const double *ll_bar,
                                const pss_ckpt *ckpt, double *ll, const pss_gamma *gbar,
                                void *m0_bar, void *N0_bar, void *ws)
{
    return Core<T, NX, NY>::loglik_vjp(c, g, m_nom, N_nom, y, ll_bar, ckpt, ll, gbar, m0_bar,
                                       N0_bar, ws);
}
template <typename T, int NX, int NY>
int Impl<T, NX, NY>::score_fisher(const Ctx &c, const void *m_nom, const void *N_nom,
                                  const void *y, const double *ll_bar, double *ll, double *grad,
                                  double *theta_bar, void *ws)
{
    return Core<T, NX, NY>::score_fisher(c, m_nom, N_nom, y, ll_bar, ll, grad, theta_bar, ws);
}
template <typename T, int NX, int NY>
size_t Impl<T, NX, NY>::ckpt_bytes(const Ctx &c, int level)
{
    return Core<T, NX, NY>::ckpt_bytes(c, level);
}
template <typename T, int NX, int NY>
int Impl<T, NX, NY>::filter_levels(const Ctx &c)
{
    return Core<T, NX, NY>::filter_levels(c);
}
template <typename T, int NX, int NY>
int Impl<T, NX, NY>::sequential(const Ctx &c, const pss_gamma *g, const void *y, int n_iter,
                                void *m_nom, void *N_nom, void *mf_out, void *Nf_out, void *ws)
{
    return Core<T, NX, NY>::sequential(c, g, y, n_iter, m_nom, N_nom, mf_out, Nf_out, ws);
}

} // namespace pss
