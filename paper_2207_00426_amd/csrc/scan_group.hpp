// Levels of a scan above the finest, one element per group of 16 lanes
// (device_group.hpp).
//
// A tile of a level (the plan's T x E consecutive elements of one sequence) is
// handled by a block of kGroups groups.  Each group folds ceil(count /
// kGroups) consecutive elements, then the groups' aggregates are scanned in LDS in
// log2(kGroups) steps that leave the inclusive prefix of every group (half of
// the groups combine per step, packed onto the first waves).  A lower level
// saves those inclusive elements; its second half starts every group with one
// apply of the tile's exclusive prefix to its left neighbour's saved element
// -- no down-sweep -- and walks the group's elements.  32 groups are two waves
// on each SIMD of a CU: one wave alone leaves half of its issue slots empty, and
// more would share them.  The bracketing depends only on the sequence's own
// length, and so does the rounding: what a lower level stores between its halves
// in FP32, the top level rounds likewise, so that a sequence's result does not
// show whether a longer one in its batch made its top level a lower one.
#pragma once

#include "device_group.hpp"
#include "kernels.hpp"

namespace pss {

constexpr int kGroups = 32;
constexpr int kGroupThreads = kGroups * grp::kLanes;

// elements and marginals stored whole, one after the other: what a group
// reads and writes is contiguous
template <typename T, int NX>
struct FAosRef {
    T *p;
};
template <typename T, int NX>
struct SAosRef {
    T *p;
};
template <typename T, int NX>
PSS_INL FSlotV<T, NX, int> view_of(const FAosRef<T, NX> &r, int64_t t)
{
    return FSlotV<T, NX, int>{r.p + t * Sizes<NX>::felem, 1};
}
template <typename T, int NX>
PSS_INL SSlotV<T, NX, int> view_of(const SAosRef<T, NX> &r, int64_t t)
{
    return SSlotV<T, NX, int>{r.p + t * Sizes<NX>::selem, 1};
}
template <typename T, int NX>
struct MargAos {
    T *p;
    PSS_INL void load(int64_t t, Marg<T, NX> &x) const
    {
        const T *q = p + t * Sizes<NX>::marg;
        visit(x, [&](int c, T &v) { v = q[c]; });
    }
};

// the operators of a scan in group form; scans without one keep one element
// per lane at every level
template <class Op>
struct GroupOp {
    static constexpr bool value = false;
};
template <typename T, int NX>
struct GroupOp<FilterScan<T, NX>> {
    static constexpr bool value = NX >= 2;
    using Ref = FAosRef<T, NX>;
    static __device__ __forceinline__ void combine(const double *a, const double *b, double *o,
                                                   const grp::Lane<NX> &ln)
    {
        grp::filter_combine<double, NX>(a, b, o, ln);
    }
    static __device__ __forceinline__ void apply(const double *p, const double *a, double *o,
                                                 const grp::Lane<NX> &ln)
    {
        grp::filter_apply<double, NX>(p, a, o, ln);
    }
};
template <typename T, int NX>
struct GroupOp<SmootherScan<T, NX>> {
    static constexpr bool value = NX >= 2;
    using Ref = SAosRef<T, NX>;
    static __device__ __forceinline__ void combine(const double *a, const double *b, double *o,
                                                   const grp::Lane<NX> &ln)
    {
        grp::smoother_combine<double, NX>(b, a, o, ln);
    }
    static __device__ __forceinline__ void apply(const double *p, const double *a, double *o,
                                                 const grp::Lane<NX> &ln)
    {
        grp::smoother_apply<double, NX>(a, p, o, ln);
    }
};

// N contiguous values moved by the 16 lanes of a group, through registers
template <typename T, int N>
struct GroupMove {
    static constexpr int K = (N + grp::kLanes - 1) / grp::kLanes;
    T v[K];
    template <typename S>
    __device__ __forceinline__ void load(const S *p)
    {
        const int l = threadIdx.x & (grp::kLanes - 1);
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (l + k * grp::kLanes < N)
                v[k] = T(p[l + k * grp::kLanes]);
    }
    template <typename D>
    __device__ __forceinline__ void store(D *p) const
    {
        const int l = threadIdx.x & (grp::kLanes - 1);
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (l + k * grp::kLanes < N)
                p[l + k * grp::kLanes] = D(v[k]);
    }
};

struct GroupGeom {
    const int64_t *elem_off; // this level's element offsets [B + 1]
    const int64_t *tile_off; // this level's tile offsets [B + 1]
    int B;
    int TS; // elements of a full tile
};

struct GroupTile {
    int64_t first; // the tile's first element
    int b, cnt, E, nvalid;
};

__device__ __forceinline__ GroupTile group_tile(const GroupGeom &g)
{
    GroupTile t;
    t.b = find_seq(g.tile_off, g.B, blockIdx.x, 0);
    const int64_t at = ((int64_t)blockIdx.x - g.tile_off[t.b]) * g.TS;
    const int64_t rem = g.elem_off[t.b + 1] - g.elem_off[t.b] - at;
    t.first = g.elem_off[t.b] + at;
    t.cnt = (int)(rem < g.TS ? rem : g.TS);
    t.E = (t.cnt + kGroups - 1) / kGroups;
    t.nvalid = (t.cnt + t.E - 1) / t.E;
    return t;
}

// fold and in-tile scan: on return slot g of `acc` (g < nvalid) holds the
// inclusive prefix of group g within the tile; ends with a block barrier
template <class Op>
__device__ __forceinline__ void group_up(const GroupTile &ti, const typename Op::T *elems,
                                         double *acc, double *in, const grp::Lane<Op::NX> &ln)
{
    using T = typename Op::T;
    constexpr int NE = Op::NE;
    const int g = threadIdx.x / grp::kLanes;
    if (g < ti.nvalid) {
        const int p0 = g * ti.E, pe = p0 + ti.E < ti.cnt ? p0 + ti.E : ti.cnt;
        const T *src = elems + (ti.first + p0) * NE;
        double *a = acc + g * NE, *x = in + g * NE;
        GroupMove<T, NE> mv;
        mv.load(src);
        mv.store(a);
        if (p0 + 1 < pe)
            mv.load(src + NE);
        for (int p = p0 + 1; p < pe; ++p) {
            mv.store(x);
            grp::lds_order();
            src += NE;
            if (p + 1 < pe) // the next element is on its way during this combine
                mv.load(src + NE);
            GroupOp<Op>::combine(a, x, a, ln);
        }
    }
    for (int k = 0; (1 << k) < ti.nvalid; ++k) {
        __syncthreads();
        const int t = ((g >> k) << (k + 1)) | (1 << k) | (g & ((1 << k) - 1));
        if (g < kGroups / 2 && t < ti.nvalid) {
            const int l = ((t >> k) << k) - 1;
            GroupOp<Op>::combine(acc + l * NE, acc + t * NE, acc + t * NE, ln);
        }
    }
    __syncthreads();
}

// the group's start prefix p (in LDS), then its elements' exclusive prefixes
template <class Op>
__device__ __forceinline__ void group_walk(const GroupTile &ti, const typename Op::T *elems,
                                           typename Op::T *pre_out, double *p, double *x,
                                           const grp::Lane<Op::NX> &ln)
{
    using T = typename Op::T;
    constexpr int NE = Op::NE, NP = Op::NP;
    const int g = threadIdx.x / grp::kLanes;
    const int p0 = g * ti.E, pe = p0 + ti.E < ti.cnt ? p0 + ti.E : ti.cnt;
    const T *src = elems + (ti.first + p0) * NE;
    T *dst = pre_out + (ti.first + p0) * NP;
    GroupMove<T, NE> mv;
    if (p0 + 1 < pe)
        mv.load(src);
    for (int q = p0;; ++q) {
        GroupMove<double, NP> out;
        out.load(p);
        out.store(dst);
        if (q + 1 >= pe)
            break;
        mv.store(x);
        grp::lds_order();
        src += NE;
        dst += NP;
        if (q + 2 < pe)
            mv.load(src);
        GroupOp<Op>::apply(p, x, p, ln);
    }
}

// lower levels, first half: saves every group's inclusive element and the
// tile's aggregate (an element of the next level)
template <class Op>
__global__ __launch_bounds__(kGroupThreads) void k_group_up(GroupGeom gm,
                                                            const typename Op::T *elems,
                                                            typename Op::T *agg,
                                                            typename Op::T *incl)
{
    using T = typename Op::T;
    __shared__ double acc[kGroups * Op::NE], in[kGroups * Op::NE];
    const grp::Lane<Op::NX> ln;
    const GroupTile ti = group_tile(gm);
    group_up<Op>(ti, elems, acc, in, ln);
    T *out = incl + (int64_t)blockIdx.x * kGroups * Op::NE;
    for (int i = threadIdx.x; i < ti.nvalid * Op::NE; i += kGroupThreads)
        out[i] = T(acc[i]);
    for (int i = threadIdx.x; i < Op::NE; i += kGroupThreads)
        agg[(int64_t)blockIdx.x * Op::NE + i] = T(acc[(ti.nvalid - 1) * Op::NE + i]);
}

// lower levels, second half
template <class Op>
__global__ __launch_bounds__(kGroupThreads) void k_group_down(GroupGeom gm,
                                                              const typename Op::T *elems,
                                                              const typename Op::T *incl,
                                                              const typename Op::T *pre_in,
                                                              typename Op::T *pre_out)
{
    using T = typename Op::T;
    __shared__ double pre[kGroups * Op::NP], in[kGroups * Op::NE];
    const grp::Lane<Op::NX> ln;
    const GroupTile ti = group_tile(gm);
    const int g = threadIdx.x / grp::kLanes;
    if (g >= ti.nvalid)
        return;
    double *p = pre + g * Op::NP, *x = in + g * Op::NE;
    GroupMove<T, Op::NP> root;
    root.load(pre_in + (int64_t)blockIdx.x * Op::NP);
    root.store(p);
    if (g > 0) {
        GroupMove<T, Op::NE> mv;
        mv.load(incl + ((int64_t)blockIdx.x * kGroups + g - 1) * Op::NE);
        mv.store(x);
        grp::lds_order();
        GroupOp<Op>::apply(p, x, p, ln);
    }
    grp::lds_order();
    group_walk<Op>(ti, elems, pre_out, p, x, ln);
}

// top level (one tile per sequence): both halves
template <class Op, class Start>
__global__ __launch_bounds__(kGroupThreads) void k_group_top(GroupGeom gm,
                                                             const typename Op::T *elems,
                                                             typename Op::T *pre_out,
                                                             Start start)
{
    using T = typename Op::T;
    __shared__ double acc[kGroups * Op::NE], in[kGroups * Op::NE], pre[kGroups * Op::NP];
    const grp::Lane<Op::NX> ln;
    const GroupTile ti = group_tile(gm);
    group_up<Op>(ti, elems, acc, in, ln);
    const int g = threadIdx.x / grp::kLanes;
    if (g >= ti.nvalid)
        return;
    double *p = pre + g * Op::NP, *x = in + g * Op::NE;
    if ((threadIdx.x & (grp::kLanes - 1)) == 0) {
        Marg<T, Op::NX> s;
        start.get(s);
        visit(s, [&](int c, T &v) { p[c] = double(v); });
    }
    const double *left = acc + (g - 1) * Op::NE;
    if constexpr (sizeof(T) == 4) { // as k_group_down takes it: rounded
        if (g > 0) {
            GroupMove<T, Op::NE> mv;
            mv.load(left);
            mv.store(x);
            left = x;
        }
    }
    grp::lds_order();
    if (g > 0)
        GroupOp<Op>::apply(p, left, p, ln);
    group_walk<Op>(ti, elems, pre_out, p, x, ln);
}

} // namespace pss
