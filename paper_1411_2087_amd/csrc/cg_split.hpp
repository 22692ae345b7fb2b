// The CG iteration on small lattices: two kernels (three on the larger of
// them), one 64-site tile per workgroup (SplitTerms).
//
// On a few hundred tiles an iteration is launches and latency, not bytes: at
// 8^4 the five kernels of the large-lattice iteration (two Dslashes with their
// epilogues, two one-workgroup finalisers, the direction update) took 39 us
// for 10 MB.  Here
//   k_cgs_Dp   every workgroup sums the |r|^2 partials of the previous
//              iteration itself and finishes it (convergence, beta) in
//              registers, t = D_oe r + beta D_oe p (which is D_oe p_new,
//              p_new = r + beta p, with products that do not wait for
//              beta), and leaves the partial of <p, A p> =
//              4 m^2 |p_new|^2 + |t|^2 of its tile;
//   k_cgs_upd  every workgroup sums those (alpha), A p = 4 m^2 p_new - D_eo t
//              in registers, p = p_new, x += alpha p, r -= alpha A p, and
//              the |r|^2 partial of its tile.
// Beyond 512 tiles the direction update is a kernel of its own again (k_cgs_p,
// which then finishes the previous iteration), see SplitIter.
// The sums run while the tile's link and vector loads are in flight.  All
// workgroups read the same partials in the same order, so they agree to the
// bit.  The state is read from one copy and written to the other (k_cgs_Dp:
// s0 -> s1, k_cgs_upd: s1 -> s0, by one thread), so no workgroup reads what
// another writes; `pending` says that the |r|^2 partials have not been folded
// in, which k_cgs_settle does before the host looks at the state.
#pragma once

#include "cg_internal.hpp"
#include "split_sums.hpp"

namespace hisq {

// FUSE: the direction update is part of this kernel (and of k_cgs_upd); else
// k_cgs_p has run, p is p_new and s1 is current.
template <class P, bool KEEP, bool FUSE>
__global__ __launch_bounds__(SPLIT_NT) void k_cgs_Dp(Geom g, const char *__restrict__ fat,
                                                     const char *__restrict__ lng,
                                                     const typename P::real *__restrict__ r,
                                                     const typename P::real *__restrict__ p,
                                                     typename P::real *__restrict__ t,
                                                     const double *__restrict__ part_rr,
                                                     double *__restrict__ part_pap, const CGState *__restrict__ s0,
                                                     CGState *__restrict__ s1, int mode)
{
    using T = SplitTerms<P, KEEP>;
    using R = typename P::real;
    using V = typename P::cvec;
    __shared__ __align__(16) R red[SPLIT * TILE_REALS];
    __shared__ double lds[SPLIT], ldp[SPLIT];
    const int tile = xcd_block(blockIdx.x, gridDim.x);  // workgroup 0 has tile 0
    if (tile >= g.ntiles) return;
    // Every load is issued before the state is looked at (it is behind the
    // same latency); the pause is acted on after the first barrier.
    const bool lead = blockIdx.x == 0 && threadIdx.x == 0;
    CGState st;
    double rr[1] = { 0.0 };
    if constexpr (FUSE) {
        st = *s0;
        strided_sums<SPLIT_NT, 1, 2>(part_rr, g.ntiles, rr);
    } else if (paused(s1->flags)) {
        return;
    }
    const int lane = threadIdx.x & 63, q = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int h = tile * TILE + lane;
    T terms;
    terms.load(g, fat, lng, 1, tile, lane, h < g.Vh ? h : g.Vh - 1, q);
    V pf[3], pl[3];
    [[maybe_unused]] V rf[3], rl[3];
    const V *rv = reinterpret_cast<const V *>(r), *pv = reinterpret_cast<const V *>(p);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if constexpr (FUSE) rf[a] = rv[(size_t)terms.nf * 3 + a];
        pf[a] = pv[(size_t)terms.nf * 3 + a];
        if constexpr (FUSE) rl[a] = rv[(size_t)terms.nl * 3 + a];
        pl[a] = pv[(size_t)terms.nl * 3 + a];
    }
    const int i = threadIdx.x;
    const bool own = i < min(TILE_REALS, (g.Vh - tile * TILE) * 6);
    const size_t at = (size_t)tile * TILE_REALS + i;
    R ro = 0, po = 0;
    if (own) {
        if constexpr (FUSE) ro = r[at];
        po = p[at];
    }
    R acc[6], beta = 0;
    terms.products(pf, pl, acc);
    if constexpr (FUSE) {
        // D p_new = D r + beta D p: the products do not wait for beta
        R accr[6];
        terms.products(rf, rl, accr);
        const double total = split_total(rr[0], lds);
        if (!paused(st.flags) && st.pending) {
            st.pending = 0;
            finalize(&st, mode, total);
        }
        if (lead) *s1 = st;
        if (paused(st.flags)) return;
        beta = (R)st.beta;
#pragma unroll
        for (int a = 0; a < 6; ++a) acc[a] = fma(beta, acc[a], accr[a]);
    }
    T::put(acc, q, lane, red);
    __syncthreads();
    double s = 0.0;
    if (own) {
        const double tv = T::result(red, i), pn = FUSE ? fma(beta, po, ro) : po;
        __builtin_nontemporal_store((R)tv, t + at);
        s = fma((FUSE ? st.m4 : s1->m4) * pn, pn, tv * tv);
    }
    split_partial(s, ldp, part_pap + tile);
}

template <class P, bool KEEP, bool FUSE>
__global__ __launch_bounds__(SPLIT_NT) HISQ_WAVES(4) void k_cgs_upd(Geom g, const char *__restrict__ fat,
                                                      const char *__restrict__ lng,
                                                      const typename P::cvec *__restrict__ t,
                                                      typename P::real *__restrict__ p,
                                                      typename P::real *__restrict__ x,
                                                      typename P::real *__restrict__ r,
                                                      const double *__restrict__ part_pap,
                                                      double *__restrict__ part_rr, const CGState *__restrict__ s1,
                                                      CGState *__restrict__ s0)
{
    using T = SplitTerms<P, KEEP>;
    using R = typename P::real;
    using V = typename P::cvec;
    __shared__ __align__(16) R red[SPLIT * TILE_REALS];
    __shared__ double lds[SPLIT], ldp[SPLIT];
    const int tile = xcd_block(blockIdx.x, gridDim.x);
    if (tile >= g.ntiles) return;
    const bool lead = blockIdx.x == 0 && threadIdx.x == 0;
    const bool closed = paused(s1->flags);
    if (!FUSE && closed) {  // a paused iteration costs its launches only; the smallest lattices gain more from not waiting
        if (lead) *s0 = *s1;
        return;
    }
    const double rr = s1->rr, m4 = s1->m4, beta = s1->beta;
    double pap[1] = { 0.0 };
    strided_sums<SPLIT_NT, 1, 2>(part_pap, g.ntiles, pap);
    const int lane = threadIdx.x & 63, q = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int h = tile * TILE + lane;
    T terms;
    terms.load(g, fat, lng, 0, tile, lane, h < g.Vh ? h : g.Vh - 1, q);
    V f[3], l[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        f[a] = t[(size_t)terms.nf * 3 + a];
        l[a] = t[(size_t)terms.nl * 3 + a];
    }
    const int i = threadIdx.x;
    const bool own = i < min(TILE_REALS, (g.Vh - tile * TILE) * 6);
    const size_t at = (size_t)tile * TILE_REALS + i;
    R po = 0, xo = 0, ro = 0;
    if (own) {
        po = p[at];
        xo = x[at];
        ro = r[at];
    }
    R acc[6];
    terms.products(f, l, acc);
    T::put(acc, q, lane, red);
    const double total = split_total(pap[0], lds);  // its barrier also publishes `red`
    if (lead) {
        *s0 = *s1;
        if (!closed) {
            finalize(s0, FIN_PAP, total);
            s0->pending = s0->flags.done ? 0 : 1;
        }
    }
    if (closed || !(total > 0.0) || !isfinite(total)) return;  // as FIN_PAP decides
    double s = 0.0;
    if (own) {
        const R a = (R)(rr / total);
        const R pn = FUSE ? fma((R)beta, po, ro) : po;
        const R ap = fma((R)m4, pn, -T::result(red, i));
        xo = fma(a, pn, xo);
        ro = fma(-a, ap, ro);
        if constexpr (FUSE) __builtin_nontemporal_store(pn, p + at);
        __builtin_nontemporal_store(xo, x + at);
        __builtin_nontemporal_store(ro, r + at);
        s = (double)ro * (double)ro;
    }
    split_partial(s, ldp, part_rr + tile);
}

// The direction update of the three-kernel form: finishes the previous
// iteration as k_cgs_Dp does, then p = r + beta p; entries of 16 bytes.
template <class P>
__global__ __launch_bounds__(SPLIT_NT) void k_cgs_p(float4 *__restrict__ p, const float4 *__restrict__ r,
                                                    long long n16, const double *__restrict__ part_rr, int nparts,
                                                    const CGState *__restrict__ s0, CGState *__restrict__ s1, int mode)
{
    using R = typename P::real;
    constexpr int U = 4, W = 16 / sizeof(R);
    __shared__ double lds[SPLIT];
    CGState st = *s0;
    if (paused(st.flags)) {
        if (blockIdx.x == 0 && threadIdx.x == 0) *s1 = st;
        return;
    }
    double rr[1] = { 0.0 };
    strided_sums<SPLIT_NT, 1, 4>(part_rr, nparts, rr);
    union Q { float4 q; R e[W]; } pv[U], rv[U];
    const long long i0 = (long long)blockIdx.x * U * SPLIT_NT + threadIdx.x;
#pragma unroll
    for (int j = 0; j < U; ++j) {
        const long long i = i0 + j * SPLIT_NT;
        if (i < n16) { pv[j].q = p[i]; rv[j].q = r[i]; }
    }
    const double total = split_total(rr[0], lds);
    if (st.pending) {
        st.pending = 0;
        finalize(&st, mode, total);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) *s1 = st;
    if (paused(st.flags)) return;
    const R beta = (R)st.beta;
#pragma unroll
    for (int j = 0; j < U; ++j) {
        const long long i = i0 + j * SPLIT_NT;
        if (i >= n16) continue;
#pragma unroll
        for (int e = 0; e < W; ++e) pv[j].e[e] = fma(beta, pv[j].e[e], rv[j].e[e]);
        nf4 o = { pv[j].q.x, pv[j].q.y, pv[j].q.z, pv[j].q.w };
        __builtin_nontemporal_store(o, reinterpret_cast<nf4 *>(p + i));
    }
}

// The last iteration's |r|^2 into the state, before the host reads it.
__global__ __launch_bounds__(SPLIT_NT) void k_cgs_settle(const double *__restrict__ part_rr, int n, CGState *s0,
                                                         int mode)
{
    __shared__ double lds[SPLIT];
    if (paused(s0->flags) || !s0->pending) return;
    double rr[1] = { 0.0 };
    strided_sums<SPLIT_NT, 1, 2>(part_rr, n, rr);
    const double v = split_total(rr[0], lds);
    if (threadIdx.x == 0) {
        s0->pending = 0;
        finalize(s0, mode, v);
    }
}

// The split iteration of one solve: kernels and the scratch they share.
struct SplitIter {
    bool on = false, fuse = false;
    CGState *s0 = nullptr, *s1 = nullptr;
    double *part_pap = nullptr, *part_rr = nullptr;
    // The second state and the per-tile partials lie in `scratch`, which the
    // solve does not use between its state checks; off where they do not fit.
    void set(const Geom &g, int prec, CGState *st, void *scratch, size_t bytes)
    {
        const size_t n = sizeof(double) * g.ntiles, head = (sizeof(CGState) + 63) & ~(size_t)63;
        on = split_pays(g, prec) && head + 2 * n <= bytes;
        fuse = g.ntiles <= CG_FUSE_TILES;
        s0 = st;
        s1 = (CGState *)scratch;
        part_pap = (double *)((char *)scratch + head);
        part_rr = part_pap + g.ntiles;
    }
    // Milliseconds per solve (mass 0.08, tol 1e-10) with these two kernels,
    // these three, and FoldIter's three:
    //   tiles   FP64              FP64 two rows     FP32              FP32 two rows     16-bit two rows
    //    512    17.5 17.1 24.7    15.8 15.6 24.8    12.8 12.9 19.7    11.9 12.2 17.9    13.6 13.9 17.8
    //    640    21.5 19.8 25.6    19.5 18.2 25.5    15.2 14.3 20.0    14.2 13.4 18.3    14.9 14.5 18.1
    //    864    29.4 26.7 28.1    25.1 22.8 27.8    19.1 16.9 21.5    17.7 15.8 19.6    16.9 15.8 18.8
    //    896    32.0 29.4 28.2    25.0 22.4 27.5    18.8 16.6 20.8    17.4 15.2 19.1    16.9 15.9 18.9
    //   1024    35.0 32.8 31.0    27.5 25.2 29.2    21.2 18.9 21.6    19.4 17.1 20.7    18.4 17.2 20.1
    //   1088    37.2 35.4 46.0    33.9 31.9 41.0    21.5 19.6 24.4    20.0 17.8 23.5    20.6 19.3 24.4
    //   1280                                        23.7 21.4 25.9    21.6 19.3 24.6    21.8 20.1 25.5
    // Two kernels gather r and p instead of p_new, which costs bandwidth where
    // the launch they save no longer counts.  FP64 links leave the last-level
    // cache between 864 and 896 tiles (links_stay_cached), and the 8 streams
    // per tile then lose to FoldIter, until its workgroups of four tiles are
    // more than the 256 CUs.  The FP64 forms end at 1088 tiles because the
    // partials lie in the gaps of the plain workspace, which hold no more; the
    // mixed ones' scratch is larger.  The sums of all tiles' partials in every
    // workgroup grow with the square of the lattice, but 16-bit links still
    // gain at 2592 tiles (33.6 against 37.5): their line could be higher.
    static constexpr int CG_FUSE_TILES = 512;
    static bool split_pays(const Geom &g, int prec)
    {
        switch (prec) {
        case HISQ_F64: return g.ntiles <= 1088 && (g.ntiles > 1024 || links_stay_cached(g, prec));
        case HISQ_F64C: return g.ntiles <= 1088;
        default: return g.ntiles <= 1280;
        }
    }
    template <class P>
    hipError_t iteration(hipStream_t q, const Geom &g, const void *fat, const void *lng, void *r, void *p, void *t,
                         void *x, int mode) const
    {
        using R = typename P::real;
        if (fuse) return launch<P, true, true>(q, g, fat, lng, r, p, t, x, mode);
        const long long n16 = (long long)g.Vh * 6 * sizeof(R) / 16;  // Vh is a multiple of 8
        hipLaunchKernelGGL(k_cgs_p<P>, dim3((unsigned)((n16 + 4 * SPLIT_NT - 1) / (4 * SPLIT_NT))), dim3(SPLIT_NT), 0,
                           q, (float4 *)p, (const float4 *)r, n16, (const double *)part_rr, g.ntiles,
                           (const CGState *)s0, s1, mode);
        // only FP64 links leave the cache below the line, from 869 tiles (1042 with two rows)
        if constexpr (P::prec == HISQ_F64 || P::prec == HISQ_F64C)
            if (!links_stay_cached(g, P::prec)) return launch<P, false, false>(q, g, fat, lng, r, p, t, x, mode);
        return launch<P, true, false>(q, g, fat, lng, r, p, t, x, mode);
    }
    template <class P, bool KEEP, bool FUSE>
    hipError_t launch(hipStream_t q, const Geom &g, const void *fat, const void *lng, void *r, void *p, void *t,
                      void *x, int mode) const
    {
        using R = typename P::real;
        const dim3 grid(xcd_grid(g.ntiles)), nt(SPLIT_NT);
        hipLaunchKernelGGL((k_cgs_Dp<P, KEEP, FUSE>), grid, nt, 0, q, g, (const char *)fat, (const char *)lng,
                           (const R *)r, (const R *)p, (R *)t, (const double *)part_rr, part_pap, (const CGState *)s0,
                           s1, mode);
        hipLaunchKernelGGL((k_cgs_upd<P, KEEP, FUSE>), grid, nt, 0, q, g, (const char *)fat, (const char *)lng,
                           (const typename P::cvec *)t, (R *)p, (R *)x, (R *)r, (const double *)part_pap, part_rr,
                           (const CGState *)s1, s0);
        return hipGetLastError();
    }
    hipError_t settle(hipStream_t q, const Geom &g, int mode) const
    {
        if (!on) return hipSuccess;
        hipLaunchKernelGGL(k_cgs_settle, dim3(1), dim3(SPLIT_NT), 0, q, (const double *)part_rr, g.ntiles, s0, mode);
        return hipGetLastError();
    }
};

}  // namespace hisq
