// Per-site HISQ Dslash, shared by every kernel that applies the operator.
//
// Sec. 3 of the paper: at each site the operator reads 16 link matrices (a
// one-link and a three-link matrix for each of the 8 directions +-mu) and 16
// neighbour colour vectors, and sums 16 matrix-vector products.  The packed
// links already hold -U^dag for the backward directions, so every term is a
// plain product M_d(n) psi(n + k_d).
#pragma once

#include "hisq_common.hpp"

namespace hisq {

// Directions in the packed layout, per field: 0..3 = +x,+y,+z,+t ; 4..7 = -x,-y,-z,-t.
// Fat links hop 1 site, long links 3 sites.

template <class P>
__device__ __forceinline__ void cmac(typename P::real acc[6], const typename P::real m[18], typename P::cvec s0,
                                     typename P::cvec s1, typename P::cvec s2)
{
    const typename P::real sr[3] = { s0.x, s1.x, s2.x };
    const typename P::real si[3] = { s0.y, s1.y, s2.y };
#pragma unroll
    for (int a = 0; a < 3; ++a) {
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const typename P::real mr = m[2 * (3 * a + b)], mi = m[2 * (3 * a + b) + 1];
            acc[2 * a] = fma(mr, sr[b], acc[2 * a]);
            acc[2 * a] = fma(-mi, si[b], acc[2 * a]);
            acc[2 * a + 1] = fma(mr, si[b], acc[2 * a + 1]);
            acc[2 * a + 1] = fma(mi, sr[b], acc[2 * a + 1]);
        }
    }
}

// acc += M psi for a two-row matrix: rows 0 and 1 from m[0..11], row 2 =
// c conj(row0 x row1) taken one entry at a time straight into acc[4..5], so
// the third row is never held in registers.
template <class P>
__device__ __forceinline__ void cmac_two_row(typename P::real acc[6], const typename P::real m[12],
                                             typename P::real c, typename P::cvec s0, typename P::cvec s1,
                                             typename P::cvec s2)
{
    using R = typename P::real;
    const R sr[3] = { s0.x, s1.x, s2.x };
    const R si[3] = { s0.y, s1.y, s2.y };
#pragma unroll
    for (int a = 0; a < 2; ++a) {
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const R mr = m[2 * (3 * a + b)], mi = m[2 * (3 * a + b) + 1];
            acc[2 * a] = fma(mr, sr[b], acc[2 * a]);
            acc[2 * a] = fma(-mi, si[b], acc[2 * a]);
            acc[2 * a + 1] = fma(mr, si[b], acc[2 * a + 1]);
            acc[2 * a + 1] = fma(mi, sr[b], acc[2 * a + 1]);
        }
    }
    R tr = 0, ti = 0;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const int j1 = (j + 1) % 3, j2 = (j + 2) % 3;
        const R ar1 = m[2 * j1], ai1 = m[2 * j1 + 1], ar2 = m[2 * j2], ai2 = m[2 * j2 + 1];
        const R br1 = m[6 + 2 * j1], bi1 = m[6 + 2 * j1 + 1], br2 = m[6 + 2 * j2], bi2 = m[6 + 2 * j2 + 1];
        // x_j = a_{j+1} b_{j+2} - a_{j+2} b_{j+1}
        const R xr = (ar1 * br2 - ai1 * bi2) - (ar2 * br1 - ai2 * bi1);
        const R xi = (ar1 * bi2 + ai1 * br2) - (ar2 * bi1 + ai2 * br1);
        // conj(x_j) s_j
        tr = fma(xr, sr[j], tr);
        tr = fma(xi, si[j], tr);
        ti = fma(xr, si[j], ti);
        ti = fma(-xi, sr[j], ti);
    }
    acc[4] = fma(c, tr, acc[4]);
    acc[5] = fma(c, ti, acc[5]);
}

// acc = (D src)(h) for the site h of parity `parity` (h < Vh), whose links
// sit at lane `lane` of tile `tile`.  The 16 terms are taken UNR at a time:
// a fully unrolled body lets the compiler hoist every load and run out of
// registers, a partly unrolled one keeps UNR matrices in flight per thread
// and leaves the latency hiding to the other resident wavefronts.
template <class P, int UNR = 1>
__device__ __forceinline__ void dslash_site(const Geom &g, const char *__restrict__ fat,
                                            const char *__restrict__ lng,
                                            const typename P::cvec *__restrict__ src, int parity, int tile,
                                            int lane, int h, typename P::real acc[6])
{
    int x, y, z, t;
    site_coords(g, h, parity, x, y, z, t);
    const size_t tix = (size_t)parity * g.ntiles + tile;
    const char *fb = fat + tix * P::Fat::tile_bytes;
    const char *lb = lng + tix * P::Long::tile_bytes;
#pragma unroll
    for (int i = 0; i < 6; ++i) acc[i] = 0;
    // one-link terms, then three-link terms (separate loops keep one loader live)
#pragma unroll UNR
    for (int d = 0; d < 8; ++d) {
        const int nh = nbr_h(g, h, x, y, z, t, d & 3, (d >> 2) ? -1 : 1);
        typename P::real m[18];
        P::Fat::load_dir(fb, d, lane, m);
        const typename P::cvec *s = src + (size_t)nh * 3;
        cmac<P>(acc, m, s[0], s[1], s[2]);
    }
#pragma unroll UNR
    for (int d = 0; d < 8; ++d) {
        const int nh = nbr_h(g, h, x, y, z, t, d & 3, (d >> 2) ? -3 : 3);
        const typename P::cvec *s = src + (size_t)nh * 3;
        if constexpr (P::Long::two_row) {
            typename P::real m[12];
            const typename P::real c = P::Long::load_rows(lb, d, lane, m);
            cmac_two_row<P>(acc, m, c, s[0], s[1], s[2]);
        } else {
            typename P::real m[18];
            P::Long::load_dir(lb, d, lane, m);
            cmac<P>(acc, m, s[0], s[1], s[2]);
        }
    }
}

// ------------------------------------------------------------------ small lattices: one tile per workgroup
// With one wavefront per 64-site tile a lattice of few tiles leaves the chip
// empty (16^4: 512 wavefronts for 1024 SIMDs) and each wavefront walks 16
// rounds of loads, of which only one or two are in flight.  The split form
// gives a tile to the 8 wavefronts of a workgroup: wavefront q takes the
// one-link and the three-link term of direction q, all its loads in flight at
// once, and the 8 partial sums meet in LDS, where they are added in the order
// of q.  Bound by latency (launch, one round trip to memory, one barrier).
// Microseconds per Dslash, the default shape at 8^4 and the fastest shape at
// the others -> split (4 and 16 wavefronts per tile are within 5 %, or slower):
//   FP64   8^4 16.2 -> 3.6, 16^4 19.6 -> 13.0
//   FP32   8^4 12.5 -> 2.9, 16^4 11.6 -> 7.7, 20^4 17.5 -> 15.6
//   I16SC  8^4 12.7 -> 3.0, 16^4 9.6 -> 5.7, 20^4 14.7 -> 9.5, 24^4 20.1 -> 17.0
// split_tiles has both sides of the lines.
// KEEP: link loads through the caches (links_stay_cached).
constexpr int SPLIT = 8;
constexpr int SPLIT_NT = SPLIT * TILE;
constexpr int TILE_REALS = 6 * TILE;  // reals of a tile's colour vectors
static_assert(TILE_REALS <= SPLIT_NT, "one real of the result per thread");

template <class P, bool KEEP> struct SplitTerms {
    using R = typename P::real;
    using V = typename P::cvec;
    R mf[18], ml[18];
    R c;          // sign of a two-row link's third row
    int nf, nl;   // neighbours
    // the loads of the wavefront's links, and its neighbours' numbers
    __device__ __forceinline__ void load(const Geom &g, const char *__restrict__ fat, const char *__restrict__ lng,
                                         int parity, int tile, int lane, int h, int q)
    {
        int x, y, z, t;
        site_coords(g, h, parity, x, y, z, t);
        const size_t tix = (size_t)parity * g.ntiles + tile;
        const char *lb = lng + tix * P::Long::tile_bytes;
        nf = nbr_h(g, h, x, y, z, t, q & 3, q >= 4 ? -1 : 1);
        nl = nbr_h(g, h, x, y, z, t, q & 3, q >= 4 ? -3 : 3);
        P::Fat::template load_dir<KEEP>(fat + tix * P::Fat::tile_bytes, q, lane, mf);
        if constexpr (P::Long::two_row) c = P::Long::template load_rows<KEEP>(lb, q, lane, ml);
        else P::Long::template load_dir<KEEP>(lb, q, lane, ml);
    }
    // the two terms of the neighbour vectors f (one hop) and l (three hops)
    __device__ __forceinline__ void products(const V f[3], const V l[3], R acc[6]) const
    {
#pragma unroll
        for (int i = 0; i < 6; ++i) acc[i] = 0;
        cmac<P>(acc, mf, f[0], f[1], f[2]);
        if constexpr (P::Long::two_row) cmac_two_row<P>(acc, ml, c, l[0], l[1], l[2]);
        else cmac<P>(acc, ml, l[0], l[1], l[2]);
    }
    __device__ __forceinline__ static void put(const R acc[6], int q, int lane, R *red)
    {
        V *o = reinterpret_cast<V *>(red + q * TILE_REALS + 6 * lane);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            V v;
            v.x = acc[2 * i];
            v.y = acc[2 * i + 1];
            o[i] = v;
        }
    }
    // after a barrier: real i of the tile's result (site i / 6; colour and re / im i % 6)
    __device__ __forceinline__ static R result(const R *red, int i)
    {
        R s = red[i];
#pragma unroll
        for (int q = 1; q < SPLIT; ++q) s += red[q * TILE_REALS + i];
        return s;
    }
};

// Whether a lattice takes the split form in this precision where no shape was
// asked for (dslash_form), and whether its packed links stay in the last-level
// cache from one launch to the next (dslash.hip).
bool split_tiles(const Geom &g, int prec);
bool links_stay_cached(const Geom &g, int prec);

// Kernel gates read from a solver's device-resident state (NULL: always run).
struct SolverFlags {
    int done;      // nonzero: solve finished (converged or broke down)
    int reliable;  // nonzero: a reliable update is pending this iteration
};
enum { GATE_ALWAYS = 0, GATE_NOT_DONE = 1, GATE_RELIABLE = 2 };

__device__ __forceinline__ bool gate_closed(const SolverFlags *f, int gate)
{
    if (gate == GATE_ALWAYS || f == nullptr) return false;
    if (f->done) return true;
    return gate == GATE_RELIABLE && !f->reliable;
}

// Launch helpers (defined in dslash.hip).  launch_dslash uses the form and the
// shape chosen for (dims, precision), launch_dslash_shape a given shape,
// launch_dslash_tiles the split form.
struct DslashShape {
    int nt;      // threads per block
    int waves;   // minimum wavefronts per SIMD the compiler must allow
    int unroll;  // terms of the 16 unrolled together
    int order;   // tile order (apply_order): 0 plain, 1 default blocks, 2 and 3 8- and 4-plane t-blocks by all z
};
constexpr int N_DSLASH_SHAPES = 13;
extern const DslashShape DSLASH_SHAPES[N_DSLASH_SHAPES];
int tuned_dslash_shape(const Geom &g, int prec);            // tune.cpp
int tuned_choice(const char *kind, const Geom &g, int prec, int n, int fallback);
void set_tuned_choice(const char *kind, const Geom &g, int prec, int n, int v);

// What a lattice that split_tiles() covers runs in this precision: the split
// form (rule), or the shape, because a caller asked for it (set) or because
// the autotuner timed it faster (tuned).  The other lattices run the shape.
enum class DslashForm { rule = 0, set = 1, tuned = 2 };
DslashForm dslash_form(const Geom &g, int prec);
void set_dslash_choice(const Geom &g, int prec, int shape, DslashForm form);

template <class P>
hipError_t launch_dslash(const Geom &g, const void *fat, const void *lng, const void *src, void *dst, int parity,
                         hipStream_t s, const SolverFlags *flags = nullptr, int gate = GATE_ALWAYS);
template <class P>
hipError_t launch_dslash_shape(int shape, const Geom &g, const void *fat, const void *lng, const void *src, void *dst,
                               int parity, hipStream_t s, const SolverFlags *flags = nullptr, int gate = GATE_ALWAYS);
template <class P>
hipError_t launch_dslash_tiles(const Geom &g, const void *fat, const void *lng, const void *src, void *dst, int parity,
                               hipStream_t s);

}  // namespace hisq
