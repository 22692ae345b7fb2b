// Link construction on the GPU: the three-link (Naik) products of Sec. 4 of
// the paper, path-summed (smeared) one-link matrices and the folding of the
// staggered phases.
//
// Fields are canonical complex128 [mu][t][z][y][x][3][3]: matrix (mu, n) is
// 9 double2 at offset 9 (mu V + lex(n)).  One thread builds one output
// matrix; the 3x3 complex products run in FP64 registers.  All indexing is
// periodic: the boundary sign enters only through hisq_fold_links.
#include <cmath>
#include <type_traits>

#include "canon.hpp"

namespace hisq {

constexpr int LNT = 256;

// c = a b, with a and/or b taken as their adjoint
template <bool DA, bool DB>
__device__ __forceinline__ M3 mm(const M3 &a, const M3 &b)
{
    M3 c;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            double re = 0, im = 0;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const double2 x = DA ? a.e[3 * k + i] : a.e[3 * i + k];
                const double2 y = DB ? b.e[3 * j + k] : b.e[3 * k + j];
                const double xi = DA ? -x.y : x.y;
                const double yi = DB ? -y.y : y.y;
                re = fma(x.x, y.x, re);
                re = fma(-xi, yi, re);
                im = fma(x.x, yi, im);
                im = fma(xi, y.x, im);
            }
            c.e[3 * i + j] = make_double2(re, im);
        }
    }
    return c;
}

__device__ __forceinline__ void axpy_m3(double a, const M3 &x, M3 &y)
{
#pragma unroll
    for (int i = 0; i < 9; ++i) y.e[i] = make_double2(fma(a, x.e[i].x, y.e[i].x), fma(a, x.e[i].y, y.e[i].y));
}

__device__ __forceinline__ long long lex_hop2(const Lex &g, long long n, const int c[4], int mu, int k, int nu, int j)
{
    int cc[4] = { c[0], c[1], c[2], c[3] };
    const long long m = lex_hop(g, n, c, mu, k);
    int v = cc[mu] + k;
    cc[mu] = v < 0 ? v + g.L[mu] : (v >= g.L[mu] ? v - g.L[mu] : v);
    return lex_hop(g, m, cc, nu, j);
}

// store the block's NT matrices to the contiguous out[n0 .. n0 + count)
template <int NT>
__device__ __forceinline__ void scatter(Stage<NT> &st, double2 *__restrict__ out, long long n0, int count, const M3 &m)
{
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 9; ++e) st.m[9 * threadIdx.x + e] = m.e[e];
    __syncthreads();
    double2 *o = out + 9 * n0;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const int q = threadIdx.x + NT * i;
        if (q < 9 * count) ntstore(st.m[q], o + q);
    }
}

// ------------------------------------------------------------------ three-link products
template <int NT>
__global__ void __launch_bounds__(NT) k_three_link(Lex g, const double2 *__restrict__ thin, double2 *__restrict__ out)
{
    __shared__ Stage<NT> st;
    const int mu = blockIdx.y;
    // Each XCD takes a contiguous range of workgroups.  Along z and t (where a
    // slice is whole workgroups) the direction's coordinate runs fastest, so that
    // n + mu and n + 2 mu are the next workgroups' own links and come from L2
    // once (32^4, all four directions: 339 -> 256 us, the rate of a copy).
    long long blk = xcd_block(blockIdx.x, gridDim.x);
    if (blk * NT >= g.V) return;
    if (mu >= 2 && g.s[mu] % NT == 0) {
        const long long per = g.s[mu] / NT, r = blk / g.L[mu];
        blk = (r / per) * per * g.L[mu] + (blk % g.L[mu]) * per + r % per;
    }
    const long long n0 = blk * NT, n = n0 + threadIdx.x;
    const bool live = n < g.V;
    int c[4] = { 0, 0, 0, 0 };
    if (live) lex_coords(g, n, c);
    const double2 *U = thin + 9 * (size_t)mu * g.V;
    const M3 a = gather<NT>(st, U, live ? n : -1);
    const M3 b = gather<NT>(st, U, live ? lex_hop(g, n, c, mu, 1) : -1);
    const M3 ab = mm<false, false>(a, b);
    const M3 d = gather<NT>(st, U, live ? lex_hop(g, n, c, mu, 2) : -1);
    const int count = (int)(g.V - n0 < NT ? g.V - n0 : NT);
    scatter<NT>(st, out + 9 * (size_t)mu * g.V, n0, count, mm<false, false>(ab, d));
}

// ------------------------------------------------------------------ staples
// For the mu-link field Vf and direction nu, at every site n:
//   S(n) = [sign + ] U_nu(n) Vf(n+nu) U_nu(n+mu)^dag
//        + [sign - ] U_nu(n-nu)^dag Vf(n-nu) U_nu(n-nu+mu)
// then  S_out(n) = S(n)                      (if S_out)
//       F(n)     = c_init Uinit(n) + c S(n)   (if Uinit)   or   F(n) += c S(n)   (if F)
enum { ST_PLUS = 1, ST_MINUS = 2 };

template <int NT>
__global__ void __launch_bounds__(NT) k_staple(Lex g, const double2 *__restrict__ thin,
                                               const double2 *__restrict__ Vf, int mu, int nu, int signs,
                                               double2 *__restrict__ S_out, double2 *__restrict__ F, double c,
                                               const double2 *__restrict__ Uinit, double c_init)
{
    __shared__ Stage<NT> st;
    const long long n0 = (long long)blockIdx.x * NT;
    const long long n = n0 + threadIdx.x;
    const bool live = n < g.V;
    const int count = (int)(g.V - n0 < NT ? g.V - n0 : NT);
    int cd[4] = { 0, 0, 0, 0 };
    if (live) lex_coords(g, n, cd);
    const double2 *Un = thin + 9 * (size_t)nu * g.V;
    M3 S;
#pragma unroll
    for (int i = 0; i < 9; ++i) S.e[i] = make_double2(0.0, 0.0);
    if (signs & ST_PLUS) {
        const M3 a = gather<NT>(st, Un, live ? n : -1);
        const M3 v = gather<NT>(st, Vf, live ? lex_hop(g, n, cd, nu, 1) : -1);
        const M3 av = mm<false, false>(a, v);
        const M3 b = gather<NT>(st, Un, live ? lex_hop(g, n, cd, mu, 1) : -1);
        axpy_m3(1.0, mm<false, true>(av, b), S);
    }
    if (signs & ST_MINUS) {
        const long long m = live ? lex_hop(g, n, cd, nu, -1) : -1;
        const M3 a = gather<NT>(st, Un, m);
        const M3 v = gather<NT>(st, Vf, m);
        const M3 av = mm<true, false>(a, v);
        const M3 b = gather<NT>(st, Un, live ? lex_hop2(g, n, cd, nu, -1, mu, 1) : -1);
        axpy_m3(1.0, mm<false, false>(av, b), S);
    }
    if (S_out) scatter<NT>(st, S_out, n0, count, S);
    if (F) {
        M3 f;
        if (Uinit) {
            const M3 u = gather<NT>(st, Uinit, live ? n : -1);
#pragma unroll
            for (int i = 0; i < 9; ++i) f.e[i] = make_double2(c_init * u.e[i].x, c_init * u.e[i].y);
        } else {
            f = gather<NT>(st, F, live ? n : -1);
        }
        axpy_m3(c, S, f);
        scatter<NT>(st, F, n0, count, f);
    }
}

// ------------------------------------------------------------------ path sums in three passes
// With T_k V = the 3-staple of the field V in the direction k (both signs), the
// path sum of a link direction mu is linear in its nested staples:
//   V_k = c5 U_mu + c7 T_k U_mu                               (3 staples)
//   X_o = c3 U_mu + sum_{i != o} T_i V_k                      (6; k the axis other than mu, o, i)
//   F   = c1 U_mu + sum_o T_o X_o + cL sum_o (T_o^+ T_o^+ + T_o^- T_o^-) U_mu
// that is 12 staples and the Lepage paths instead of one staple per member of
// the path families (21), and three launches per mu instead of 27.
//
// Fields are in 64-site tiles [tile][element][site], so that a wavefront's
// loads are contiguous, with the sites numbered in blocks of 4 (or 2) along
// each axis: 256 consecutive sites are a 4^4 block where the extents allow it.
// The thin links are brought into that form once; F leaves it through LDS.
//
// What bounds the passes is the fabric: with one site per thread, nothing
// staged and lexicographic order, an XCD's wavefronts touch 10 MB between two
// uses of a line, so three reads in four miss its 4 MB L2 and the passes ran
// at 7 TB/s on 4-6 times the fields (32^4: V 0.37, X 0.85, F 0.65 ms per mu).
// Workgroups that hold their block's thin links (or V) in LDS read only the
// faces again: X 6.0 -> 1.7 GB and 0.57 ms, F 4.3 -> 3.6 GB and 0.55 ms, V
// unchanged.  The path sum at 32^4: 21.0 ms staple by staple, 5.8 ms.
struct PathGeo {
    Lex g;
    int lb[4], is[4], ts[4];  // block extents 2^lb; strides inside a block and between blocks
    int lt;                   // sites of a block, 2^lt
    const double2 *U;         // four fields of `stride` double2
    double2 *V, *X;           // three each
    size_t stride;
    int ntiles;
};

__device__ __forceinline__ M3 ld_tile(const double2 *__restrict__ f, int n)
{
    const double2 *p = f + (size_t)(n >> 6) * (9 * TILE) + (n & 63);
    M3 m;
#pragma unroll
    for (int e = 0; e < 9; ++e) m.e[e] = p[e * TILE];
    return m;
}
__device__ __forceinline__ void st_tile(double2 *__restrict__ f, int n, const M3 &m)
{
    double2 *p = f + (size_t)(n >> 6) * (9 * TILE) + (n & 63);
#pragma unroll
    for (int e = 0; e < 9; ++e) p[e * TILE] = m.e[e];
}

// The site: its number n in the blocked order and lex in the canonical one,
// and its moves along each axis in n: up[d], dn[d] to the next and the
// previous site, up2, dn2 two away.  Moves along different axes add.
struct PathSite {
    int n, up[4], dn[4], up2[4], dn2[4];
    long long lex;
    bool live;
};
__device__ __forceinline__ int pick(const int v[4], int i) { return i == 0 ? v[0] : i == 1 ? v[1] : i == 2 ? v[2] : v[3]; }
__device__ __forceinline__ PathSite path_site(const PathGeo &p, long long n)
{
    PathSite s;
    s.live = n < p.g.V;
    s.n = s.live ? (int)n : (int)p.g.V - 1;
    s.lex = 0;
    int in = s.n & ((1 << p.lt) - 1), b = s.n >> p.lt;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const int L = p.g.L[d], lb = p.lb[d], nb_d = L >> lb, bc = b % nb_d;
        const int c = (bc << lb) + (in & ((1 << lb) - 1));
        b /= nb_d;
        in >>= lb;
        s.lex += c * p.g.s[d];
        auto at = [&](int v) {
            v += v < 0 ? L : 0;
            v -= v >= L ? L : 0;
            return (v >> lb) * p.ts[d] + (v & ((1 << lb) - 1)) * p.is[d];
        };
        const int here = at(c);
        s.up[d] = at(c + 1) - here;
        s.dn[d] = at(c - 1) - here;
        s.up2[d] = at(c + 2) - here;
        s.dn2[d] = at(c - 2) - here;
    }
    return s;
}

// the directions other than MU, in order
template <int MU> __device__ constexpr int other(int j) { return j < MU ? j : j + 1; }

// S += av b^dag (up) or av b (down).  Each entry of the product is summed by
// itself and added once: terms added to the running sum one by one round at
// the sum's size each.  Root-mean-square error of the path sums against
// extended precision, over that of the staple-by-staple schedule: 1.03-1.23
// that way, 0.73-1.00 this way.  A row at a time, as the scheduling barriers
// ask: more sums in flight spill 10-20 registers (32^4: 5.95 ms against 5.81;
// term by term 5.88).
template <bool DOWN> __device__ __forceinline__ void add_right(M3 &S, const M3 &av, const M3 &b)
{
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            double re = 0.0, im = 0.0;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const double2 x = av.e[3 * i + k], y = DOWN ? b.e[3 * k + j] : b.e[3 * j + k];
                const double yi = DOWN ? y.y : -y.y;
                re = fma(x.x, y.x, re);
                re = fma(-x.y, yi, re);
                im = fma(x.x, yi, im);
                im = fma(x.y, y.x, im);
            }
            S.e[3 * i + j] = make_double2(S.e[3 * i + j].x + re, S.e[3 * i + j].y + im);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// An index offset of 0 that the compiler takes to depend on m: what is loaded
// through it is not loaded before m is there.
__device__ __forceinline__ void after(int &zero, const M3 &m)
{
    asm volatile("" : "+v"(zero) : "v"(m.e[0].x), "v"(m.e[4].y), "v"(m.e[8].x), "v"(m.e[8].y));
}
// S += a v b^dag (up) or a^dag v b (down), the two halves of a staple, on
// operands loaded when their turn comes (each takes `zero`): b when a and v
// are consumed, and nothing of the next staple before that.  Three matrices
// and the sum are what a thread's registers hold at 3 wavefronts per SIMD.
struct NoInit {};
// init: where S comes from, if it is not there yet
template <bool DOWN, class FA, class FV, class FB, class FS = NoInit>
__device__ __forceinline__ void load_staple(M3 &S, int &zero, FA a, FV v, FB b, FS init = FS())
{
    M3 av;
    {
        const M3 x = a(), y = v();
        av = mm<DOWN, false>(x, y);
    }
    after(zero, av);
    if constexpr (!std::is_same<FS, NoInit>::value) S = init();
    add_right<DOWN>(S, av, b());
    after(zero, S);
}

__device__ __forceinline__ M3 scaled(double c, const M3 &m)
{
    M3 r;
#pragma unroll
    for (int i = 0; i < 9; ++i) r.e[i] = make_double2(c * m.e[i].x, c * m.e[i].y);
    return r;
}

// canonical thin links to the blocked tiles, one direction per blockIdx.y
__global__ void __launch_bounds__(LNT) k_path_tiles(PathGeo p, const double2 *__restrict__ thin, double2 *__restrict__ U)
{
    __shared__ Stage<LNT> st;
    const PathSite s = path_site(p, (long long)blockIdx.x * LNT + threadIdx.x);
    const M3 m = gather<LNT>(st, thin + 9 * (size_t)blockIdx.y * p.g.V, s.live ? s.lex : -1);
    if (s.live) st_tile(U + blockIdx.y * p.stride, s.n, m);
}

// ---- the three passes: 256 consecutive sites per workgroup, three threads per
// site, one for each axis other than mu (group j, four wavefronts).  The
// sites' own matrices of the thin fields (and of V) are in LDS, so that what
// a hop finds inside the workgroup's block is read there; only the block's
// faces come from memory again.
constexpr int PNT = 3 * LNT;
constexpr int PTILE = 9 * LNT;  // double2 of one field's block: four tiles

struct PathLds {
    double2 t[4][PTILE];
};
static_assert(sizeof(PathLds) <= 160 * 1024, "LDS of a CU");

// Site n of field f, whose block of sites n0 .. n0 + 255 has its image in t:
// a lane's address is in one or the other, one load instruction serves both
// (branches per matrix instead of flat addresses spill 60-360 registers).
__device__ __forceinline__ M3 ld_block(const double2 *t, const double2 *f, int n, int n0)
{
    const int q = n - n0;
    const double2 *in = t + (q >> 6) * (9 * TILE) + (q & 63), *out = f + (size_t)(n >> 6) * (9 * TILE) + (n & 63);
    const double2 *p = (unsigned)q < (unsigned)LNT ? in : out;
    M3 m;
#pragma unroll
    for (int e = 0; e < 9; ++e) m.e[e] = p[e * TILE];
    return m;
}
// the block's image (zero past the lattice's last tile)
__device__ __forceinline__ void copy_block(double2 *t, const double2 *__restrict__ f, int n0, int ntiles)
{
    const double2 *b = f + (size_t)(n0 >> 6) * (9 * TILE);
    const int have = min(PTILE, (ntiles - (n0 >> 6)) * 9 * TILE);
    for (int q = threadIdx.x; q < PTILE; q += PNT) t[q] = q < have ? b[q] : make_double2(0.0, 0.0);
}

// V_k = c5 U_mu + c7 A_k for the three axes k.  SEVEN: c7 is not zero.
template <int MU, bool SEVEN> __global__ void __launch_bounds__(PNT) k_path_v(PathGeo p, double c5, double c7)
{
    __shared__ PathLds l;
    const int blk = xcd_block(blockIdx.x, gridDim.x), j = __builtin_amdgcn_readfirstlane(threadIdx.x / LNT);
    const int i = threadIdx.x % LNT, n0 = blk * LNT, k = other<MU>(j);
    if ((long long)n0 >= p.g.V) return;
    const PathSite s = path_site(p, n0 + i);
    const double2 *Um = p.U + MU * p.stride, *Uk = p.U + k * p.stride;
    M3 S;
    int zero = 0;
    if constexpr (SEVEN) {
#pragma unroll
        for (int f = 0; f < 3; ++f) copy_block(l.t[f], p.U + other<MU>(f) * p.stride, n0, p.ntiles);
        copy_block(l.t[3], Um, n0, p.ntiles);
        __syncthreads();
        const int up = pick(s.up, k), m = s.n + pick(s.dn, k);
        auto uk = [&](int n) { return [&, n] { return ld_block(l.t[j], Uk, n + zero, n0); }; };
        auto um = [&](int n) { return [&, n] { return ld_block(l.t[3], Um, n + zero, n0); }; };
        load_staple<false>(S, zero, uk(s.n), um(s.n + up), uk(s.n + s.up[MU]), [] { return scaled(0.0, M3{}); });
        load_staple<true>(S, zero, uk(m), um(m), uk(m + s.up[MU]));
        const M3 u = ld_tile(l.t[3], i + zero);
#pragma unroll
        for (int e = 0; e < 9; ++e)
            S.e[e] = make_double2(fma(c7, S.e[e].x, c5 * u.e[e].x), fma(c7, S.e[e].y, c5 * u.e[e].y));
    } else {
        S = scaled(c5, ld_tile(Um, s.n));
    }
    if (s.live) st_tile(p.V + j * p.stride, s.n, S);
}

// X_o for the three axes o: V_k of the block in t[k], U_i of one axis after the other in t[3].
template <int MU> __global__ void __launch_bounds__(PNT) k_path_x(PathGeo p, double c3)
{
    __shared__ PathLds l;
    const int blk = xcd_block(blockIdx.x, gridDim.x), o = __builtin_amdgcn_readfirstlane(threadIdx.x / LNT);
    const int i = threadIdx.x % LNT, n0 = blk * LNT;
    if ((long long)n0 >= p.g.V) return;
    const PathSite s = path_site(p, n0 + i);
#pragma unroll
    for (int f = 0; f < 3; ++f) copy_block(l.t[f], p.V + f * p.stride, n0, p.ntiles);
    M3 X = scaled(c3, ld_tile(p.U + MU * p.stride, s.n));
    int zero = 0;
#pragma unroll 1
    for (int ji = 0; ji < 3; ++ji) {
        const int d = other<MU>(ji), k = 3 - ji - o;
        const double2 *Ui = p.U + d * p.stride;
        if (ji) __syncthreads();  // the previous axis is done with t[3]
        copy_block(l.t[3], Ui, n0, p.ntiles);
        __syncthreads();
        if (ji == o) continue;
        const double2 *Vk = p.V + k * p.stride;
        const int up = pick(s.up, d), m = s.n + pick(s.dn, d);
        auto ui = [&](int n) { return [&, n] { return ld_block(l.t[3], Ui, n + zero, n0); }; };
        auto vk = [&](int n) { return [&, n] { return ld_block(l.t[k], Vk, n + zero, n0); }; };
        load_staple<false>(X, zero, ui(s.n), vk(s.n + up), ui(s.n + s.up[MU]));
        load_staple<true>(X, zero, ui(m), vk(m), ui(m + s.up[MU]));
    }
    if (s.live) st_tile(p.X + o * p.stride, s.n, X);
}

// F.  HASX: X holds the inner sums; else they are c3 U_mu alone (c3 may be 0).  LEP: the Lepage paths.
template <int MU, bool HASX, bool LEP>
__global__ void __launch_bounds__(PNT) k_path_f(PathGeo p, double2 *__restrict__ F, double c1, double c3, double cl)
{
    __shared__ PathLds l;
    __shared__ long long lex[LNT];
    const int blk = xcd_block(blockIdx.x, gridDim.x), j = __builtin_amdgcn_readfirstlane(threadIdx.x / LNT);
    const int i = threadIdx.x % LNT, n0 = blk * LNT, o = other<MU>(j);
    if ((long long)n0 >= p.g.V) return;
    const PathSite s = path_site(p, n0 + i);
    const double2 *Um = p.U + MU * p.stride, *Uo = p.U + o * p.stride, *Xo = p.X + j * p.stride;
#pragma unroll
    for (int b = 0; b < 3; ++b) copy_block(l.t[b], p.U + other<MU>(b) * p.stride, n0, p.ntiles);
    copy_block(l.t[3], Um, n0, p.ntiles);
    if (j == 0) lex[i] = s.live ? s.lex : -1;
    __syncthreads();
    M3 f = scaled(j == 0 ? c1 : 0.0, ld_tile(l.t[3], i));
    int zero = 0;
    const int up = pick(s.up, o), dn = pick(s.dn, o);
    auto half = [&](auto dir) {
        constexpr bool DN = decltype(dir)::value;
        const int at = DN ? s.n + dn : s.n, v = DN ? at : s.n + up;
        auto uo = [&](int n) { return [&, n] { return ld_block(l.t[j], Uo, n + zero, n0); }; };
        auto um = [&](int n) { return [&, n] { return ld_block(l.t[3], Um, n + zero, n0); }; };
        auto inner = [&] { return HASX ? ld_tile(Xo, v + zero) : scaled(c3, um(v)()); };
        M3 w;
        if constexpr (LEP) {
            // the half staple of U_mu at v on the same side
            const int q = DN ? s.n + pick(s.dn2, o) : v, u = DN ? q : s.n + pick(s.up2, o);
            load_staple<DN>(w, zero, [&] { return scaled(cl, uo(q)()); }, um(u), uo(q + s.up[MU]), inner);
        } else {
            w = inner();
        }
        load_staple<DN>(f, zero, uo(at), [&] { return w; }, uo(at + s.up[MU]));
    };
    half(std::false_type{});
    half(std::true_type{});
    // the three groups' sums in order, then out in the canonical form: [site][element] in t[0]
    __syncthreads();
    st_tile(l.t[1 + j], i, f);
    __syncthreads();
    for (int q = threadIdx.x; q < PTILE; q += PNT) {
        const double2 a = l.t[1][q], b = l.t[2][q], c = l.t[3][q];
        const int tile = q / (9 * TILE), r = q % (9 * TILE);
        l.t[0][9 * (tile * TILE + r % TILE) + r / TILE] = make_double2((a.x + b.x) + c.x, (a.y + b.y) + c.y);
    }
    __syncthreads();
    for (int q = threadIdx.x; q < PTILE; q += PNT) {
        const long long n = lex[q / 9];
        if (n >= 0) ntstore(l.t[0][q], F + 9 * n + q % 9);
    }
}

static PathGeo path_geo(const Lex &l)
{
    PathGeo p;
    p.g = l;
    p.lt = 0;
    for (int d = 0; d < 4; ++d) {
        p.lb[d] = l.L[d] % 4 == 0 ? 2 : 1;
        p.is[d] = 1 << p.lt;
        p.lt += p.lb[d];
    }
    int t = 1 << p.lt;
    for (int d = 0; d < 4; ++d) {
        p.ts[d] = t;
        t *= l.L[d] >> p.lb[d];
    }
    return p;
}

template <int MU>
static void launch_paths(const PathGeo &p, double2 *F, const double c[5], hipStream_t s)
{
    const double c1 = c[0], c3 = c[1], c5 = c[2], c7 = c[3], cl = c[4];
    const dim3 grid(xcd_grid((int)((p.g.V + LNT - 1) / LNT))), blk(PNT);
    const bool x = c5 != 0 || c7 != 0;
    if (x) {
        auto kv = c7 != 0 ? k_path_v<MU, true> : k_path_v<MU, false>;
        hipLaunchKernelGGL(kv, grid, blk, 0, s, p, c5, c7);
        hipLaunchKernelGGL(k_path_x<MU>, grid, blk, 0, s, p, c3);
    }
    auto kf = x ? (cl != 0 ? k_path_f<MU, true, true> : k_path_f<MU, true, false>)
                : (cl != 0 ? k_path_f<MU, false, true> : k_path_f<MU, false, false>);
    hipLaunchKernelGGL(kf, grid, blk, 0, s, p, F, c1, c3, cl);
}

// out = c U (the one-link term alone, when no staple is summed)
template <int NT>
__global__ void __launch_bounds__(NT) k_scale_links(long long n9, const double2 *__restrict__ in,
                                                    double2 *__restrict__ out, double c)
{
    const long long i = (long long)blockIdx.x * NT + threadIdx.x;
    if (i >= n9) return;
    const double2 v = in[i];
    out[i] = make_double2(c * v.x, c * v.y);
}

// ------------------------------------------------------------------ phases
// links_mu(n) *= eta_mu(n) b_mu(n): eta_x = 1, eta_y = (-1)^x, eta_z = (-1)^(x+y),
// eta_t = (-1)^(x+y+z); b = -1 on t-links with t + hop >= Lt when antiperiodic.
template <int NT>
__global__ void __launch_bounds__(NT) k_fold(Lex g, double2 *__restrict__ links, int hop, int anti)
{
    const long long n = (long long)blockIdx.x * NT + threadIdx.x;
    const int mu = blockIdx.y;
    if (n >= g.V) return;
    int c[4];
    lex_coords(g, n, c);
    int e = 0;
    for (int k = 0; k < mu; ++k) e += c[k];
    bool neg = (e & 1) != 0;
    if (mu == 3 && anti && c[3] + hop >= g.L[3]) neg = !neg;
    if (!neg) return;
    double2 *p = links + 9 * ((size_t)mu * g.V + n);
#pragma unroll
    for (int i = 0; i < 9; ++i) p[i] = make_double2(-p[i].x, -p[i].y);
}

static bool overlaps(const void *a, size_t na, const void *b, size_t nb)
{
    const char *x = (const char *)a, *y = (const char *)b;
    return x < y + nb && y < x + na;
}

static size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

static int check_launch(const char *what)
{
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? HISQ_OK : hip_fail(e, what);
}

// One tiled field, and the workspace of the three-pass schedule: the four
// thin fields, A and X (three each).  A caller with room for three fields only
// gets the staple-by-staple schedule.
static size_t tiled_field_bytes(const Lex &l) { return (size_t)((l.V + TILE - 1) / TILE) * TILE * 144; }
static size_t fat_paths_min_bytes(const Lex &l) { return 3 * align_up((size_t)l.V * 144, 256); }
static size_t fat_paths_pass_bytes(const Lex &l) { return 10 * tiled_field_bytes(l); }

// What the workspace query asks for: beyond 64 GiB (48 million sites) three
// fields, not ten.  thin and out take eight more, so that with ten a 96^3 x 192
// lattice needs 440 GB; with three it fits the card (269 of 288 GB).
size_t fat_paths_ws_bytes(const int dims[4])
{
    Lex l;
    if (make_lex(dims, l)) return 0;
    const size_t full = fat_paths_pass_bytes(l);
    return full <= (size_t)64 << 30 ? full : fat_paths_min_bytes(l);
}

}  // namespace hisq

using namespace hisq;

extern "C" int hisq_three_link(const void *thin, void *out, const int dims[4], void *stream)
{
    Lex l;
    int rc = make_lex(dims, l);
    if (rc) return rc;
    if (!thin || !out) return fail(HISQ_EINVAL, "hisq_three_link: NULL pointer");
    if (!aligned16({thin, out}))
        return fail(HISQ_EINVAL, "hisq_three_link: device pointers must be 16-byte aligned");
    const size_t bytes = (size_t)l.V * 4 * 144;
    if (overlaps(thin, bytes, out, bytes)) return fail(HISQ_EALIAS, "hisq_three_link: out overlaps thin");
    dim3 grid((unsigned)xcd_grid((int)((l.V + LNT - 1) / LNT)), 4);
    hipLaunchKernelGGL(k_three_link<LNT>, grid, dim3(LNT), 0, (hipStream_t)stream, l, (const double2 *)thin,
                       (double2 *)out);
    return check_launch("hisq_three_link");
}

extern "C" int hisq_fat_paths(const void *thin, const double coeff[5], void *out, const int dims[4], void *workspace,
                              size_t ws_bytes, void *stream)
{
    Lex l;
    int rc = make_lex(dims, l);
    if (rc) return rc;
    if (!thin || !out || !coeff) return fail(HISQ_EINVAL, "hisq_fat_paths: NULL pointer");
    if (!aligned16({thin, out, workspace}))
        return fail(HISQ_EINVAL, "hisq_fat_paths: device pointers must be 16-byte aligned");
    for (int i = 0; i < 5; ++i)
        if (!std::isfinite(coeff[i])) return fail(HISQ_EINVAL, "hisq_fat_paths: coefficient not finite");
    const size_t bytes = (size_t)l.V * 4 * 144;
    if (overlaps(thin, bytes, out, bytes)) return fail(HISQ_EALIAS, "hisq_fat_paths: out overlaps thin");
    const bool passes = ws_bytes >= fat_paths_pass_bytes(l) && l.V < (1LL << 31);  // sites are ints there
    const size_t need = passes ? fat_paths_pass_bytes(l) : fat_paths_min_bytes(l);
    if (!workspace || ws_bytes < need)
        return fail(HISQ_EWORKSPACE, "hisq_fat_paths: workspace NULL or smaller than hisq_workspace_bytes()");
    if (overlaps(workspace, need, thin, bytes) || overlaps(workspace, need, out, bytes))
        return fail(HISQ_EALIAS, "hisq_fat_paths: workspace overlaps a link field");
    hipStream_t s = (hipStream_t)stream;
    const size_t fb = align_up((size_t)l.V * 144, 256);
    double2 *T3 = (double2 *)workspace;
    double2 *T5 = (double2 *)((char *)workspace + fb);
    double2 *TL = (double2 *)((char *)workspace + 2 * fb);
    const double c1 = coeff[0], c3 = coeff[1], c5 = coeff[2], c7 = coeff[3], cl = coeff[4];
    const dim3 grid((unsigned)((l.V + LNT - 1) / LNT)), blk(LNT);
    const double2 *U = (const double2 *)thin;
    const bool need3 = c3 != 0 || c5 != 0 || c7 != 0;
    if (passes && (need3 || cl != 0)) {
        PathGeo p = path_geo(l);
        p.stride = tiled_field_bytes(l) / 16;
        p.ntiles = (int)(p.stride / (9 * TILE));
        p.U = (const double2 *)workspace;
        p.V = (double2 *)workspace + 4 * p.stride;
        p.X = (double2 *)workspace + 7 * p.stride;
        hipLaunchKernelGGL(k_path_tiles, dim3(grid.x, 4), blk, 0, s, p, U, (double2 *)workspace);
        double2 *F = (double2 *)out;
        launch_paths<0>(p, F, coeff, s);
        launch_paths<1>(p, F + 9 * (size_t)l.V, coeff, s);
        launch_paths<2>(p, F + 18 * (size_t)l.V, coeff, s);
        launch_paths<3>(p, F + 27 * (size_t)l.V, coeff, s);
        return check_launch("hisq_fat_paths");
    }
    for (int mu = 0; mu < 4; ++mu) {
        const double2 *Umu = U + 9 * (size_t)mu * l.V;
        double2 *F = (double2 *)out + 9 * (size_t)mu * l.V;
        bool init = true;  // the first launch that touches F writes c1 U_mu + c S
        if (!need3 && cl == 0) {
            hipLaunchKernelGGL(k_scale_links<LNT>, dim3((unsigned)((9 * l.V + LNT - 1) / LNT)), blk, 0, s, 9 * l.V,
                               Umu, F, c1);
            continue;
        }
        for (int nu = 0; nu < 4; ++nu) {
            if (nu == mu) continue;
            if (need3) {
                hipLaunchKernelGGL(k_staple<LNT>, grid, blk, 0, s, l, U, Umu, mu, nu, ST_PLUS | ST_MINUS,
                                   (c5 != 0 || c7 != 0) ? T3 : (double2 *)nullptr, F, c3, init ? Umu : nullptr, c1);
                init = false;
            }
            if (cl != 0) {
                for (int sg = ST_PLUS; sg <= ST_MINUS; sg <<= 1) {
                    hipLaunchKernelGGL(k_staple<LNT>, grid, blk, 0, s, l, U, Umu, mu, nu, sg, TL,
                                       (double2 *)nullptr, 0.0, (const double2 *)nullptr, 0.0);
                    hipLaunchKernelGGL(k_staple<LNT>, grid, blk, 0, s, l, U, (const double2 *)TL, mu, nu, sg,
                                       (double2 *)nullptr, F, cl, init ? Umu : nullptr, c1);
                    init = false;
                }
            }
            if (c5 == 0 && c7 == 0) continue;
            for (int rho = 0; rho < 4; ++rho) {
                if (rho == mu || rho == nu) continue;
                hipLaunchKernelGGL(k_staple<LNT>, grid, blk, 0, s, l, U, (const double2 *)T3, mu, rho,
                                   ST_PLUS | ST_MINUS, c7 != 0 ? T5 : (double2 *)nullptr, F, c5, nullptr, 0.0);
                if (c7 == 0) continue;
                const int sig = 6 - mu - nu - rho;
                hipLaunchKernelGGL(k_staple<LNT>, grid, blk, 0, s, l, U, (const double2 *)T5, mu, sig,
                                   ST_PLUS | ST_MINUS, (double2 *)nullptr, F, c7, nullptr, 0.0);
            }
        }
    }
    return check_launch("hisq_fat_paths");
}

extern "C" int hisq_fold_links(void *links, const int dims[4], int hop, int antiperiodic_t, void *stream)
{
    Lex l;
    int rc = make_lex(dims, l);
    if (rc) return rc;
    if (!links) return fail(HISQ_EINVAL, "hisq_fold_links: NULL pointer");
    if (!aligned16({links}))
        return fail(HISQ_EINVAL, "hisq_fold_links: device pointers must be 16-byte aligned");
    if (hop != 1 && hop != 3) return fail(HISQ_EINVAL, "hisq_fold_links: hop must be 1 or 3");
    dim3 grid((unsigned)((l.V + LNT - 1) / LNT), 4);
    hipLaunchKernelGGL(k_fold<LNT>, grid, dim3(LNT), 0, (hipStream_t)stream, l, (double2 *)links, hop,
                       antiperiodic_t ? 1 : 0);
    return check_launch("hisq_fold_links");
}
