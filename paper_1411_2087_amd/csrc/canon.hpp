// Canonical link fields, complex128 [mu][t][z][y][x][3][3]: geometry and the
// staging of their matrices, shared by link construction and packing.
#pragma once

#include "hisq_common.hpp"

namespace hisq {

struct M3 {
    double2 e[9];
};

struct Lex {
    int L[4];
    long long s[4];  // lex strides 1, Lx, Lx Ly, Lx Ly Lz
    long long V;
};

__device__ __forceinline__ void lex_coords(const Lex &g, long long n, int c[4])
{
    c[0] = (int)(n % g.L[0]);
    n /= g.L[0];
    c[1] = (int)(n % g.L[1]);
    n /= g.L[1];
    c[2] = (int)(n % g.L[2]);
    c[3] = (int)(n / g.L[2]);
}

// lex index of the site n whose coordinates are c, moved by k along mu (|k| < L_mu)
__device__ __forceinline__ long long lex_hop(const Lex &g, long long n, const int c[4], int mu, int k)
{
    int v = c[mu] + k;
    v += (v < 0) ? g.L[mu] : 0;
    v -= (v >= g.L[mu]) ? g.L[mu] : 0;
    return n + (long long)(v - c[mu]) * g.s[mu];
}

inline int make_lex(const int dims[4], Lex &l)
{
    Geom g;
    int rc = make_geom(dims, g);
    if (rc) return rc;
    for (int i = 0; i < 4; ++i) l.L[i] = dims[i];
    l.s[0] = 1;
    for (int i = 1; i < 4; ++i) l.s[i] = l.s[i - 1] * dims[i - 1];
    l.V = l.s[3] * dims[3];
    return HISQ_OK;
}

// ------------------------------------------------------------------ LDS staging
// A canonical matrix is 144 contiguous bytes, so a lane that loads its own
// matrix touches a new cache line with every 16-byte load.  The block instead
// reads the NT matrices its threads need cooperatively, consecutive lanes on
// consecutive 16-byte words (contiguous wherever the sites' matrices are),
// through LDS laid out [thread][element]; each thread then takes its 9
// words.  Reads of 16 bytes at a 144-byte lane stride touch 16 different
// bank groups per quarter-wave, so the LDS side runs conflict-free.
template <int NT>
struct Stage {
    double2 m[NT * 9];
    long long idx[NT];
};

// Matrix idx of `base` for every thread (idx < 0: none) into st.m[9 thread ..];
// every thread of the block calls this, and st.m may be read afterwards.
template <int NT>
__device__ __forceinline__ void stage_in(Stage<NT> &st, const double2 *__restrict__ base, long long idx)
{
    __syncthreads();  // the previous use of st is finished
    st.idx[threadIdx.x] = idx;
    __syncthreads();
    double2 v[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const int q = threadIdx.x + NT * i;
        const int j = q / 9;
        const long long s = st.idx[j];
        v[i] = base[s >= 0 ? 9 * s + (q - 9 * j) : 0];
    }
#pragma unroll
    for (int i = 0; i < 9; ++i) st.m[threadIdx.x + NT * i] = v[i];
    __syncthreads();
}
template <int NT>
__device__ __forceinline__ M3 gather(Stage<NT> &st, const double2 *__restrict__ base, long long idx)
{
    stage_in<NT>(st, base, idx);
    M3 m;
#pragma unroll
    for (int e = 0; e < 9; ++e) m.e[e] = st.m[9 * threadIdx.x + e];
    return m;
}

}  // namespace hisq
