// Link packing: canonical [mu][lex][3][3] complex128 -> the tiled packed
// form read by the Dslash kernels.
//
// For every output site n of each parity the packed field holds the 8
// matrices that multiply n's neighbours: U_mu(n) for +mu and
// -U_mu(n - k mu)^dag for -mu (k = 1 fat, 3 long).  Storing the backward
// links at the output site doubles the storage but makes every link read of
// the Dslash contiguous and single-use, the locality argument of Sec. 4
// ("both forward and backward links are stored at each site").
#include <type_traits>

#include "canon.hpp"

namespace hisq {

template <int PREC>
__device__ __forceinline__ void store_block(char *blk, int lane, const double m[18]);

template <>
__device__ __forceinline__ void store_block<HISQ_F64>(char *blk, int lane, const double m[18])
{
    double2 *p = reinterpret_cast<double2 *>(blk) + lane;
#pragma unroll
    for (int e = 0; e < 9; ++e) ntstore(make_double2(m[2 * e], m[2 * e + 1]), p + e * TILE);
}

template <>
__device__ __forceinline__ void store_block<HISQ_F32>(char *blk, int lane, const double m[18])
{
    float4 *p4 = reinterpret_cast<float4 *>(blk) + lane;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        p4[q * TILE] = make_float4((float)m[4 * q], (float)m[4 * q + 1], (float)m[4 * q + 2], (float)m[4 * q + 3]);
    float2 *p2 = reinterpret_cast<float2 *>(blk + 4 * TILE * 16) + lane;
    *p2 = make_float2((float)m[16], (float)m[17]);
}

template <>
__device__ __forceinline__ void store_block<HISQ_F16S>(char *blk, int lane, const double m[18])
{
    double mx = 0.0;
#pragma unroll
    for (int i = 0; i < 18; ++i) mx = fmax(mx, fabs(m[i]));
    const float scale = (float)mx;
    const double inv = scale > 0.0f ? 1.0 / (double)scale : 0.0;
    unsigned w[9];
#pragma unroll
    for (int e = 0; e < 9; ++e) {
        __half2 hv = __floats2half2_rn((float)(m[2 * e] * inv), (float)(m[2 * e + 1] * inv));
        w[e] = *reinterpret_cast<unsigned *>(&hv);
    }
    uint4 *p4 = reinterpret_cast<uint4 *>(blk) + lane;
    p4[0] = make_uint4(w[0], w[1], w[2], w[3]);
    p4[TILE] = make_uint4(w[4], w[5], w[6], w[7]);
    uint2 *p2 = reinterpret_cast<uint2 *>(blk + 2 * TILE * 16) + lane;
    *p2 = make_uint2(w[8], __float_as_uint(scale));
}

template <>
__device__ __forceinline__ void store_block<HISQ_I16S>(char *blk, int lane, const double m[18])
{
    double mx = 0.0;
#pragma unroll
    for (int i = 0; i < 18; ++i) mx = fmax(mx, fabs(m[i]));
    const float scale = (float)mx;
    const double inv = scale > 0.0f ? 32767.0 / (double)scale : 0.0;
    unsigned w[9];
#pragma unroll
    for (int e = 0; e < 9; ++e) {
        int qr = (int)rint(m[2 * e] * inv), qi = (int)rint(m[2 * e + 1] * inv);
        qr = qr > 32767 ? 32767 : (qr < -32767 ? -32767 : qr);
        qi = qi > 32767 ? 32767 : (qi < -32767 ? -32767 : qi);
        w[e] = ((unsigned)qr & 0xFFFFu) | (((unsigned)qi & 0xFFFFu) << 16);
    }
    uint4 *p4 = reinterpret_cast<uint4 *>(blk) + lane;
    p4[0] = make_uint4(w[0], w[1], w[2], w[3]);
    p4[TILE] = make_uint4(w[4], w[5], w[6], w[7]);
    uint2 *p2 = reinterpret_cast<uint2 *>(blk + 2 * TILE * 16) + lane;
    *p2 = make_uint2(w[8], __float_as_uint(scale));
}

template <int PREC, class R>
__device__ __forceinline__ void store_rows(char *tile_base, int d, int lane, const double m[18], bool valid, int *status)
{
    constexpr size_t BB = R::block_bytes;
    bool neg = false;
    if (valid) {
        // det by cofactors of row 0; c = sign(Re det)
        const double c0r = m[8] * m[16] - m[9] * m[17] - (m[10] * m[14] - m[11] * m[15]);
        const double c0i = m[8] * m[17] + m[9] * m[16] - (m[10] * m[15] + m[11] * m[14]);
        const double c1r = m[10] * m[12] - m[11] * m[13] - (m[6] * m[16] - m[7] * m[17]);
        const double c1i = m[10] * m[13] + m[11] * m[12] - (m[6] * m[17] + m[7] * m[16]);
        const double c2r = m[6] * m[14] - m[7] * m[15] - (m[8] * m[12] - m[9] * m[13]);
        const double c2i = m[6] * m[15] + m[7] * m[14] - (m[8] * m[13] + m[9] * m[12]);
        const double dr = m[0] * c0r - m[1] * c0i + m[2] * c1r - m[3] * c1i + m[4] * c2r - m[5] * c2i;
        const double di = m[0] * c0i + m[1] * c0r + m[2] * c1i + m[3] * c1r + m[4] * c2i + m[5] * c2r;
        neg = dr < 0.0;
        const double cs = neg ? -1.0 : 1.0;
        // unitarity of the stored rows and agreement of row 2 with its rebuild
        double dev = fabs(dr - cs) + fabs(di);
        double rb[18];
#pragma unroll
        for (int e = 0; e < 18; ++e) rb[e] = m[e];
        third_row<double>(rb, cs);
#pragma unroll
        for (int e = 12; e < 18; ++e) dev = fmax(dev, fabs(rb[e] - m[e]));
        if (!(dev <= 1e-6)) atomicOr(status, 1);
    }
    const unsigned long long word = __ballot(neg);
    if (lane == 0) *reinterpret_cast<unsigned long long *>(tile_base + 8 * BB + 8 * (size_t)d) = word;
    if constexpr (PREC == HISQ_F64C) {
        double2 *q = reinterpret_cast<double2 *>(tile_base + (size_t)d * BB) + lane;
#pragma unroll
        for (int e = 0; e < 6; ++e) ntstore(make_double2(m[2 * e], m[2 * e + 1]), q + e * TILE);
    } else if constexpr (PREC == HISQ_I16SC) {
        // rows 0 and 1 in 16-bit fixed point against their largest |re|, |im|
        double mx = 0.0;
#pragma unroll
        for (int i = 0; i < 12; ++i) mx = fmax(mx, fabs(m[i]));
        const float scale = (float)mx;
        const double inv = scale > 0.0f ? 32767.0 / (double)scale : 0.0;
        unsigned w[6];
#pragma unroll
        for (int e = 0; e < 6; ++e) {
            int qr = (int)rint(m[2 * e] * inv), qi = (int)rint(m[2 * e + 1] * inv);
            qr = qr > 32767 ? 32767 : (qr < -32767 ? -32767 : qr);
            qi = qi > 32767 ? 32767 : (qi < -32767 ? -32767 : qi);
            w[e] = ((unsigned)qr & 0xFFFFu) | (((unsigned)qi & 0xFFFFu) << 16);
        }
        char *blk = tile_base + (size_t)d * BB;
        reinterpret_cast<uint4 *>(blk)[lane] = make_uint4(w[0], w[1], w[2], w[3]);
        reinterpret_cast<uint2 *>(blk + TILE * 16)[lane] = make_uint2(w[4], w[5]);
        reinterpret_cast<float *>(blk + TILE * 24)[lane] = scale;
    } else {
        float4 *q = reinterpret_cast<float4 *>(tile_base + (size_t)d * BB) + lane;
#pragma unroll
        for (int k = 0; k < 3; ++k)
            q[k * TILE] = make_float4((float)m[4 * k], (float)m[4 * k + 1], (float)m[4 * k + 2], (float)m[4 * k + 3]);
    }
}

// Two consecutive tiles of both parities per workgroup (256 consecutive
// canonical sites), direction by direction: the workgroup brings the 256
// source matrices through LDS, so that its loads are contiguous, and each
// wavefront takes the 64 of its (tile, parity).  A lane that reads its own
// matrix touches 64 cache lines with every 16-byte load, half of each for the
// other parity (32^4, us per field: F64 544 -> 436, F64C long 516 -> 311, I16S
// 342 -> 238, I16SC long 860 -> 229).  Bound by the fabric at 5.5-6.7 TB/s: the
// canonical field comes twice (forward and, `hop` away, backward), the packed
// one goes out once, in FP64 with streaming stores (through the caches: 478
// and 372 us).
//
// ROWS = void: full matrices of precision PREC.  Else the two-row form: rows 0
// and 1 of every matrix, plus the sign word of each (tile, direction) built
// with a wavefront ballot; `status` is set when a matrix is not +-SU(3) to
// 1e-6 (padding lanes are exempt).
//
// STAGED = false, on few sites: each lane reads its own matrix after all.  There
// the barriers and the way through LDS cost more than the lines (both
// fields, FP32, us, through LDS and read directly: 4^4 7.7, 6.1; 8^4 8.3, 6.7;
// 10x8x10x8 9.1, 7.9; 8x12x12x12 11.2, 11.1; 12^4 14.9, 16.9; 14^4 21.3, 24.7).
constexpr int PACK_NT = 256;
constexpr long long PACK_DIRECT_SITES = 16384;
template <int PREC, class ROWS, bool STAGED>
__global__ __launch_bounds__(PACK_NT) void k_pack(Lex l, Geom g, const double2 *__restrict__ canon,
                                                  char *__restrict__ out, int hop, size_t block_bytes, int *status)
{
    __shared__ Stage<STAGED ? PACK_NT : 1> st;
    // without ROWS: a status word to clear for the kernel that follows (a fill launch of its own costs more than
    // this kernel on the smallest lattices)
    if constexpr (std::is_void<ROWS>::value)
        if (status && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *status = 0;
    const int blk = xcd_block(blockIdx.x, gridDim.x);
    const long long n = (long long)blk * PACK_NT + threadIdx.x;
    if ((long long)blk * PACK_NT >= l.V) return;
    int cs[4] = { 0, 0, 0, 0 };
    if (STAGED && n < l.V) lex_coords(l, n, cs);
    // this wavefront's tile and parity; its lane's site is canonical site 2 h + bit
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, parity = w & 1, tile = 2 * blk + (w >> 1);
    const int h = tile * TILE + lane;
    const bool valid = h < g.Vh;
    int c[4];
    site_coords(g, valid ? h : g.Vh - 1, parity, c[0], c[1], c[2], c[3]);
    const int mine = 2 * TILE * (w >> 1) + 2 * lane + (c[0] & 1);
    const long long pt = (long long)parity * g.ntiles + tile;
    // blockIdx.y: this workgroup's share of the 8 directions, each axis's two together
    const int per = 8 / gridDim.y;
#pragma unroll 1
    for (int k = blockIdx.y * per; k < (int)(blockIdx.y + 1) * per; ++k) {
        const int mu = k >> 1, d = mu + 4 * (k & 1);
        const bool bwd = d >= 4;
        if constexpr (STAGED) {
            long long src = -1;
            if (n < l.V) src = (long long)mu * l.V + (bwd ? lex_hop(l, n, cs, mu, -hop) : n);
            stage_in<PACK_NT>(st, canon, src);
        }
        if (tile >= g.ntiles) continue;  // wave-uniform; the barriers are in stage_in
        double m[18];
#pragma unroll
        for (int e = 0; e < 18; ++e) m[e] = 0.0;
        if (valid) {
            const double2 *u;
            if constexpr (STAGED) {
                u = st.m + 9 * mine;
            } else {
                const long long own = 2LL * h + (c[0] & 1);
                u = canon + 9 * ((long long)mu * l.V + (bwd ? lex_hop(l, own, c, mu, -hop) : own));
            }
            // backward: -U^dag, entry (a, b) = -conj(U_ba)
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int b = 0; b < 3; ++b) {
                    const double2 v = u[bwd ? 3 * b + a : 3 * a + b];
                    m[2 * (3 * a + b)] = bwd ? -v.x : v.x;
                    m[2 * (3 * a + b) + 1] = v.y;
                }
        }
        if constexpr (std::is_void<ROWS>::value) {
            store_block<PREC>(out + ((size_t)pt * 8 + d) * block_bytes, lane, m);
        } else {
            store_rows<PREC, ROWS>(out + (size_t)pt * ROWS::tile_bytes, d, lane, m, valid, status);
        }
    }
}

size_t dir_block_bytes(int prec)
{
    switch (prec) {
    case HISQ_F64: return PF64::block_bytes;
    case HISQ_F32: return PF32::block_bytes;
    case HISQ_F16S: return PF16S::block_bytes;
    case HISQ_I16S: return PI16S::block_bytes;
    case HISQ_F64C: return PF64::block_bytes;  // the fat field
    case HISQ_F32C: return PF32::block_bytes;
    case HISQ_I16SC: return PI16S::block_bytes;
    default: return 0;
    }
}

// fat: full blocks; long of the compressed precisions: two-row tiles plus a
// 256-byte status word after the last tile
static size_t long_field_bytes(const Geom &g, int prec)
{
    if (prec == HISQ_F64C) return 2ull * g.ntiles * PF64R::tile_bytes + 256;
    if (prec == HISQ_F32C) return 2ull * g.ntiles * PF32R::tile_bytes + 256;
    if (prec == HISQ_I16SC) return 2ull * g.ntiles * PI16R::tile_bytes + 256;
    return 2ull * g.ntiles * 8 * dir_block_bytes(prec);
}

size_t packed_field_bytes(const Geom &g, int prec)
{
    const size_t f = 2ull * g.ntiles * 8 * dir_block_bytes(prec), l = long_field_bytes(g, prec);
    return dir_block_bytes(prec) ? (f > l ? f : l) : 0;
}

}  // namespace hisq

using namespace hisq;

extern "C" size_t hisq_packed_link_bytes(const int dims[4], int prec)
{
    Geom g;
    if (make_geom(dims, g)) return 0;
    return packed_field_bytes(g, prec);
}

extern "C" int hisq_pack_links(const void *fat_canon, const void *long_canon, const int dims[4], int prec,
                               void *fat_out, void *long_out, void *stream)
{
    Geom g;
    int rc = make_geom(dims, g);
    if (rc) return rc;
    if (!fat_canon || !long_canon || !fat_out || !long_out) return fail(HISQ_EINVAL, "hisq_pack_links: NULL pointer");
    if (!aligned16({fat_canon, long_canon, fat_out, long_out}))
        return fail(HISQ_EINVAL, "hisq_pack_links: device pointers must be 16-byte aligned");
    if (fat_out == long_out) return fail(HISQ_EALIAS, "hisq_pack_links: fat_out and long_out alias");
    if (!dir_block_bytes(prec)) return fail(HISQ_EINVAL, "hisq_pack_links: unknown precision");
    hipStream_t s = (hipStream_t)stream;
    Lex l;
    if (make_lex(dims, l)) return HISQ_EDIMS;
    // where the sites alone do not fill the chip (4 workgroups per CU), the directions are shared out too
    const int nb = (int)((l.V + PACK_NT - 1) / PACK_NT), split = nb >= 1024 ? 1 : nb >= 256 ? 4 : 8;
    const dim3 grid(xcd_grid(nb), split), block(PACK_NT);
    auto launch = [&](auto kernel, const void *in, void *out, int hop, size_t bytes, int *status = nullptr) {
        hipLaunchKernelGGL(kernel, grid, block, 0, s, l, g, (const double2 *)in, (char *)out, hop, bytes, status);
    };
    const bool staged = l.V > PACK_DIRECT_SITES;
    auto full = [&](int fp, const void *in, void *out, int hop, int *clear = nullptr) {
        auto kernel = fp == HISQ_F64    ? (staged ? k_pack<HISQ_F64, void, true> : k_pack<HISQ_F64, void, false>)
                      : fp == HISQ_F32  ? (staged ? k_pack<HISQ_F32, void, true> : k_pack<HISQ_F32, void, false>)
                      : fp == HISQ_F16S ? (staged ? k_pack<HISQ_F16S, void, true> : k_pack<HISQ_F16S, void, false>)
                                        : (staged ? k_pack<HISQ_I16S, void, true> : k_pack<HISQ_I16S, void, false>);
        launch(kernel, in, out, hop, dir_block_bytes(fp), clear);
    };
    if (prec == HISQ_F64C || prec == HISQ_F32C || prec == HISQ_I16SC) {
        const int fp = prec == HISQ_F64C ? HISQ_F64 : (prec == HISQ_F32C ? HISQ_F32 : HISQ_I16S);
        int *status = reinterpret_cast<int *>((char *)long_out + long_field_bytes(g, prec) - 256);
        full(fp, fat_canon, fat_out, 1, status);
        auto rows = prec == HISQ_F64C
                        ? (staged ? k_pack<HISQ_F64C, PF64R, true> : k_pack<HISQ_F64C, PF64R, false>)
                    : prec == HISQ_F32C
                        ? (staged ? k_pack<HISQ_F32C, PF32R, true> : k_pack<HISQ_F32C, PF32R, false>)
                        : (staged ? k_pack<HISQ_I16SC, PI16R, true> : k_pack<HISQ_I16SC, PI16R, false>);
        launch(rows, long_canon, long_out, 3, (size_t)0, status);
        HISQ_HIP(hipGetLastError());
        int h_status = 0;
        HISQ_HIP(hipMemcpyAsync(&h_status, status, sizeof(int), hipMemcpyDeviceToHost, s));
        HISQ_HIP(hipStreamSynchronize(s));
        if (h_status) return fail(HISQ_EINVAL, "hisq_pack_links: a long link is not +-SU(3) to 1e-6; use an uncompressed precision");
        return HISQ_OK;
    }
    full(prec, fat_canon, fat_out, 1);
    full(prec, long_canon, long_out, 3);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "hisq_pack_links launch");
    return HISQ_OK;
}
