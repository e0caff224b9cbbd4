// Layout kernels: canonical complex128 fields <-> the site-tiled
// even-odd layout, and the per-precision copies of the gauge links.
#include <algorithm>

#include "reduce.hpp"

namespace {

// |third column - conj(col0 x col1)| of one link, largest entry, in FP64: how
// far the link is from what the two-column forms rebuild
__device__ __forceinline__ float recon12_error(const double2 (&m)[9]) {
    double e = 0.0;
#pragma unroll
    for (int r = 0; r < 3; r++) {
        const int r1 = (r + 1) % 3, r2 = (r + 2) % 3;
        // row r of conj(c0 x c1): conj(c0[r1] c1[r2] - c0[r2] c1[r1])
        const double2 a = m[3 * r1], b = m[3 * r2 + 1], c = m[3 * r2], d = m[3 * r1 + 1];
        const double re = (a.x * b.x - a.y * b.y) - (c.x * d.x - c.y * d.y);
        const double im = -((a.x * b.y + a.y * b.x) - (c.x * d.y + c.y * d.x));
        const double2 t = m[3 * r + 2];
        e = fmax(e, sqrt((t.x - re) * (t.x - re) + (t.y - im) * (t.y - im)));
    }
    return (float)e;
}

// Canonical fields hold a site's entries together, and consecutive sites
// alternate in parity: EO index i of both parities is the canonical pair 2i,
// 2i + 1, so a 64-site tile of both parities is 128 consecutive canonical sites.
// Loading links and unpacking spinors take such a tile per workgroup of two
// wavefronts, move its canonical side as one contiguous block through LDS, and
// give each wavefront one parity of the tiled side.  Lane by lane the canonical
// side would be one 16-byte piece per 288 or 384 bytes, 64 lines per instruction.
constexpr int kPair = 128;  // threads: both parities of a tile

// position, among the pair's 128 canonical sites, of EO index i of parity par
__device__ __forceinline__ int pair_site(const Geom &g, int i, int par) {
    const SiteCoord c = eo_coords(g, i, par);
    return 2 * (i & (kTile - 1)) + (c.x & 1);
}

// A workgroup converts several tiles and posts its largest error once: one
// posting per wavefront and tile went to the same word 83000 times at 24^3x48
// and took most of the kernel's 501 us there.  It now takes 150 us (6.2 TB/s of
// the canonical links in and the three copies out).
constexpr int kLoadBlocks = 2048;

__global__ __launch_bounds__(kPair) void k_load_links(Geom g, const double2 *U, double2 *l64, float4 *l32, char *l16,
                                                      unsigned *err_bits) {
    __shared__ double2 sh[2 * kTile * 9];
    __shared__ float worst;
    const int par = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int tiles = pad_sites(g.Vh) / kTile;
    float err = 0.f;
    for (int unit = blockIdx.x; unit < 4 * tiles; unit += gridDim.x) {
        const int mu = unit / tiles, tile = unit - mu * tiles;
        const int live = min(kTile, g.Vh - tile * kTile);
        const double2 *src = U + ((size_t)mu * 2 * g.Vh + (size_t)2 * kTile * tile) * 9;
        if (live == kTile) {
            double2 v[9];
#pragma unroll
            for (int k = 0; k < 9; k++) v[k] = ld_stream(src + threadIdx.x + kPair * k);
#pragma unroll
            for (int k = 0; k < 9; k++) sh[threadIdx.x + kPair * k] = v[k];
        } else {
            for (int k = threadIdx.x; k < 2 * live * 9; k += kPair) sh[k] = src[k];
        }
        __syncthreads();
        if (lane < live) {
            const int i = tile * kTile + lane, slab = 2 * mu + par;
            const double2 *m0 = sh + 9 * pair_site(g, i, par);
            double2 m[9];
#pragma unroll
            for (int k = 0; k < 9; k++) m[k] = m0[k];
            char *d64 = (char *)l64 + (size_t)slab * link_slab_bytes(P64, g.Vh);
#pragma unroll
            for (int k = 0; k < 9; k++) *tp<double2, 144>(d64, i, 16 * k) = m[k];
            // columns 0 and 1: U00 U10 | U20 U01 | U11 U21
            char *d32 = (char *)l32 + (size_t)slab * link_slab_bytes(P32, g.Vh);
            *tp<float4, 48>(d32, i, 0) = make_float4((float)m[0].x, (float)m[0].y, (float)m[3].x, (float)m[3].y);
            *tp<float4, 48>(d32, i, 16) = make_float4((float)m[6].x, (float)m[6].y, (float)m[1].x, (float)m[1].y);
            *tp<float4, 48>(d32, i, 32) = make_float4((float)m[4].x, (float)m[4].y, (float)m[7].x, (float)m[7].y);
            char *b16 = l16 + (size_t)slab * link_slab_bytes(P16, g.Vh);
            uint4 u;
            u.x = f2h((float)m[0].x, (float)m[0].y);
            u.y = f2h((float)m[3].x, (float)m[3].y);
            u.z = f2h((float)m[6].x, (float)m[6].y);
            u.w = f2h((float)m[1].x, (float)m[1].y);
            *tp<uint4, 24>(b16, i, 0) = u;
            *tp<uint2, 24>(b16, i, 16) = make_uint2(f2h((float)m[4].x, (float)m[4].y), f2h((float)m[7].x, (float)m[7].y));
            bool finite = true;
#pragma unroll
            for (int k = 0; k < 9; k++) finite = finite && isfinite(m[k].x) && isfinite(m[k].y);
            // a non-finite entry posts +inf, which orders above every finite error
            // (a NaN would be dropped by the max below)
            err = fmaxf(err, finite ? recon12_error(m) : INFINITY);
        }
        __syncthreads();  // the tile's links are read before the next tile's arrive
    }
    // non-negative floats order like their bits
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) err = fmaxf(err, __shfl_xor(err, off));
    if (threadIdx.x == 64) worst = err;
    __syncthreads();
    if (threadIdx.x == 0) atomicMax(err_bits, __float_as_uint(fmaxf(err, worst)));
}

// the full FP32 copy of the FP64 links (row-major, four float4 and a float2)
__global__ __launch_bounds__(kBlock) void k_links_full32(Geom g, const char *l64, char *l18) {
    const int i = blockIdx.x * kBlock + threadIdx.x;
    const int slab = blockIdx.y;  // 2 mu + parity
    if (i >= g.Vh) return;
    const char *src = l64 + (size_t)slab * link_slab_bytes(P64, g.Vh);
    double2 m[9];
#pragma unroll
    for (int k = 0; k < 9; k++) m[k] = *tp<double2, 144>(src, i, 16 * k);
    char *d = l18 + (size_t)slab * link18_slab_bytes(g.Vh);
#pragma unroll
    for (int k = 0; k < 4; k++)
        *tp<float4, 72>(d, i, 16 * k) = make_float4((float)m[2 * k].x, (float)m[2 * k].y, (float)m[2 * k + 1].x,
                                                    (float)m[2 * k + 1].y);
    *tp<float2, 72>(d, i, 64) = make_float2((float)m[8].x, (float)m[8].y);
}

// reconstruct-8 copy of the FP64 links and the smallest N = |U01|^2 + |U02|^2
// (as FP32 bits, which order like the non-negative values they encode)
__global__ __launch_bounds__(kBlock) void k_links_recon8(Geom g, const char *l64, char *l8, unsigned *min_bits) {
    const int i = blockIdx.x * kBlock + threadIdx.x;
    const int slab = blockIdx.y;  // 2 mu + parity
    float n32 = 3.0e38f;
    if (i < g.Vh) {
        const char *src = l64 + (size_t)slab * link_slab_bytes(P64, g.Vh);
        double2 m[9];
#pragma unroll
        for (int k = 0; k < 9; k++) m[k] = *tp<double2, 144>(src, i, 16 * k);
        const double2 a2 = m[1], a3 = m[2], b1 = m[3], c1 = m[6];
        const bool swap = (b1.x * b1.x + b1.y * b1.y) > (c1.x * c1.x + c1.y * c1.y);
        const double2 y = swap ? c1 : b1, z = swap ? b1 : c1;
        const double ta = atan2(m[0].y, m[0].x) / M_PI;
        double tz = atan2(z.y, z.x) / M_PI;
        if (tz < 0.0) tz += 2.0;  // [0, 2]: the sign bit is free for the flag
        char *d = l8 + (size_t)slab * link8_slab_bytes(g.Vh);
        const float4 p0 = make_float4((float)a2.x, (float)a2.y, (float)a3.x, (float)a3.y);
        *tp<float4, 32>(d, i, 0) = p0;
        const float tzf = (float)tz;
        *tp<float4, 32>(d, i, 16) = make_float4((float)y.x, (float)y.y, (float)ta, swap ? -tzf : tzf);
        n32 = p0.x * p0.x + p0.y * p0.y + p0.z * p0.z + p0.w * p0.w;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) n32 = fminf(n32, __shfl_xor(n32, off));
    if ((threadIdx.x & 63) == 0) atomicMin(min_bits, __float_as_uint(n32));
}

// Packing reads its canonical side lane by lane all the same: the reads of the
// two parities meet in the caches and it runs at the rate of a copy (5.1 TB/s at
// 24^3x48, 18 us at 20x12x28x36), where the way through LDS took 22 us.
template <int P>
__global__ __launch_bounds__(kBlock) void k_pack(Geom g, char *eo, const double2 *canon, size_t slab_bytes) {
    using R = typename Real<P>::T;
    const int i = blockIdx.x * kBlock + threadIdx.x;
    const int par = blockIdx.y;
    if (i >= g.Vh) return;
    const SiteCoord c = eo_coords(g, i, par);
    const size_t n = (size_t)c.x + (size_t)g.L[0] * c.row;
    const double2 *src = canon + n * 12;
    Spinor<R> s;
#pragma unroll
    for (int k = 0; k < 12; k++) {
        double2 v = src[k];
        s.c[k] = {(R)v.x, (R)v.y};
    }
    SpinorIO<P>::store(eo + par * slab_bytes, g.Vh, i, s);
}

// LDS stride of a spinor site: 13 entries, so that lanes two sites apart start
// 8 banks apart (12 would put them on two bank groups)
constexpr int kPadSpin = 13;

// 55 -> 45 us at 24^3x48 against lane-by-lane stores (5.7 TB/s)
template <int P>
__global__ __launch_bounds__(kPair) void k_unpack(Geom g, double2 *canon, const char *eo, size_t slab_bytes) {
    using R = typename Real<P>::T;
    __shared__ double2 sh[2 * kTile * kPadSpin];
    const int par = threadIdx.x >> 6, lane = threadIdx.x & 63, tile = blockIdx.x;
    const int live = min(kTile, g.Vh - tile * kTile);
    if (lane < live) {
        const int i = tile * kTile + lane;
        const Spinor<R> s = SpinorIO<P>::load(eo + par * slab_bytes, g.Vh, i);
        double2 *p = sh + kPadSpin * pair_site(g, i, par);
#pragma unroll
        for (int k = 0; k < 12; k++) p[k] = make_double2((double)s.c[k].re, (double)s.c[k].im);
    }
    __syncthreads();
    double2 *dst = canon + (size_t)2 * kTile * tile * 12;
#pragma unroll
    for (int k = 0; k < 12; k++) {
        const int e = threadIdx.x + kPair * k;
        if (e < 2 * live * 12) st_stream(dst + e, sh[e / 12 * kPadSpin + e % 12]);
    }
}

}  // namespace

int launch_load_links(wc_lattice *lat, const void *U, unsigned *err_bits) {
    const dim3 grid(std::min(kLoadBlocks, 4 * (pad_sites(lat->Vh) / kTile)));
    hipLaunchKernelGGL(k_load_links, grid, dim3(kPair), 0, lat->stream, lat->g, (const double2 *)U,
                       (double2 *)lat->links[P64], (float4 *)lat->links[P32], (char *)lat->links[P16], err_bits);
    WC_HIP(hipGetLastError());
    return WC_OK;
}

int launch_links_full32(wc_lattice *lat) {
    dim3 grid((lat->Vh + kBlock - 1) / kBlock, 8);
    hipLaunchKernelGGL(k_links_full32, grid, dim3(kBlock), 0, lat->stream, lat->g, (const char *)lat->links[P64],
                       (char *)lat->links18);
    WC_HIP(hipGetLastError());
    return WC_OK;
}

int launch_links_recon8(wc_lattice *lat, unsigned *min_bits) {
    dim3 grid((lat->Vh + kBlock - 1) / kBlock, 8);
    hipLaunchKernelGGL(k_links_recon8, grid, dim3(kBlock), 0, lat->stream, lat->g, (const char *)lat->links[P64],
                       (char *)lat->links8, min_bits);
    WC_HIP(hipGetLastError());
    return WC_OK;
}

int launch_pack_spinor(wc_lattice *lat, int prec, void *eo_out, const void *canon_in) {
    dim3 grid((lat->Vh + kBlock - 1) / kBlock, 2);
    const size_t sb = spinor_bytes(prec, lat->Vh);
    if (prec == P64)
        hipLaunchKernelGGL(k_pack<P64>, grid, dim3(kBlock), 0, lat->stream, lat->g, (char *)eo_out,
                           (const double2 *)canon_in, sb);
    else if (prec == P32)
        hipLaunchKernelGGL(k_pack<P32>, grid, dim3(kBlock), 0, lat->stream, lat->g, (char *)eo_out,
                           (const double2 *)canon_in, sb);
    else
        hipLaunchKernelGGL(k_pack<P16>, grid, dim3(kBlock), 0, lat->stream, lat->g, (char *)eo_out,
                           (const double2 *)canon_in, sb);
    WC_HIP(hipGetLastError());
    return WC_OK;
}

int launch_unpack_spinor(wc_lattice *lat, int prec, void *canon_out, const void *eo_in) {
    const dim3 grid(pad_sites(lat->Vh) / kTile);
    const size_t sb = spinor_bytes(prec, lat->Vh);
    if (prec == P64)
        hipLaunchKernelGGL(k_unpack<P64>, grid, dim3(kPair), 0, lat->stream, lat->g, (double2 *)canon_out,
                           (const char *)eo_in, sb);
    else if (prec == P32)
        hipLaunchKernelGGL(k_unpack<P32>, grid, dim3(kPair), 0, lat->stream, lat->g, (double2 *)canon_out,
                           (const char *)eo_in, sb);
    else
        hipLaunchKernelGGL(k_unpack<P16>, grid, dim3(kPair), 0, lat->stream, lat->g, (double2 *)canon_out,
                           (const char *)eo_in, sb);
    WC_HIP(hipGetLastError());
    return WC_OK;
}
