// Clover term (Sec. II-A; packed as two 6x6 Hermitian blocks as in Sec. III-A)
// and its inverse, built once per (links, kappa, c_SW) in FP64.
//
//   Q_{mu nu}(n) = sum of the four counter-clockwise plaquettes at n
//   Fhat_{mu nu} = (Q_{mu nu} - Q_{mu nu}^dagger) / 8
//   F = 1 - kappa c_SW sum_{mu<nu} g_mu g_nu (x) Fhat_{mu nu}
//
// In the Dirac representation g_k g_l = diag(s_k s_l, s_k s_l) and
// g_k g_t = [[0, i s_k], [i s_k, 0]], so F = [[A, B], [B, A]] with
//   A = 1 - kappa c_SW [ i s_z (x) Fhat_xy - i s_y (x) Fhat_xz + i s_x (x) Fhat_yz ]
//   B = -kappa c_SW i [ s_x (x) Fhat_xt + s_y (x) Fhat_yt + s_z (x) Fhat_zt ].
// F commutes with g5 = -[[0, 1], [1, 0]]; on the g5 = +1 space (u, -u) it acts
// as A - B and on the g5 = -1 space (u, u) as A + B.  Stored per site are
// M1 = (A - B)/2 and M2 = (A + B)/2 (and the same for the inverses), which
// is what the Dirac-basis epilogue of the stencil consumes.
//
// What bounds it: the six stored copies (2024 B a site) and the FP64 products
// (60 of 3x3 matrices a site).  At 24^3x48 it takes 634 us, 2.1 TB/s of stores;
// one thread per site with indexed 6x6 arrays in scratch took 5095 us.
//
// One workgroup builds the 64 sites of a tile.  Six wavefronts, one per plane,
// first leave Fhat of their plane in LDS; four of them then each produce one of
// the four stored blocks (F and F^-1 of either chirality).  Everything lives in
// registers: the products are unrolled, and a block is inverted in place as its
// 36 packed reals.
#include "mat3.hpp"
#include "reduce.hpp"

namespace {

// Fhat_{mu nu} at site n (EO index i of parity par), anti-Hermitian.  Only
// Q - Q^dagger is wanted, so the leaves 1 and 3 enter as minus their adjoints,
// and all four close on the same two links at either end (10 products):
//   [U_nu(n) E - U_nu(n-nu)^dag K] U_mu(n-mu) + [U_nu(n-nu)^dag H - U_nu(n) G] U_mu(n)^dag
//   E = U_mu(n+nu-mu)^dag U_nu(n-mu)^dag    G = U_mu(n+nu) U_nu(n+mu)^dag
//   H = U_mu(n-nu) U_nu(n+mu-nu)            K = U_mu(n-mu-nu)^dag U_nu(n-mu-nu)
__device__ __forceinline__ AntiHerm fhat(const Geom &g, const double2 *l64, const SiteCoord &c, int par, int mu, int nu) {
    const int n = c.x + g.L[0] * c.row;
    const int pm = lex_step(g, c, mu, true), mm = lex_step(g, c, mu, false);
    const int pn = lex_step(g, c, nu, true), mn = lex_step(g, c, nu, false);
    const size_t ls = link_slab_bytes(P64, g.Vh);
    // links rooted at n + off; odd: the root has the other parity
    auto U = [&](int dir, int off, int odd) {
        return LinkIO<P64>::load<false>((const char *)l64 + (size_t)(2 * dir + (par ^ odd)) * ls, g.Vh, (n + off) >> 1);
    };
    M3 left = mzero(), right = mzero();  // factors of U_mu(n-mu) and of U_mu(n)^dag
    {
        const M3 un = U(nu, 0, 0);
        {
            M3 et = mzero();  // E^dagger
            mmac(et, U(nu, mm, 1), U(mu, pn + mm, 0));
            mmac_d(left, un, et);
        }
        M3 gm = mzero();
        mmac_d(gm, U(mu, pn, 1), U(nu, pm, 1));
        mmac(right, un, gm);
    }
#pragma unroll
    for (int k = 0; k < 9; k++) {
        left.m[k] = -left.m[k];
        right.m[k] = -right.m[k];
    }
    {
        const M3 ub = U(nu, mn, 1);
        {
            M3 k = mzero();
            mdmac(k, U(mu, mm + mn, 0), U(nu, mm + mn, 0));
            mdmac(left, ub, k);
        }
        M3 h = mzero();
        mmac(h, U(mu, mn, 1), U(nu, pm + mn, 0));
        mdmac(right, ub, h);
    }
#pragma unroll
    for (int k = 0; k < 9; k++) left.m[k] = -left.m[k];
    M3 q = mzero();
    mmac(q, left, U(mu, mm, 1));
    mmac_d(q, right, U(mu, 0, 0));
    AntiHerm f;
#pragma unroll
    for (int k = 0; k < 3; k++) f.d[k] = 0.25 * q.m[4 * k].im;
#pragma unroll
    for (int k = 0; k < 3; k++) {
        const int a = k == 2 ? 1 : 0, b = k == 0 ? 1 : 2;  // (0,1) (0,2) (1,2)
        f.o[k] = 0.125 * (q.m[3 * a + b] - conjx(q.m[3 * b + a]));
    }
    return f;
}

// position of (i, j), i < j, among the entries above the diagonal of a Herm6
__device__ constexpr int upper(int i, int j) { return i * (11 - i) / 2 + j - i - 1; }

// In-place inverse of a Hermitian 6x6 by symmetric elimination (sweeps over the
// diagonal without row exchanges).  The pivots met on the way are the ratios of
// successive leading principal minors, so they are all positive exactly when
// the matrix is positive definite, for which elimination without exchanges is
// stable; the return value counts the pivots that are not (non-positive or
// non-finite).
__device__ __forceinline__ int inv6(Herm6<double> &m) {
    int bad = 0;
#pragma unroll
    for (int k = 0; k < 6; k++) {
        const double d = m.d[k];
        if (!(d > 0.0) || !isfinite(d)) bad++;
        const double inv = 1.0 / d;
        C v[6];  // column k
#pragma unroll
        for (int i = 0; i < 6; i++) {
            if (i == k) continue;
            v[i] = i < k ? m.o[upper(i, k)] : conjx(m.o[upper(k, i)]);
        }
#pragma unroll
        for (int i = 0; i < 6; i++) {
            if (i == k) continue;
            const C w = inv * v[i];
            m.d[i] = fmar(-w.re, v[i].re, fmar(-w.im, v[i].im, m.d[i]));
#pragma unroll
            for (int j = i + 1; j < 6; j++) {
                if (j == k) continue;
                cmacc(m.o[upper(i, j)], v[j], -w);  // -= w conj(v_j)
            }
            if (i < k) m.o[upper(i, k)] = w;
            else m.o[upper(k, i)] = conjx(w);
        }
        m.d[k] = -inv;
    }
#pragma unroll
    for (int k = 0; k < 6; k++) m.d[k] = -m.d[k];
#pragma unroll
    for (int k = 0; k < 15; k++) m.o[k] = -m.o[k];
    return bad;
}

struct CloverOut {
    char *f64, *i64;  // tiled slabs [parity], 576 B/site
    char *f32, *i32;  // 288 B/site
    char *f16, *i16;  // 148 B/site
};

constexpr int kPlanes = 6;  // (0,1) (0,2) (0,3) (1,2) (1,3) (2,3)

// bad_blocks: device counter of the 6x6 blocks (two per site) that are not
// positive definite, incremented by the kernel
__global__ __launch_bounds__(64 * kPlanes) void k_build_clover(Geom g, const double2 *l64, CloverOut o, double kc,
                                                               unsigned *bad_blocks) {
    __shared__ double fh[kPlanes][9][64];
    __shared__ float mx[4][64];  // largest entry of each stored block
    const int lb = xcd_block(blockIdx.x, gridDim.x, 64);  // both parities of a tile run on one XCD
    const int tile = lb >> 1, par = lb & 1;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int i = tile * 64 + lane;
    const bool active = i < g.Vh;
    if (active) {
        const int mu = w < 3 ? 0 : (w < 5 ? 1 : 2), nu = w < 3 ? w + 1 : (w < 5 ? w - 1 : 3);
        const AntiHerm f = fhat(g, l64, eo_coords(g, i, par), par, mu, nu);
#pragma unroll
        for (int k = 0; k < 3; k++) {
            fh[w][k][lane] = f.d[k];
            fh[w][3 + 2 * k][lane] = f.o[k].re;
            fh[w][4 + 2 * k][lane] = f.o[k].im;
        }
    }
    __syncthreads();
    const int blk = w & 1;  // 0: A - B (g5 = +1), 1: A + B (g5 = -1)
    const bool inverse = w & 2;
    Herm6<double> m;
    if (w < 4 && active) {
        // the blocks of M = A + s B in spin, from the anti-Hermitian sums
        //   P = F01 + s F23,  R = F02 - s F13,  T = F12 + s F03:
        //   M00 = 1 - i kc P,  M11 = 1 + i kc P,  M01 = kc (R - i T)
        const double s = blk ? 1.0 : -1.0;
        auto sum = [&](int p, int q, double sg) {
            AntiHerm x;
#pragma unroll
            for (int k = 0; k < 3; k++) {
                x.d[k] = fmar(sg, fh[q][k][lane], fh[p][k][lane]);
                x.o[k].re = fmar(sg, fh[q][3 + 2 * k][lane], fh[p][3 + 2 * k][lane]);
                x.o[k].im = fmar(sg, fh[q][4 + 2 * k][lane], fh[p][4 + 2 * k][lane]);
            }
            return x;
        };
        {
            const AntiHerm P = sum(0, 5, s);
#pragma unroll
            for (int a = 0; a < 3; a++) {
                m.d[a] = fmar(kc, P.d[a], 1.0);
                m.d[3 + a] = fmar(-kc, P.d[a], 1.0);
            }
#pragma unroll
            for (int k = 0; k < 3; k++) {
                const int a = k == 2 ? 1 : 0, b = k == 0 ? 1 : 2;
                m.o[upper(a, b)] = {kc * P.o[k].im, -kc * P.o[k].re};
                m.o[upper(3 + a, 3 + b)] = {-kc * P.o[k].im, kc * P.o[k].re};
            }
        }
        const AntiHerm R = sum(1, 4, -s), T = sum(3, 2, s);
#pragma unroll
        for (int a = 0; a < 3; a++)
#pragma unroll
            for (int b = 0; b < 3; b++) {
                C &e = m.o[upper(a, 3 + b)];
                if (a == b) {
                    e = {kc * T.d[a], kc * R.d[a]};
                } else {
                    const C r = ah_off(R, a, b), t = ah_off(T, a, b);
                    e = {kc * (r.re + t.im), kc * (r.im - t.re)};
                }
            }
        if (inverse && inv6(m)) atomicAdd(bad_blocks, 1u);
        // halves are stored; record order: 6 diagonal entries, then the 15 above
        double f[36];
#pragma unroll
        for (int k = 0; k < 6; k++) f[k] = 0.5 * m.d[k];
#pragma unroll
        for (int k = 0; k < 15; k++) {
            f[6 + 2 * k] = 0.5 * m.o[k].re;
            f[7 + 2 * k] = 0.5 * m.o[k].im;
        }
        char *d64 = (inverse ? o.i64 : o.f64) + (size_t)par * clover_slab_bytes(P64, g.Vh);
        char *d32 = (inverse ? o.i32 : o.f32) + (size_t)par * clover_slab_bytes(P32, g.Vh);
        double big = 0.0;
#pragma unroll
        for (int k = 0; k < 36; k++) big = fmax(big, fabs(f[k]));
        mx[w][lane] = (float)big;
#pragma unroll
        for (int k = 0; k < 18; k++)
            st_stream(tp<double2, 576>(d64, i, 16 * (18 * blk + k)), make_double2(f[2 * k], f[2 * k + 1]));
#pragma unroll
        for (int k = 0; k < 9; k++)
            st_stream(tp<float4, 288>(d32, i, 16 * (9 * blk + k)),
                      make_float4((float)f[4 * k], (float)f[4 * k + 1], (float)f[4 * k + 2], (float)f[4 * k + 3]));
    }
    __syncthreads();
    if (w >= 4 || !active) return;
    // the FP16 record shares one scale between the two blocks
    char *d16 = (inverse ? o.i16 : o.f16) + (size_t)par * clover_slab_bytes(P16, g.Vh);
    const float sc = fmaxf(mx[w & 2][lane], mx[(w & 2) + 1][lane]);
    const float inv_s = sc > 0.f ? 1.0f / sc : 0.f;
    uint32_t h[18];
#pragma unroll
    for (int k = 0; k < 18; k++) {
        const double a = k < 3 ? m.d[2 * k % 6] : m.o[(k + 12) % 15].re;
        const double b = k < 3 ? m.d[(2 * k + 1) % 6] : m.o[(k + 12) % 15].im;
        h[k] = f2h((float)(0.5 * a) * inv_s, (float)(0.5 * b) * inv_s);
    }
#pragma unroll
    for (int k = 0; k < 4; k++)
        *tp<uint4, 148>(d16, i, 72 * blk + 16 * k) = make_uint4(h[4 * k], h[4 * k + 1], h[4 * k + 2], h[4 * k + 3]);
    *tp<uint2, 148>(d16, i, 72 * blk + 64) = make_uint2(h[16], h[17]);
    if (blk == 0) *tp<float, 148>(d16, i, 144) = sc;
}

}  // namespace

int launch_build_clover(wc_lattice *lat, double kappa, double csw, unsigned *bad_blocks) {
    CloverOut o;
    o.f64 = (char *)lat->clov[P64];
    o.i64 = (char *)lat->clovinv[P64];
    o.f32 = (char *)lat->clov[P32];
    o.i32 = (char *)lat->clovinv[P32];
    o.f16 = (char *)lat->clov[P16];
    o.i16 = (char *)lat->clovinv[P16];
    const dim3 grid(2 * (pad_sites(lat->Vh) / 64));
    hipLaunchKernelGGL(k_build_clover, grid, dim3(64 * kPlanes), 0, lat->stream, lat->g,
                       (const double2 *)lat->links[P64], o, kappa * csw, bad_blocks);
    WC_HIP(hipGetLastError());
    return WC_OK;
}
