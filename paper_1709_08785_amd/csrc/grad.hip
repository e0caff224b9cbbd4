// Gradient of a solve with respect to the gauge links.
//
// For L = Re<eta, D^-1 b> (or any real loss with dL = Re<eta, dx>) the adjoint
// solve gives lam = D^-dagger eta = g5 D^-1 g5 eta (D is gamma5-Hermitian),
// and dL = -Re<lam, (dD) x> with dD = dF - kappa dH (eq. 3).  The gradient G
// of a link (torch convention: dL = Re sum conj(G_ab) dU_ab) has
//
//   hopping part (eq. 4), link U_mu(m):
//     G += kappa sum_alpha [ lam(m)_alpha ((1 - g_mu) x(m+mu))_alpha^dagger
//                          + ((1 + g_mu) x(m))_alpha lam(m+mu)_alpha^dagger ]
//   clover part: per site n and plane mu<nu,
//     M_ab = sum conj(lam_{alpha a}) (g_mu g_nu)_{alpha beta} x_{beta b},  N = M - M^dagger,
//     and a leaf f1 f2 f3 f4 of Q_{mu nu}(n) whose factor k is the link contributes
//     (kappa c_SW / 8) (B N^T A)^dagger (or B N^T A when the factor is daggered),
//     A = f1..f_{k-1}, B = f_{k+1}..f4.
//
// Summed over the four leaf sites of a plaquette the clover part closes into
// staples with X = N^T inserted at the corners.  For link d at m, other
// direction e, and the path a b c from m+d back to m around the plaquette,
//   S = X(m+d) a b c + a X(.) b c + a b X(.) c + a b c X(m)
//     = ((X1 a + a X2) b + (a b) X3) c + (a b c) X0,
// and the link receives +-(S_up - S_down)^dagger, + for d < e: where the
// plaquette holds the link daggered, its term is S taken with X^dagger in
// place of X, and X^dagger = -X.
//
// The clover part is a gather: one thread per link visits its 6 plaquettes,
// so no two threads write the same link and the result is deterministic.
#include "mat3.hpp"
#include "reduce.hpp"

namespace {

// (1 - s g_mu) psi for s = +1, (1 + g_mu) psi for s = -1, Dirac representation
__device__ void one_minus_gamma(int mu, bool minus, const Spinor<double> &p, Spinor<double> &o) {
#pragma unroll
    for (int a = 0; a < 3; a++) {
        const C p0 = p.c[a], p1 = p.c[3 + a], p2 = p.c[6 + a], p3 = p.c[9 + a];
        C o0, o1, o2, o3;
        if (mu == 0) {
            if (minus) { o0 = p0 + mul_i(p3); o1 = p1 + mul_i(p2); o2 = p2 - mul_i(p1); o3 = p3 - mul_i(p0); }
            else       { o0 = p0 - mul_i(p3); o1 = p1 - mul_i(p2); o2 = p2 + mul_i(p1); o3 = p3 + mul_i(p0); }
        } else if (mu == 1) {
            if (minus) { o0 = p0 + p3; o1 = p1 - p2; o2 = p2 - p1; o3 = p3 + p0; }
            else       { o0 = p0 - p3; o1 = p1 + p2; o2 = p2 + p1; o3 = p3 - p0; }
        } else if (mu == 2) {
            if (minus) { o0 = p0 + mul_i(p2); o1 = p1 - mul_i(p3); o2 = p2 - mul_i(p0); o3 = p3 + mul_i(p1); }
            else       { o0 = p0 - mul_i(p2); o1 = p1 + mul_i(p3); o2 = p2 + mul_i(p0); o3 = p3 - mul_i(p1); }
        } else {
            const C z = {0, 0};
            if (minus) { o0 = z; o1 = z; o2 = p2 + p2; o3 = p3 + p3; }
            else       { o0 = p0 + p0; o1 = p1 + p1; o2 = z; o3 = z; }
        }
        o.c[a] = o0;
        o.c[3 + a] = o1;
        o.c[6 + a] = o2;
        o.c[9 + a] = o3;
    }
}

// (g_mu g_nu) psi for plane p = (0,1) (0,2) (0,3) (1,2) (1,3) (2,3)
__device__ void gamma_pair(int plane, const Spinor<double> &p, Spinor<double> &o) {
#pragma unroll
    for (int a = 0; a < 3; a++) {
        const C p0 = p.c[a], p1 = p.c[3 + a], p2 = p.c[6 + a], p3 = p.c[9 + a];
        C o0, o1, o2, o3;
        switch (plane) {
        case 0: o0 = mul_i(p0); o1 = mul_mi(p1); o2 = mul_i(p2); o3 = mul_mi(p3); break;   // i s_z
        case 1: o0 = -p1; o1 = p0; o2 = -p3; o3 = p2; break;                               // -i s_y
        case 2: o0 = mul_i(p3); o1 = mul_i(p2); o2 = mul_i(p1); o3 = mul_i(p0); break;     // off-diag i s_x
        case 3: o0 = mul_i(p1); o1 = mul_i(p0); o2 = mul_i(p3); o3 = mul_i(p2); break;     // i s_x
        case 4: o0 = p3; o1 = -p2; o2 = p1; o3 = -p0; break;                               // off-diag i s_y
        default: o0 = mul_i(p2); o1 = mul_mi(p3); o2 = mul_i(p0); o3 = mul_mi(p1); break;  // off-diag i s_z
        }
        o.c[a] = o0;
        o.c[3 + a] = o1;
        o.c[6 + a] = o2;
        o.c[9 + a] = o3;
    }
}

__device__ __forceinline__ int plane_of(int mu, int nu) {
    // mu < nu
    return mu == 0 ? nu - 1 : (mu == 1 ? nu + 1 : 5);
}

// X_{mu nu}(n) = N^T = (M - M^dagger)^T for the 6 planes: per (plane, parity) a slab of
// 64-site tiles, the 9 reals of AntiHerm plane after plane
constexpr int kXSite = 9 * 8;  // bytes per site
__host__ __device__ inline size_t x_slab_bytes(int Vh) { return (size_t)pad_sites(Vh) * kXSite; }

__device__ __forceinline__ AntiHerm load_x(const char *slab, int i) {
    AntiHerm x;
#pragma unroll
    for (int k = 0; k < 3; k++) x.d[k] = *tp<double, kXSite>(slab, i, 8 * k);
#pragma unroll
    for (int k = 0; k < 3; k++)
        x.o[k] = {*tp<double, kXSite>(slab, i, 24 + 16 * k), *tp<double, kXSite>(slab, i, 32 + 16 * k)};
    return x;
}

__global__ __launch_bounds__(kBlock) void k_grad_X(Geom g, const char *lam, const char *x, size_t sb, char *X) {
    const int i = blockIdx.x * kBlock + threadIdx.x;
    const int par = blockIdx.y;
    if (i >= g.Vh) return;
    const Spinor<double> l = SpinorIO<P64>::load(lam + par * sb, g.Vh, i);
    const Spinor<double> xv = SpinorIO<P64>::load(x + par * sb, g.Vh, i);
#pragma unroll
    for (int p = 0; p < 6; p++) {
        Spinor<double> y;
        gamma_pair(p, xv, y);
        C M[9];
#pragma unroll
        for (int a = 0; a < 3; a++)
#pragma unroll
            for (int b = 0; b < 3; b++) {
                C s = {0, 0};
#pragma unroll
                for (int al = 0; al < 4; al++) cmacc(s, l.c[3 * al + a], y.c[3 * al + b]);
                M[3 * a + b] = s;
            }
        char *slab = X + (size_t)(2 * p + par) * x_slab_bytes(g.Vh);
#pragma unroll
        for (int k = 0; k < 3; k++) *tp<double, kXSite>(slab, i, 8 * k) = 2.0 * M[4 * k].im;
#pragma unroll
        for (int k = 0; k < 3; k++) {
            const int a = k == 2 ? 1 : 0, b = k == 0 ? 1 : 2;  // (0,1) (0,2) (1,2)
            const C v = M[3 * b + a] - conjx(M[3 * a + b]);
            *tp<double, kXSite>(slab, i, 24 + 16 * k) = v.re;
            *tp<double, kXSite>(slab, i, 32 + 16 * k) = v.im;
        }
    }
}

// h += sum over spin of a b^dagger
__device__ __forceinline__ void outer_mac(M3 &h, const Spinor<double> &a, const Spinor<double> &b) {
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++)
#pragma unroll
            for (int al = 0; al < 4; al++) cmacc(h.m[3 * i + j], b.c[3 * al + j], a.c[3 * al + i]);
}

// The gradient of a tile of 64 sites of one parity, one wavefront per link
// direction.  The clover part sums 6 plaquettes of 8 matrix products each, the
// hopping part is added, and the link is written once.
//
// What bounds it: with the clover part, FP64 arithmetic (48 products of 3x3
// matrices, about 10 kflop a link) and the loads that feed it, 3.9 KB a link
// through the caches; the four directions of a tile sit in one workgroup so
// that they find each other's links and X in L1.  At 24^3x48 it takes 1067 us
// (26 TFLOP/s; k_grad_X 97 us before it), where a gather over 24 leaf slots and
// a separate hopping kernel took 5351 + 506 us.  The links leave through LDS:
// a lane's 9 entries are 144 bytes at a stride of 288 (the other parity's sites
// lie between), which as lane-wise stores touches 64 lines per instruction.
template <bool CLOVER>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2))) void k_grad(
    Geom g, const char *lam, const char *x, size_t sb, const double2 *l64, const char *X, double2 *G, double kappa,
    double fac) {
    __shared__ double2 sh[kWaves][64 * 9];
    const int lb = xcd_block(blockIdx.x, gridDim.x, 64);  // both parities of a tile run on one XCD
    const int tile = lb >> 1, par = lb & 1;
    const int d = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int i = tile * 64 + lane;
    const int live = min(64, g.Vh - tile * 64);
    if (lane < live) {
        const SiteCoord c = eo_coords(g, i, par);
        const int n = c.x + g.L[0] * c.row;
        const int sd = lex_step(g, c, d, true);
        const int nd = (n + sd) >> 1;
        M3 acc = mzero();
        if (CLOVER) {
            const size_t ls = link_slab_bytes(P64, g.Vh);
            const char *L = (const char *)l64;
            M3 sum = mzero();
#pragma unroll 1
            for (int k = 0; k < 6; k++) {
                const int e = (k >> 1) + ((k >> 1) >= d ? 1 : 0);
                const bool up = !(k & 1);
                const int se = lex_step(g, c, e, up);
                const int ne = (n + se) >> 1, nde = (n + sd + se) >> 1;
                const int mu = min(d, e), nu = max(d, e);
                const char *xs0 = X + (size_t)(2 * plane_of(mu, nu) + par) * x_slab_bytes(g.Vh);
                const char *xs1 = X + (size_t)(2 * plane_of(mu, nu) + 1 - par) * x_slab_bytes(g.Vh);
                // path m+d -> m+d+-e -> m+-e -> m: the e link beside m+d, the d
                // link across (always daggered) and the e link beside m
                const Mat3<double> ue = LinkIO<P64>::load<false>(L + (size_t)(2 * e + (up ? 1 - par : par)) * ls, g.Vh,
                                                                 up ? nd : nde);
                const M3 a = up ? ue : mdag(ue);
                M3 q = mzero();
                xmac(q, load_x(xs1, nd), a);
                macx(q, a, load_x(xs0, nde));
                const Mat3<double> ud = LinkIO<P64>::load<false>(L + (size_t)(2 * d + 1 - par) * ls, g.Vh, ne);
                M3 r = mzero(), q2 = mzero();
                mmac_d(r, a, ud);
                mmac_d(q2, q, ud);
                macx(q2, r, load_x(xs1, ne));
                const Mat3<double> uc = LinkIO<P64>::load<false>(L + (size_t)(2 * e + (up ? par : 1 - par)) * ls, g.Vh,
                                                                 up ? i : ne);
                const M3 cc = up ? mdag(uc) : uc;
                M3 rc = mzero(), s = mzero();
                mmac(rc, r, cc);
                mmac(s, q2, cc);
                macx(s, rc, load_x(xs0, i));
                const double sg = ((d < e) == up) ? 1.0 : -1.0;
#pragma unroll
                for (int j = 0; j < 9; j++) sum.m[j] = sum.m[j] + sg * s.m[j];
            }
#pragma unroll
            for (int a = 0; a < 3; a++)
#pragma unroll
                for (int b = 0; b < 3; b++) acc.m[3 * a + b] = fac * conjx(sum.m[3 * b + a]);
        }
        {
            // kappa [lam(m) ((1 - g_d) x(m+d))^dag + ((1 + g_d) x(m)) lam(m+d)^dag]
            M3 h = mzero();
            Spinor<double> y;
            {
                const Spinor<double> lm = SpinorIO<P64>::load(lam + par * sb, g.Vh, i);
                one_minus_gamma(d, true, SpinorIO<P64>::load(x + (1 - par) * sb, g.Vh, nd), y);
                outer_mac(h, lm, y);
            }
            {
                const Spinor<double> lp = SpinorIO<P64>::load(lam + (1 - par) * sb, g.Vh, nd);
                one_minus_gamma(d, false, SpinorIO<P64>::load(x + par * sb, g.Vh, i), y);
                outer_mac(h, y, lp);
            }
#pragma unroll
            for (int k = 0; k < 9; k++) acc.m[k] = acc.m[k] + kappa * h.m[k];
        }
#pragma unroll
        for (int k = 0; k < 9; k++) sh[d][lane * 9 + k] = make_double2(acc.m[k].re, acc.m[k].im);
    }
    __syncthreads();
    double2 *out = G + (size_t)d * 2 * g.Vh * 9;
    for (int k = lane; k < live * 9; k += 64) {
        const int s = k / 9;
        const SiteCoord c = eo_coords(g, tile * 64 + s, par);
        out[(size_t)(c.x + g.L[0] * c.row) * 9 + (k - 9 * s)] = sh[d][k];
    }
}

}  // namespace

size_t grad_x_bytes(const wc_lattice *lat) { return 12 * x_slab_bytes(lat->Vh); }

int launch_link_grad(wc_lattice *lat, const void *lam_eo, const void *x_eo, void *G, void *Xbuf, double kappa,
                     double csw, bool clover) {
    const size_t sb = spinor_bytes(P64, lat->Vh);
    const dim3 grid(2 * (pad_sites(lat->Vh) / 64));
    if (!clover) {
        hipLaunchKernelGGL(k_grad<false>, grid, dim3(kBlock), 0, lat->stream, lat->g, (const char *)lam_eo,
                           (const char *)x_eo, sb, (const double2 *)lat->links[P64], (const char *)nullptr,
                           (double2 *)G, kappa, 0.0);
        WC_HIP(hipGetLastError());
        return WC_OK;
    }
    dim3 gridX((lat->Vh + kBlock - 1) / kBlock, 2);
    hipLaunchKernelGGL(k_grad_X, gridX, dim3(kBlock), 0, lat->stream, lat->g, (const char *)lam_eo,
                       (const char *)x_eo, sb, (char *)Xbuf);
    WC_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_grad<true>, grid, dim3(kBlock), 0, lat->stream, lat->g, (const char *)lam_eo,
                       (const char *)x_eo, sb, (const double2 *)lat->links[P64], (const char *)Xbuf, (double2 *)G,
                       kappa, kappa * csw / 8.0);
    WC_HIP(hipGetLastError());
    return WC_OK;
}
