// The hopping stencil with spin projection and its clover epilogues (MULT of
// Sec. II-B, eq. 9, and the Schur operator D-hat_ee of eq. 8).
//
// k_mult takes one thread per output site of one parity, k_mult_split four (a
// wavefront per direction of a 64-site tile), and k_mult_multi one tile for all
// systems of a batch.  For each of the 8 directions the
// neighbour spinor (opposite parity) is projected to a two-spin half spinor,
// multiplied by U_mu(n) (forward) or U_mu(n - mu)^dagger (backward), and
// expanded back into the accumulator (eq. 4).  In the Dirac representation:
//   (1 - g_k) psi = (h, -i s_k h),  h = psi_u + i s_k psi_d     (k = x, y, z)
//   (1 + g_k) psi = (h',  i s_k h'), h' = psi_u - i s_k psi_d
//   (1 - g_t) psi = (0, 2 psi_d),    (1 + g_t) psi = (2 psi_u, 0)
// so each direction costs two 3x3 complex matrix-vector products.
// Neighbour spinors are ordinary cached loads (each is read by 8 output sites);
// clover blocks, and links too large for the last-level cache, are read exactly
// once per launch and use non-temporal loads so they do not evict the spinor
// working set (OperatorReads below).
//
// Workgroups are handed to the 8 XCDs round-robin, and each XCD has its own
// L2.  The block index is remapped (xcd_block) so that XCD k sweeps contiguous
// chunks of the lattice: the y and z neighbours a block needs were then loaded by
// blocks of the same XCD shortly before, and hit in that XCD's L2.
#include <hip/hip_cooperative_groups.h>

#include <algorithm>

#include "reduce.hpp"

namespace {

struct MultKArgs {
    Geom g;
    int out_par;
    void *out;
    const void *in;
    const void *center;
    const void *aux;
    const char *links;   // base of the 8 link slabs of this precision
    size_t link_slab;    // bytes per (mu, parity) slab
    const void *clov;    // clover slab (F or F^-1) of the output parity
    double coef;
    RedTarget red;
    const int *done;
    int nblk;            // blocks of this system
};

struct MultBatch {
    BatchHdr h;
    MultKArgs d[kMaxSys];
};

// the fused reductions: v[0..1] += <ax, out>, and with NORM v[2] += ||out||^2
template <bool DOT, bool NORM, int NC, class R>
__device__ __forceinline__ void red_add(double *v, const cx<R> *ax, const cx<R> *out) {
#pragma unroll
    for (int k = 0; k < NC; k++) {
        const double orr = out[k].re, oi = out[k].im;
        if (DOT) {
            const double ar = ax[k].re, ai = ax[k].im;
            v[0] += ar * orr + ai * oi;
            v[1] += ar * oi - ai * orr;
        }
        if (NORM) v[2] += orr * orr + oi * oi;
    }
}

// g = U h (dag = false) or U^dagger h (dag = true), two spin components
template <class R, bool DAG>
__device__ __forceinline__ void su3_mul2(const Mat3<R> &U, const cx<R> (&h)[2][3], cx<R> (&g)[2][3]) {
#pragma unroll
    for (int s = 0; s < 2; s++) {
#pragma unroll
        for (int a = 0; a < 3; a++) {
            cx<R> acc = {R(0), R(0)};
#pragma unroll
            for (int b = 0; b < 3; b++) {
                if (DAG)
                    cmacc(acc, U.m[3 * b + a], h[s][b]);
                else
                    cmac(acc, U.m[3 * a + b], h[s][b]);
            }
            g[s][a] = acc;
        }
    }
}

// accumulate (1 -+ g_mu) U psi for direction mu; FWD selects the forward hop.
// SC: psi holds stored values whose site scale is sc (FP16 storage); the
// scale then rides on the accumulation, where every update is an FMA anyway.
template <class R, int MU, bool FWD, bool SC>
__device__ __forceinline__ void hop_term(const Spinor<R> &p, const Mat3<R> &U, Spinor<R> &acc, R sc) {
    cx<R> h[2][3], g[2][3];
#pragma unroll
    for (int a = 0; a < 3; a++) {
        const cx<R> p0 = p.c[a], p1 = p.c[3 + a], p2 = p.c[6 + a], p3 = p.c[9 + a];
        if (MU == 0) {
            h[0][a] = FWD ? p0 + mul_i(p3) : p0 - mul_i(p3);
            h[1][a] = FWD ? p1 + mul_i(p2) : p1 - mul_i(p2);
        } else if (MU == 1) {
            h[0][a] = FWD ? p0 + p3 : p0 - p3;
            h[1][a] = FWD ? p1 - p2 : p1 + p2;
        } else if (MU == 2) {
            h[0][a] = FWD ? p0 + mul_i(p2) : p0 - mul_i(p2);
            h[1][a] = FWD ? p1 - mul_i(p3) : p1 + mul_i(p3);
        } else {
            h[0][a] = FWD ? p2 + p2 : p0 + p0;
            h[1][a] = FWD ? p3 + p3 : p1 + p1;
        }
    }
    su3_mul2<R, !FWD>(U, h, g);
    auto S = [&](cx<R> v) { return SC ? sc * v : v; };
#pragma unroll
    for (int a = 0; a < 3; a++) {
        const cx<R> g0 = g[0][a], g1 = g[1][a];
        if (MU == 3) {
            if (FWD) {
                acc.c[6 + a] = acc.c[6 + a] + S(g0);
                acc.c[9 + a] = acc.c[9 + a] + S(g1);
            } else {
                acc.c[a] = acc.c[a] + S(g0);
                acc.c[3 + a] = acc.c[3 + a] + S(g1);
            }
            continue;
        }
        acc.c[a] = acc.c[a] + S(g0);
        acc.c[3 + a] = acc.c[3 + a] + S(g1);
        if (MU == 0) {
            acc.c[6 + a] = acc.c[6 + a] + S(FWD ? mul_mi(g1) : mul_i(g1));
            acc.c[9 + a] = acc.c[9 + a] + S(FWD ? mul_mi(g0) : mul_i(g0));
        } else if (MU == 1) {
            acc.c[6 + a] = FWD ? acc.c[6 + a] - S(g1) : acc.c[6 + a] + S(g1);
            acc.c[9 + a] = FWD ? acc.c[9 + a] + S(g0) : acc.c[9 + a] - S(g0);
        } else {
            acc.c[6 + a] = acc.c[6 + a] + S(FWD ? mul_mi(g0) : mul_i(g0));
            acc.c[9 + a] = acc.c[9 + a] + S(FWD ? mul_i(g1) : mul_mi(g1));
        }
    }
}

// one neighbour: load its spinor and add its hop; FP16 storage leaves the
// site scale to the accumulation (hop_term, SC)
template <int P, int MU, bool FWD>
__device__ __forceinline__ void hop_one(const void *in, int Vh, int n, const Mat3<typename Real<P>::T> &U,
                                        Spinor<typename Real<P>::T> &acc) {
    using R = typename Real<P>::T;
    if constexpr (P == P16) {
        float sc;
        const Spinor<R> psi = SpinorIO<P16>::load_raw(in, Vh, n, sc);
        hop_term<R, MU, FWD, true>(psi, U, acc, sc);
    } else {
        hop_term<R, MU, FWD, false>(SpinorIO<P>::load(in, Vh, n), U, acc, R(1));
    }
}

template <int P, int MU, bool NT, int LR>
__device__ __forceinline__ void hop_dir(const MultKArgs &a, const SiteCoord &c, int i,
                                        Spinor<typename Real<P>::T> &acc) {
    using R = typename Real<P>::T;
    const int Vh = a.g.Vh;
    if constexpr (P == P16) {
        // FP16 storage: every load of both hops is issued before the first
        // conversion.  Its loads are small (half the bytes of FP32), and with
        // one hop's loads in flight at a time the waves waited on latency;
        // two hops' loads in flight took the MULT from 86.6-87.9 to 83.9-84.7
        // us at 32^3x64, with results bit for bit the same.
        const int nf = eo_neighbour(a.g, c, MU, +1);
        const int nb = eo_neighbour(a.g, c, MU, -1);
        const char *lf = a.links + (size_t)(2 * MU + a.out_par) * a.link_slab;
        const char *lk = a.links + (size_t)(2 * MU + 1 - a.out_par) * a.link_slab;
        const uint4 fa = ld_op<NT>(tp<uint4, 24>(lf, i, 0));
        const uint2 fb = ld_op<NT>(tp<uint2, 24>(lf, i, 16));
        const uint4 ba = ld_op<NT>(tp<uint4, 24>(lk, nb, 0));
        const uint2 bb = ld_op<NT>(tp<uint2, 24>(lk, nb, 16));
        uint4 sf[3], sb[3];
#pragma unroll
        for (int k = 0; k < 3; k++) {
            sf[k] = *tp<uint4, 52>(a.in, nf, 16 * k);
            sb[k] = *tp<uint4, 52>(a.in, nb, 16 * k);
        }
        const float scf = *tp<float, 52>(a.in, nf, 48), scb = *tp<float, 52>(a.in, nb, 48);
        hop_term<R, MU, true, true>(SpinorIO<P16>::decode(sf), LinkIO<P16>::decode(fa, fb), acc, scf);
        hop_term<R, MU, false, true>(SpinorIO<P16>::decode(sb), LinkIO<P16>::decode(ba, bb), acc, scb);
        return;
    }
    if constexpr (P == P32 && LR == 8) {
        // reconstruct-8 links: both hops' links and spinors are loaded before
        // either hop is computed, so the loads overlap the rebuild of the
        // links (MULT 144.2 -> 140.3 us, D-hat half 154.8 -> 147.3 us at
        // 32^3x64, bit for bit the same).  The two-column and full forms
        // gain nothing from it and keep the one-hop order.
        const int nf = eo_neighbour(a.g, c, MU, +1);
        const int nb = eo_neighbour(a.g, c, MU, -1);
        const Mat3<R> Uf = LinkLoad<P, LR>::template load<NT>(a.links + (size_t)(2 * MU + a.out_par) * a.link_slab, Vh, i);
        const Mat3<R> Ub =
            LinkLoad<P, LR>::template load<NT>(a.links + (size_t)(2 * MU + 1 - a.out_par) * a.link_slab, Vh, nb);
        const Spinor<R> pf = SpinorIO<P32>::load(a.in, Vh, nf);
        const Spinor<R> pb = SpinorIO<P32>::load(a.in, Vh, nb);
        hop_term<R, MU, true, false>(pf, Uf, acc, R(1));
        hop_term<R, MU, false, false>(pb, Ub, acc, R(1));
        return;
    }
    {
        const int nf = eo_neighbour(a.g, c, MU, +1);
        const Mat3<R> U = LinkLoad<P, LR>::template load<NT>(a.links + (size_t)(2 * MU + a.out_par) * a.link_slab, Vh, i);
        hop_one<P, MU, true>(a.in, Vh, nf, U, acc);
    }
    {
        const int nb = eo_neighbour(a.g, c, MU, -1);
        const Mat3<R> U =
            LinkLoad<P, LR>::template load<NT>(a.links + (size_t)(2 * MU + 1 - a.out_par) * a.link_slab, Vh, nb);
        hop_one<P, MU, false>(a.in, Vh, nb, U, acc);
    }
}

// How a stencil launch reads the operator.  SHARED: links and clover through the
// cache, since the launch serves several systems (or both parities) on one
// lattice.  STREAM: each read once by its one system, non-temporal.  KEEP: the
// clover streams, the links go through the cache: MULT and the D-hat half after
// it read the same links, and where they fit in the last-level cache
// the next launch finds them there.  The clover, read by every second launch
// only, would push them out: cached as well, a solve at 24^2x32x48 took 429 us
// per inner iteration instead of 387 (streamed links: 409).
//
// kKeepLinkBytes: up to which size of a launch's links, over all its lattices.
// The cache holds 256 MB, and spinors and clover pass through it too.  us per
// inner iteration, STREAM -> KEEP: FP32 16^4 (13 MB) 69.9 -> 65.2, 16^3x32 91.1
// -> 85.3, 24^3x48 (127 MB) 322 -> 306, 24^2x32x48 (170 MB) 409 -> 387, but
// 28^2x32x48 (231 MB) 539 -> 548 and 32^3x48 (302 MB) 687 -> 735; FP64
// 12x14x10x18 67.8 -> 63.1, 20^3x40 (184 MB) 352 -> 332, 24^3x48 (382 MB) 679 ->
// 697; FP16 24^3x48 (64 MB) 219 -> 214, 32^3x48 (151 MB) 417 -> 384.  The
// multi-system kernel reads a link once for all its systems and gained nothing.
// Reconstruct-8 links keep to it in a solve (us per iteration 32^4 (134 MB) 448 ->
// 429, 28^2x32x48 (154 MB) 528 -> 505), but a launch by itself, with fewer waves
// in flight than the other forms, gains only up to kKeepLinkBytes8: D-hat_ee
// 24^3x48 (85 MB) 106.6 -> 104.2, 24^2x32x48 (113 MB) 133 -> 132, 32^4 150 -> 155,
// 28^2x32x48 180 -> 183.
constexpr double kKeepLinkBytes = 192e6, kKeepLinkBytes8 = 120e6;
enum OperatorReads { SHARED = 0, KEEP = 1, STREAM = 2 };
// The one-system FP16 MULT and D-hat instances are held to four waves per
// SIMD (128 VGPRs; they use about 103 with both hops' loads in flight, hop_dir).
// Five waves at 96 VGPRs helped the form with one hop's loads in flight
// (MULT 88.2 -> 85.5 us at 32^3x64), but with two hops' loads it spills and
// runs at 100.7 us; four waves with two hops' loads run at 83.9-84.7 us.
// The reconstruct-8 FP32 instances, with both hops' loads in flight, are held
// to four waves per SIMD in the same way (118-122 VGPRs).
template <int P, int MODE, int RED, int OPR, int LR>
constexpr int stencil_waves() {
    return ((P == P16 || (P == P32 && LR == 8)) && OPR != SHARED && (MODE == M_HOPINV || MODE == M_DHAT)) ? 4 : 1;
}
template <int P, int MODE, int RED, int OPR, int LR>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(stencil_waves<P, MODE, RED, OPR, LR>())))
void k_mult(MultBatch B) {
    using R = typename Real<P>::T;
    constexpr bool NT = OPR != SHARED, LNT = OPR == STREAM;  // clover, links
    int s, lb;
    batch_locate(B.h, xcd_block(blockIdx.x, gridDim.x, B.h.chunk), s, lb);
    const MultKArgs &a = B.d[s];
    if (a.done && *a.done) return;
    const int i = lb * (int)blockDim.x + threadIdx.x;  // 64, 128 or 256 sites per block
    const bool active = i < a.g.Vh;
    const int Vh = a.g.Vh;
    Spinor<R> out;
    // R_STEP's first operand, the centre vector (read once); the other operand
    // is loaded after the output is stored
    Spinor<R> ax;
    if (active) {
        Spinor<R> acc;
#pragma unroll
        for (int k = 0; k < 12; k++) acc.c[k] = {R(0), R(0)};
        if (MODE != M_CLOV) {
            const SiteCoord c = eo_coords(a.g, i, a.out_par);
            hop_dir<P, 0, LNT, LR>(a, c, i, acc);
            hop_dir<P, 1, LNT, LR>(a, c, i, acc);
            hop_dir<P, 2, LNT, LR>(a, c, i, acc);
            hop_dir<P, 3, LNT, LR>(a, c, i, acc);
        }
        const R coef = (R)a.coef;
        if (MODE == M_HOPINV) {
            clover_apply<P, R, NT>(a.clov, Vh, i, acc, out);
        } else if (MODE == M_DHAT) {
            Spinor<R> t;
            clover_apply<P, R, NT>(a.clov, Vh, i, acc, t);
            const Spinor<R> cen = SpinorIO<P>::template load<true>(a.center, Vh, i);
            if (RED == R_STEP) ax = cen;
#pragma unroll
            for (int k = 0; k < 12; k++) out.c[k] = cen.c[k] + coef * t.c[k];
        } else if (MODE == M_DFULL) {
            const Spinor<R> cen = SpinorIO<P>::template load<true>(a.center, Vh, i);
            clover_apply<P, R, NT>(a.clov, Vh, i, cen, out);
#pragma unroll
            for (int k = 0; k < 12; k++) out.c[k] = out.c[k] + coef * acc.c[k];
        } else if (MODE == M_INVSRC) {
            Spinor<R> s = SpinorIO<P>::template load<true>(a.center, Vh, i);
#pragma unroll
            for (int k = 0; k < 12; k++) s.c[k] = s.c[k] + coef * acc.c[k];
            clover_apply<P, R, NT>(a.clov, Vh, i, s, out);
        } else {  // M_CLOV
            const Spinor<R> cen = SpinorIO<P>::template load<true>(a.center, Vh, i);
            clover_apply<P, R, NT>(a.clov, Vh, i, cen, out);
        }
        SpinorIO<P>::template store<P == P64>(a.out, Vh, i, out);
    }
    if constexpr (RED != R_NONE) {
        constexpr int N = red_values(RED);
        double v[N];
#pragma unroll
        for (int k = 0; k < N; k++) v[k] = 0.0;
        if (active) {
            if (RED == R_STEP) {
                red_add<true, true, 12>(v, ax.c, out.c);
                as_stored<P>(out);
                red_add<true, false, 12>(v + 3, SpinorIO<P>::template load<true>(a.aux, Vh, i).c, out.c);
            } else {
                red_add<true, RED == R_DOTNORM, 12>(v, SpinorIO<P>::template load<true>(a.aux, Vh, i).c, out.c);
            }
        }
        block_partials<N>(v, a.red.partials, a.nblk, lb);
    }
}

// ---------------------------------------------------------------------------
// The one-system stencil with a tile's four directions on four wavefronts.
// k_mult gives a site to one thread: eight hops one after the other, each
// waiting for its neighbour.  On a lattice of a few tiles per compute unit
// nothing else runs meanwhile, and a launch costs that chain of latencies.
// Here a workgroup takes one 64-site tile: wavefront mu adds both hops of
// direction mu, with the loads of both in flight, the four partial sums meet in
// LDS, and two wavefronts apply one chiral clover block each (loaded before the
// hops) and store one half of the spinor.
// It also pays on large lattices: four wavefronts on 64 sites instead of 256
// keep a quarter of the neighbourhood in flight, and more of it stays in L2.
// D-hat_ee, k_mult -> k_mult_split, us: FP64 12x14x10x18 34.8 -> 17.6, 24^3x48
// 266 -> 242, 48^3x96 4029 -> 3891; FP32 24^3x48 119 -> 107 (5.7 TB/s), 32^3x64
// 326 -> 315, 48^3x96 1843 -> 1772; full links 141 -> 128, 397 -> 384, 2151 ->
// 2112.  Which lattices take it: split_stencil.
//
// D on canonical fields (M_DCANON) moves memory too, and its two parities read
// the same links: as two launches and an unpack it fetched them twice and the
// result made a round trip through the tiled layout.  One launch with the
// parities' tiles interleaved meets the links in L2 and writes the result where
// the caller wants it.  The whole call, pack included, us: FP64 8^4 20 -> 14,
// 20x12x28x36 140 -> 99, 32^3x64 1140 -> 825; FP32 82 -> 63, 638 -> 540 at the
// larger two.
// ---------------------------------------------------------------------------
constexpr int kSplitWaves = 4;
constexpr int kSplitBlock = -64;  // "block size" that selects it: 64 sites per workgroup

// the upper (h = 0) or lower (h = 1) two spin components of a stored spinor
template <int P, bool NT>
__device__ __forceinline__ void half_load(const void *base, int i, int h, cx<typename Real<P>::T> (&o)[6]) {
    if constexpr (P == P64) {
#pragma unroll
        for (int k = 0; k < 6; k++) {
            const double2 v = ld_op<NT>(tp<double2, 192>(base, i, 16 * (6 * h + k)));
            o[k] = {v.x, v.y};
        }
    } else if constexpr (P == P32) {
#pragma unroll
        for (int k = 0; k < 3; k++) {
            const float4 v = ld_op<NT>(tp<float4, 96>(base, i, 16 * (3 * h + k)));
            o[2 * k] = {v.x, v.y};
            o[2 * k + 1] = {v.z, v.w};
        }
    } else {
        // components 0-3 | 4-7 | 8-11 per plane: the middle plane is shared
        const float s = ld_op<NT>(tp<float, 52>(base, i, 48));
        const uint4 a = ld_op<NT>(tp<uint4, 52>(base, i, 32 * h));
        const uint4 m = ld_op<NT>(tp<uint4, 52>(base, i, 16));
        const uint32_t w[6] = {h ? m.z : a.x, h ? m.w : a.y, h ? a.x : a.z, h ? a.y : a.w, h ? a.z : m.x, h ? a.w : m.y};
#pragma unroll
        for (int k = 0; k < 6; k++) {
            const float2 v = h2f(w[k]);
            o[k] = {s * v.x, s * v.y};
        }
    }
}

// m: FP16's site scale, the largest magnitude of all 24 reals
template <int P>
__device__ __forceinline__ void half_store(void *base, int i, int h, const cx<typename Real<P>::T> (&v)[6], float m) {
    if constexpr (P == P64) {
#pragma unroll
        for (int k = 0; k < 6; k++)
            st_op<true>(tp<double2, 192>(base, i, 16 * (6 * h + k)), make_double2(v[k].re, v[k].im));
    } else if constexpr (P == P32) {
#pragma unroll
        for (int k = 0; k < 3; k++)
            *tp<float4, 96>(base, i, 16 * (3 * h + k)) = make_float4(v[2 * k].re, v[2 * k].im, v[2 * k + 1].re, v[2 * k + 1].im);
    } else {
        const float inv = m > 0.f ? 1.0f / m : 0.f;
        uint32_t w[6];
#pragma unroll
        for (int k = 0; k < 6; k++) w[k] = f2h(v[k].re * inv, v[k].im * inv);
        uint2 *mid = (uint2 *)tp<uint4, 52>(base, i, 16);
        if (h == 0) {
            *tp<uint4, 52>(base, i, 0) = make_uint4(w[0], w[1], w[2], w[3]);
            mid[0] = make_uint2(w[4], w[5]);
            *tp<float, 52>(base, i, 48) = m;
        } else {
            mid[1] = make_uint2(w[0], w[1]);
            *tp<uint4, 52>(base, i, 32) = make_uint4(w[2], w[3], w[4], w[5]);
        }
    }
}

// Held to the waves per SIMD that the loads of a direction leave registers for
// (the reductions alone would cost the FP32 D-hat half its fourth wave).
template <int P, int MODE, int LR> constexpr int split_waves() {
    return P == P64 ? 2 : (LR == 8 || MODE == M_DFULL || MODE == M_DCANON || MODE == M_INVSRC) ? 3 : 4;
}
template <int P, int MODE, int RED, int OPR, int LR>
__global__ __launch_bounds__(64 * kSplitWaves) __attribute__((amdgpu_waves_per_eu(split_waves<P, MODE, LR>())))
void k_mult_split(MultBatch B) {
    using R = typename Real<P>::T;
    alignas(16) __shared__ cx<R> part[kSplitWaves][12][64];  // M_DCANON: sites of double2 as well
    __shared__ cx<R> yb[2][6][64];
    __shared__ float mx[2][64];
    int s, lb;
    batch_locate(B.h, xcd_block(blockIdx.x, gridDim.x, B.h.chunk), s, lb);
    const MultKArgs &a = B.d[s];
    if (a.done && *a.done) return;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int i = lb * 64 + lane;
    const bool active = i < a.g.Vh;
    const bool site = active && w < 2;  // wavefronts 0 and 1 finish the sites
    const int Vh = a.g.Vh;
    constexpr bool CEN = MODE != M_HOPINV;
    constexpr bool FULL = MODE == M_DFULL || MODE == M_DCANON;
    constexpr bool LNT = OPR == STREAM;
    // the clover block b acts on up - dn (0) or up + dn (1)
    Herm6<R> M;
    R cs = R(1);
    cx<R> cen[6], oth[6];  // the centre's own half and, where the clover takes the centre, the other half
    if (site) {
        if constexpr (P == P16) {
            M = CloverIO<P16>::template load_scaled<true>(a.clov, Vh, i, w, 1.0f);
            cs = CloverIO<P16>::scale(a.clov, i);
        } else {
            M = CloverIO<P>::template load<true>(a.clov, Vh, i, w);
        }
        // (both wavefronts read the whole centre here, through the cache)
        if constexpr (FULL || MODE == M_INVSRC) half_load<P, false>(a.center, i, 1 - w, oth);
    }
    // wavefronts 2 and 3 hold a half of the fused dot's operand in its place
    if constexpr (CEN) {
        if (RED != R_NONE ? active : site)
            half_load<P, MODE == M_DHAT>(RED != R_NONE && w >= 2 ? a.aux : a.center, i, w & 1, cen);
    }
    {
        Spinor<R> acc;
#pragma unroll
        for (int k = 0; k < 12; k++) acc.c[k] = {R(0), R(0)};
        if (active) {
            const SiteCoord c = eo_coords(a.g, i, a.out_par);
            switch (w) {
            case 0: hop_dir<P, 0, LNT, LR>(a, c, i, acc); break;
            case 1: hop_dir<P, 1, LNT, LR>(a, c, i, acc); break;
            case 2: hop_dir<P, 2, LNT, LR>(a, c, i, acc); break;
            default: hop_dir<P, 3, LNT, LR>(a, c, i, acc); break;
            }
        }
#pragma unroll
        for (int k = 0; k < 12; k++) part[w][k][lane] = acc.c[k];
    }
    __syncthreads();
    const R coef = (R)a.coef;
    cx<R> own[6];  // the hopping sum's own half (FULL)
    if (site) {
        cx<R> v[6], y[6];
#pragma unroll
        for (int k = 0; k < 6; k++) {
            cx<R> h[2];  // upper, lower
#pragma unroll
            for (int q = 0; q < 2; q++)
                h[q] = (part[0][6 * q + k][lane] + part[1][6 * q + k][lane]) +
                       (part[2][6 * q + k][lane] + part[3][6 * q + k][lane]);
            if (FULL) {
                own[k] = w ? h[1] : h[0];
                h[0] = w ? oth[k] : cen[k];
                h[1] = w ? cen[k] : oth[k];
            } else if (MODE == M_INVSRC) {
                h[0] = (w ? oth[k] : cen[k]) + coef * h[0];
                h[1] = (w ? cen[k] : oth[k]) + coef * h[1];
            }
            v[k] = w ? h[0] + h[1] : h[0] - h[1];
        }
        herm6_apply(M, v, y);
#pragma unroll
        for (int k = 0; k < 6; k++) yb[w][k][lane] = y[k];
    }
    __syncthreads();
    cx<R> out[6];
    if (site) {
#pragma unroll
        for (int k = 0; k < 6; k++) {
            const cx<R> ym = yb[0][k][lane], yp = yb[1][k][lane];
            cx<R> t = w ? yp - ym : yp + ym;
            if (P == P16) t = cs * t;
            if (MODE == M_DHAT) t = cen[k] + coef * t;
            if (FULL) t = t + coef * own[k];
            out[k] = t;
        }
    }
    float m = 0.f;
    if constexpr (P == P16) {
        if (site) {
#pragma unroll
            for (int k = 0; k < 6; k++) m = fmaxf(m, fmaxf(fabsf(out[k].re), fabsf(out[k].im)));
            mx[w][lane] = m;
        }
        __syncthreads();
        if (site) m = fmaxf(m, mx[1 - w][lane]);
    }
    if constexpr (MODE == M_DCANON) {
        // through LDS, so that the canonical sites leave as whole 192-byte pieces
        double2(*st)[13] = reinterpret_cast<double2(*)[13]>(part);  // 13: as kPadSpin in layout.hip
        static_assert(sizeof(part) >= 64 * sizeof(*st), "the sites of a tile fit the hops' sums");
        if (site) {
#pragma unroll
            for (int k = 0; k < 6; k++) st[lane][6 * w + k] = make_double2((double)out[k].re, (double)out[k].im);
        }
        __syncthreads();
        const int live = min(64, Vh - lb * 64) * 12;
        for (int e = threadIdx.x; e < live; e += 64 * kSplitWaves) {
            const int q = e / 12;
            const SiteCoord c = eo_coords(a.g, lb * 64 + q, a.out_par);
            st_stream((double2 *)a.out + (size_t)(c.x + a.g.L[0] * c.row) * 12 + (e - 12 * q), st[q][e - 12 * q]);
        }
    } else {
        if (site) half_store<P>(a.out, i, w, out, m);
    }
    if constexpr (RED != R_NONE) {
        // wavefronts 0 and 1 sum what they hold, 2 and 3 the dot with the
        // operand they loaded
        constexpr int N = red_values(RED);
        double v[N];
#pragma unroll
        for (int k = 0; k < N; k++) v[k] = 0.0;
        // (left to itself the compiler widens the operand to FP64 where it is
        // loaded, and the hops lose the registers)
#pragma unroll
        for (int k = 0; k < 6; k++) keep(cen[k]);
        if (site) {
#pragma unroll
            for (int k = 0; k < 6; k++) {
                if constexpr (P == P16 && RED == R_STEP) part[w][k][lane] = stored16(out[k], m, m > 0.f ? 1.0f / m : 0.f);
                else part[w][k][lane] = out[k];
            }
            red_add<RED == R_STEP, RED != R_DOT, 6>(v, cen, out);
        }
        __syncthreads();
        if (active && w >= 2) {
            cx<R> o[6];
#pragma unroll
            for (int k = 0; k < 6; k++) o[k] = part[w - 2][k][lane];
            red_add<true, false, 6>(RED == R_STEP ? v + 3 : v, cen, o);
        }
        block_partials<N>(v, a.red.partials, a.nblk, lb);
    }
}

// lds: dynamic LDS bytes that cap the workgroups per CU of the one-system
// instances; the kernels use none of it
template <int P, int MODE, int RED, int OPR, int LR>
void launch_as(const MultBatch &B, int blocks, int bs, unsigned lds, hipStream_t s) {
    if constexpr (MODE == M_DCANON || (OPR != SHARED && MODE != M_CLOV && (MODE != M_DFULL || P == P64))) {
        if (MODE == M_DCANON || bs == kSplitBlock) {
            // the cap counts the kernel's own LDS
            constexpr unsigned own = sizeof(cx<typename Real<P>::T>) * 64 * (12 * kSplitWaves + 12);
            const unsigned dyn = lds > own ? lds - own : 0;
            hipLaunchKernelGGL((k_mult_split<P, MODE, RED, OPR, LR>), dim3(blocks), dim3(64 * kSplitWaves), dyn, s, B);
            return;
        }
    }
    if constexpr (MODE != M_DCANON)
        hipLaunchKernelGGL((k_mult<P, MODE, RED, OPR, LR>), dim3(blocks), dim3(bs), lds, s, B);
}

template <int P, int MODE, int RED, int LR>
void launch_nt(const MultBatch &B, int blocks, int bs, unsigned lds, hipStream_t s, bool keep) {
    if (MODE == M_DCANON || B.h.interleave) return launch_as<P, MODE, RED, SHARED, LR>(B, blocks, bs, lds, s);
    if constexpr (MODE == M_HOPINV || MODE == M_DHAT) {
        if (keep) return launch_as<P, MODE, RED, KEEP, LR>(B, blocks, bs, lds, s);
    }
    if constexpr (MODE != M_DCANON) launch_as<P, MODE, RED, STREAM, LR>(B, blocks, bs, lds, s);
}

// reconstruct-8 and full-link instances exist for the FP32 stencil only
template <int P, int MODE, int RED>
void launch_one(const MultBatch &B, int blocks, int bs, unsigned lds, hipStream_t s, int lr, bool keep) {
    if constexpr (P == P32) {
        if (lr == 8) {
            launch_nt<P, MODE, RED, 8>(B, blocks, bs, lds, s, keep);
            return;
        }
        if (lr == 18) {
            launch_nt<P, MODE, RED, 18>(B, blocks, bs, lds, s, keep);
            return;
        }
    }
    launch_nt<P, MODE, RED, 12>(B, blocks, bs, lds, s, keep);
}

template <int P>
void dispatch_mode(const MultBatch &B, int mode, int red, int blocks, int bs, unsigned lds, hipStream_t s, int lr, bool keep) {
    switch (mode) {
    case M_HOPINV: launch_one<P, M_HOPINV, R_NONE>(B, blocks, bs, lds, s, lr, keep); break;
    case M_DHAT:
        if (red == R_DOT) launch_one<P, M_DHAT, R_DOT>(B, blocks, bs, lds, s, lr, keep);
        else if (red == R_STEP) launch_one<P, M_DHAT, R_STEP>(B, blocks, bs, lds, s, lr, keep);
        else if (red == R_DOTNORM) {
            if constexpr (P == P64) launch_one<P, M_DHAT, R_DOTNORM>(B, blocks, bs, lds, s, lr, keep);  // outer loop only
        } else launch_one<P, M_DHAT, R_NONE>(B, blocks, bs, lds, s, lr, keep);
        break;
    case M_DFULL: launch_one<P, M_DFULL, R_NONE>(B, blocks, bs, lds, s, lr, keep); break;
    case M_DCANON:
        if constexpr (P != P16) launch_one<P, M_DCANON, R_NONE>(B, blocks, bs, lds, s, lr, keep);
        break;
    case M_INVSRC: launch_one<P, M_INVSRC, R_NONE>(B, blocks, bs, lds, s, lr, keep); break;
    case M_CLOV: launch_one<P, M_CLOV, R_NONE>(B, blocks, bs, lds, s, lr, keep); break;
    }
}

// algorithmic bytes of one call (per output site: inputs and outputs at the
// stored precision, each link once, one clover pair).  The spinor part is per
// call; the link and clover part is per lattice, since calls of one batch on
// the same lattice read the same operator.
double mult_spinor_bytes(int prec, int mode, int red, int Vh) {
    const double S = (double)spinor_site_bytes(prec) * Vh;
    double b = 2 * S;                                                    // input (once) + output
    if (mode == M_DHAT || mode == M_DFULL || mode == M_INVSRC) b += S;  // centre vector
    if (mode == M_DCANON) b += (double)spinor_site_bytes(P64) * Vh;     // centre, and a complex128 output
    if (red != R_NONE) b += S;                                           // aux vector
    return b;
}
int link_bytes_per_site(int prec, int lr) { return lr == 8 ? 32 : lr == 18 ? 72 : link_site_bytes(prec); }
double mult_operator_bytes(int prec, int mode, int lr, int Vh) {
    double b = 0;
    if (mode != M_CLOV) b += 8 * (double)link_bytes_per_site(prec, lr) * Vh;
    b += (mode == M_DCANON ? 2 : 1) * (double)clover_site_bytes(prec) * Vh;  // M_DCANON: both parities'
    return b;
}


// ---------------------------------------------------------------------------
// Several right-hand sides on one lattice (many solutions per gauge field,
// Sec. II-A), in two forms.
//
// k_mult_multi: a workgroup of two wavefronts takes a 64-site tile (or, where
// tiles alone would leave compute units idle, a tile and some of the systems)
// and goes through its systems one after the other.  Wavefront 0 holds the links
// of the x and y hops, wavefront 1 those of z and t, each also one chiral clover
// block: the operator is read and rebuilt once for all systems and stays in
// registers.  Per system the two exchange half sums through LDS, apply their
// block and store one half of the spinor.  Many fields are bound by what the L2
// must fetch: their neighbourhoods do not fit it together.  Here a workgroup has
// one system in flight, all workgroups of an XCD go through the systems in step,
// and the L2 holds one system's neighbourhood at a time: for 12 fields at
// 32^3x64 it fetches 3.5 GB a MULT, where one wavefront per pair of systems
// fetched 4.5.  The four neighbours are loaded plane by plane, so that those
// along x and y find each other's lines in L1 (24% fewer L2 requests).  FP32,
// us before -> now, MULT | D-hat_ee: 12 fields 16^3x32 72 -> 53 | 160 -> 116,
// 24^3x48 351 -> 295 | 746 -> 622, 32^3x64 1012 -> 846 | 2178 -> 1786; 2 fields
// 32^3x64 314 -> 231 | 657 -> 490.  Loading the next system's neighbours ahead,
// with the clover blocks in LDS, was slower: 895 us for the 32^3x64 MULT, since
// two systems in flight fetch 5.0 GB.
//
// k_mult_mrhs: one thread takes one output site for G systems at once and applies
// each link and clover block, loaded once, to all G.  A wavefront covers the 64
// sites of one tile for one group of G systems, the waves of all groups of a tile
// form one workgroup.  It remains where it is the faster one (multi_by_tile).
// ---------------------------------------------------------------------------
struct MrhsSys {
    void *out;
    const void *in;
    const void *center;
    const void *aux;
    double *partials;  // [N][ntiles] of this system
    const int *done;
};

struct MrhsArgs {
    Geom g;
    int out_par;
    const char *links;
    size_t link_slab;
    const void *clov;
    double coef;
    int nsys;     // systems of the launch
    int ngroups;  // groups of systems (k_mult_mrhs: of G systems, ceil(nsys / G))
    int ntiles;   // 64-site tiles of one parity
    int chunk;    // workgroups per XCD chunk of the block remap (0: one slab per XCD)
    bool loop;    // MultCall::loop
    MrhsSys s[kMaxSys];
};

// one stored 6x6 block; FP16 blocks without their site scale
template <int P>
__device__ __forceinline__ Herm6<typename Real<P>::T> clover_block(const void *slab, int Vh, int i, int b) {
    if constexpr (P == P16) return CloverIO<P16>::template load_scaled<false>(slab, Vh, i, b, 1.0f);
    else return CloverIO<P>::template load<false>(slab, Vh, i, b);
}

// out_j = M_blk(w_j) applied blockwise as in clover_apply, for G spinors, each
// 6x6 block loaded once: on entry acc[j] holds the hopping sum, on exit the
// clover result
template <int P, int G, class R>
__device__ __forceinline__ void clover_apply_multi(const void *slab, int Vh, int i, Spinor<R> (&acc)[G],
                                                   const bool (&live)[G]) {
    // acc.up <- wp = up + dn, acc.dn <- M1 (up - dn)
    {
        const Herm6<R> M1 = clover_block<P>(slab, Vh, i, 0);
#pragma unroll
        for (int j = 0; j < G; j++) {
            if (!live[j]) continue;
            cx<R> wm[6], ym[6];
#pragma unroll
            for (int k = 0; k < 6; k++) {
                wm[k] = acc[j].c[k] - acc[j].c[k + 6];
                acc[j].c[k] = acc[j].c[k] + acc[j].c[k + 6];
            }
            herm6_apply(M1, wm, ym);
#pragma unroll
            for (int k = 0; k < 6; k++) acc[j].c[k + 6] = ym[k];
        }
    }
    const Herm6<R> M2 = clover_block<P>(slab, Vh, i, 1);
    R s = R(1);
    if constexpr (P == P16) s = CloverIO<P16>::scale(slab, i);
#pragma unroll
    for (int j = 0; j < G; j++) {
        if (!live[j]) continue;
        cx<R> yp[6];
        herm6_apply(M2, acc[j].c, yp);
#pragma unroll
        for (int k = 0; k < 6; k++) {
            const cx<R> ym = acc[j].c[k + 6];
            acc[j].c[k] = s * (yp[k] + ym);
            acc[j].c[k + 6] = s * (yp[k] - ym);
        }
    }
}

template <int P, int MU, int LR, int G>
__device__ __forceinline__ void hop_dir_multi(const MrhsArgs &A, const SiteCoord &c, int i, int q,
                                              Spinor<typename Real<P>::T> (&acc)[G], const bool (&live)[G]) {
    using R = typename Real<P>::T;
    const int Vh = A.g.Vh;
    {
        const int nf = eo_neighbour(A.g, c, MU, +1);
        const Mat3<R> U = LinkLoad<P, LR>::template load<false>(A.links + (size_t)(2 * MU + A.out_par) * A.link_slab, Vh, i);
#pragma unroll
        for (int j = 0; j < G; j++)
            if (live[j]) hop_one<P, MU, true>(A.s[q * G + j].in, Vh, nf, U, acc[j]);
    }
    {
        const int nb = eo_neighbour(A.g, c, MU, -1);
        const Mat3<R> U =
            LinkLoad<P, LR>::template load<false>(A.links + (size_t)(2 * MU + 1 - A.out_par) * A.link_slab, Vh, nb);
#pragma unroll
        for (int j = 0; j < G; j++)
            if (live[j]) hop_one<P, MU, false>(A.s[q * G + j].in, Vh, nb, U, acc[j]);
    }
}

// One workgroup per 64-site tile, one wavefront per group of G systems, so the
// waves that share a tile's links and clover blocks run on one compute unit;
// the tiles are handed to the XCDs in the lattice's chunks, as for the
// one-system stencil.
constexpr int kMrhsMaxGroups = 8;  // 16 systems at 2 per thread
template <int P, int MODE, int RED, int LR, int G>
__global__ __launch_bounds__(64 * kMrhsMaxGroups) void k_mult_mrhs(MrhsArgs A) {
    using R = typename Real<P>::T;
    const int tile = xcd_block(blockIdx.x, gridDim.x, A.chunk);
    const int q = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));  // uniform across the wave
    if (tile >= A.ntiles || q >= A.ngroups) return;  // whole waves only
    bool live[G];
    bool any = false;
#pragma unroll
    for (int j = 0; j < G; j++) {
        const int s = q * G + j;
        live[j] = s < A.nsys && !(A.s[s].done && *A.s[s].done);
        any = any || live[j];
    }
    if (!any) return;  // every system of this wave has stopped
    const int Vh = A.g.Vh;
    const int i = tile * 64 + (int)(threadIdx.x & 63);
    const bool active = i < Vh;
    constexpr int NR = RED == R_NONE ? 1 : red_values(RED);  // values of the fused reduction
    double red[G][NR];
#pragma unroll
    for (int j = 0; j < G; j++)
#pragma unroll
        for (int k = 0; k < NR; k++) red[j][k] = 0.0;
    Spinor<R> acc[G];
#pragma unroll
    for (int j = 0; j < G; j++)
#pragma unroll
        for (int k = 0; k < 12; k++) acc[j].c[k] = {R(0), R(0)};
    if (active) {
        const SiteCoord c = eo_coords(A.g, i, A.out_par);
        hop_dir_multi<P, 0, LR, G>(A, c, i, q, acc, live);
        hop_dir_multi<P, 1, LR, G>(A, c, i, q, acc, live);
        hop_dir_multi<P, 2, LR, G>(A, c, i, q, acc, live);
        hop_dir_multi<P, 3, LR, G>(A, c, i, q, acc, live);
        clover_apply_multi<P, G>(A.clov, Vh, i, acc, live);
        const R coef = (R)A.coef;
#pragma unroll
        for (int j = 0; j < G; j++) {
            if (!live[j]) continue;
            const MrhsSys &S = A.s[q * G + j];
            if (MODE == M_DHAT) {
                // the centre, and the reduction's operand beside it
                const Spinor<R> cen = SpinorIO<P>::template load<true>(S.center, Vh, i);
                Spinor<R> ax;
                if (RED != R_NONE) ax = SpinorIO<P>::template load<true>(S.aux, Vh, i);
#pragma unroll
                for (int k = 0; k < 12; k++) acc[j].c[k] = cen.c[k] + coef * acc[j].c[k];
                SpinorIO<P>::template store<false>(S.out, Vh, i, acc[j]);
                if (RED == R_DOT) red_add<true, false, 12>(red[j], ax.c, acc[j].c);
                if (RED == R_STEP) {
                    red_add<true, true, 12>(red[j], cen.c, acc[j].c);
                    as_stored<P>(acc[j]);
                    red_add<true, false, 12>(red[j] + 3, ax.c, acc[j].c);
                }
            } else {
                SpinorIO<P>::template store<false>(S.out, Vh, i, acc[j]);
            }
        }
    }
    if (RED != R_NONE) {
#pragma unroll
        for (int j = 0; j < G; j++) {
            if (!live[j]) continue;
            wave_fold<NR>(red[j]);
            if ((threadIdx.x & 63) == 0) {
                double *part = A.s[q * G + j].partials;
#pragma unroll
                for (int k = 0; k < NR; k++) part[(size_t)k * A.ntiles + tile] = red[j][k];
            }
        }
    }
}

// both links of direction MU at a site, and the two neighbours
template <int P, int MU, int LR>
__device__ __forceinline__ void load_dir(const MrhsArgs &A, const SiteCoord &c, int i, Mat3<typename Real<P>::T> *U,
                                         int *n) {
    const int Vh = A.g.Vh;
    n[0] = eo_neighbour(A.g, c, MU, +1);
    n[1] = eo_neighbour(A.g, c, MU, -1);
    U[0] = LinkLoad<P, LR>::template load<true>(A.links + (size_t)(2 * MU + A.out_par) * A.link_slab, Vh, i);
    U[1] = LinkLoad<P, LR>::template load<true>(A.links + (size_t)(2 * MU + 1 - A.out_par) * A.link_slab, Vh, n[1]);
}

// a neighbour's spinor as it is stored
template <int P> struct RawSpinor {
    float4 v[6];
};
template <> struct RawSpinor<P16> {
    uint4 v[3];
    float s;
};
// four neighbours, plane by plane: those along x and y lie in the same lines
template <int P> __device__ __forceinline__ void raw_load4(RawSpinor<P> (&r)[4], const void *in, const int (&n)[4]) {
    if constexpr (P == P16) {
#pragma unroll
        for (int k = 0; k < 3; k++)
#pragma unroll
            for (int j = 0; j < 4; j++) r[j].v[k] = *tp<uint4, 52>(in, n[j], 16 * k);
#pragma unroll
        for (int j = 0; j < 4; j++) r[j].s = *tp<float, 52>(in, n[j], 48);
    } else {
#pragma unroll
        for (int k = 0; k < 6; k++)
#pragma unroll
            for (int j = 0; j < 4; j++) r[j].v[k] = *tp<float4, 96>(in, n[j], 16 * k);
    }
}
template <int P, int MU, bool FWD>
__device__ __forceinline__ void raw_hop(const RawSpinor<P> &r, const Mat3<float> &U, Spinor<float> &acc) {
    if constexpr (P == P16) {
        hop_term<float, MU, FWD, true>(SpinorIO<P16>::decode(r.v), U, acc, r.s);
    } else {
        Spinor<float> p;
#pragma unroll
        for (int k = 0; k < 6; k++) {
            p.c[2 * k] = {r.v[k].x, r.v[k].y};
            p.c[2 * k + 1] = {r.v[k].z, r.v[k].w};
        }
        hop_term<float, MU, FWD, false>(p, U, acc, 1.0f);
    }
}

constexpr int kMultiWaves = 2;

// a clover block put away in LDS, and read back
__device__ __forceinline__ void park(float4 (*p)[64], int lane, const Herm6<float> &M) {
    p[0][lane] = make_float4(M.d[0], M.d[1], M.d[2], M.d[3]);
    p[1][lane] = make_float4(M.d[4], M.d[5], M.o[0].re, M.o[0].im);
#pragma unroll
    for (int k = 0; k < 7; k++)
        p[2 + k][lane] = make_float4(M.o[1 + 2 * k].re, M.o[1 + 2 * k].im, M.o[2 + 2 * k].re, M.o[2 + 2 * k].im);
}
__device__ __forceinline__ Herm6<float> unpark(const float4 (*p)[64], int lane) {
    Herm6<float> M;
    const float4 a = p[0][lane], b = p[1][lane];
    M.d[0] = a.x;
    M.d[1] = a.y;
    M.d[2] = a.z;
    M.d[3] = a.w;
    M.d[4] = b.x;
    M.d[5] = b.y;
    M.o[0] = {b.z, b.w};
#pragma unroll
    for (int k = 0; k < 7; k++) {
        const float4 f = p[2 + k][lane];
        M.o[1 + 2 * k] = {f.x, f.y};
        M.o[2 + 2 * k] = {f.z, f.w};
    }
    return M;
}

// Two wavefronts per SIMD: a wavefront keeps 72 registers of links, 36 of clover
// block and four neighbours in flight.
template <int P, int MODE, int RED, int LR>
__global__ __launch_bounds__(64 * kMultiWaves) __attribute__((amdgpu_waves_per_eu(2))) void k_mult_multi(MrhsArgs A) {
    using R = typename Real<P>::T;
    constexpr int NR = RED == R_NONE ? 1 : red_values(RED);
    __shared__ cx<R> xch[2][6][64], ych[2][6][64];
    __shared__ float mx[2][64];
    __shared__ double rs[2][kMaxSys][NR];
    // with a reduction the registers do not hold the clover block as well: it
    // waits in LDS between the systems
    constexpr bool kParkM = P == P32 && RED != R_NONE;
    __shared__ float4 parked[2][kParkM ? 9 : 1][64];
    const int L = xcd_block(blockIdx.x, gridDim.x, A.chunk);
    const int tile = L / A.ngroups, grp = L - tile * A.ngroups;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    // the systems of this group that still run
    const int s0 = grp * A.nsys / A.ngroups, s1 = (grp + 1) * A.nsys / A.ngroups;
    unsigned live = 0;
    {
        // (every flag is read before the first is looked at)
        int flag[kMaxSys];
#pragma unroll
        for (int s = 0; s < kMaxSys; s++) {
            const int *d = A.s[s < A.nsys ? s : 0].done;
            flag[s] = *(d ? d : (const int *)A.links);
        }
#pragma unroll
        for (int s = 0; s < kMaxSys; s++)
            if (s >= s0 && s < s1 && !(A.s[s].done && flag[s])) live |= 1u << s;
    }
    if (!live) return;
    const int Vh = A.g.Vh;
    const int i = tile * 64 + lane;
    const bool active = i < Vh;
    Herm6<R> M;
    Mat3<R> U[4];
    int n[4] = {0, 0, 0, 0};
    R cs = R(1);
    if (active) {
        const SiteCoord c = eo_coords(A.g, i, A.out_par);
        if (w == 0) {
            load_dir<P, 0, LR>(A, c, i, U, n);
            load_dir<P, 1, LR>(A, c, i, U + 2, n + 2);
        } else {
            load_dir<P, 2, LR>(A, c, i, U, n);
            load_dir<P, 3, LR>(A, c, i, U + 2, n + 2);
        }
        if constexpr (P == P16) {
            M = CloverIO<P16>::template load_scaled<true>(A.clov, Vh, i, w, 1.0f);
            cs = CloverIO<P16>::scale(A.clov, i);
        } else {
            M = CloverIO<P>::template load<true>(A.clov, Vh, i, w);
        }
    }
    if constexpr (kParkM) {
        if (active) park(parked[w], lane, M);
    }
    const R coef = (R)A.coef;
    for (unsigned todo = live; todo;) {
        const int s = __builtin_ctz(todo);
        todo &= todo - 1;
        const MrhsSys &S = A.s[s];
        cx<R> cen[6], ax[6], v[6], out[6];
        if (active) {
            Spinor<R> acc;
#pragma unroll
            for (int k = 0; k < 12; k++) acc.c[k] = {R(0), R(0)};
            RawSpinor<P> psi[4];
            raw_load4<P>(psi, S.in, n);
            if (w == 0) {
                raw_hop<P, 0, true>(psi[0], U[0], acc);
                raw_hop<P, 0, false>(psi[1], U[1], acc);
                raw_hop<P, 1, true>(psi[2], U[2], acc);
                raw_hop<P, 1, false>(psi[3], U[3], acc);
            } else {
                raw_hop<P, 2, true>(psi[0], U[0], acc);
                raw_hop<P, 2, false>(psi[1], U[1], acc);
                raw_hop<P, 3, true>(psi[2], U[2], acc);
                raw_hop<P, 3, false>(psi[3], U[3], acc);
            }
            if constexpr (MODE == M_DHAT) {
                half_load<P, true>(S.center, i, w, cen);
                if constexpr (RED != R_NONE) half_load<P, true>(S.aux, i, w, ax);
            }
#pragma unroll
            for (int k = 0; k < 6; k++) {
                const cx<R> m = acc.c[k] - acc.c[k + 6], q = acc.c[k] + acc.c[k + 6];
                v[k] = w ? q : m;
                xch[w][k][lane] = w ? m : q;
            }
        }
        __syncthreads();
        if (active) {
            cx<R> y[6];
#pragma unroll
            for (int k = 0; k < 6; k++) v[k] = v[k] + xch[1 - w][k][lane];
            if constexpr (kParkM) M = unpark(parked[w], lane);
            herm6_apply(M, v, y);
#pragma unroll
            for (int k = 0; k < 6; k++) {
                v[k] = y[k];
                ych[w][k][lane] = y[k];
            }
        }
        __syncthreads();
        if (active) {
#pragma unroll
            for (int k = 0; k < 6; k++) {
                const cx<R> o = ych[1 - w][k][lane];
                cx<R> t = w ? v[k] - o : o + v[k];  // yp - ym, yp + ym
                if (P == P16) t = cs * t;
                if (MODE == M_DHAT) t = cen[k] + coef * t;
                out[k] = t;
            }
        }
        float m = 0.f;
        if constexpr (P == P16) {
            if (active) {
#pragma unroll
                for (int k = 0; k < 6; k++) m = fmaxf(m, fmaxf(fabsf(out[k].re), fabsf(out[k].im)));
                mx[w][lane] = m;
            }
            __syncthreads();
            if (active) m = fmaxf(m, mx[1 - w][lane]);
        }
        if (active) half_store<P>(S.out, i, w, out, m);
        if constexpr (RED != R_NONE) {
            double r[NR];
#pragma unroll
            for (int k = 0; k < NR; k++) r[k] = 0.0;
            if (active) {
#pragma unroll
                for (int k = 0; k < 6; k++) {
                    keep(cen[k]);
                    keep(ax[k]);
                }
                if (RED == R_STEP) {
                    red_add<true, true, 6>(r, cen, out);
                    if constexpr (P == P16) {
#pragma unroll
                        for (int k = 0; k < 6; k++) out[k] = stored16(out[k], m, m > 0.f ? 1.0f / m : 0.f);
                    }
                    red_add<true, false, 6>(r + 3, ax, out);
                } else {
                    red_add<true, false, 6>(r, ax, out);
                }
            }
            wave_fold<NR>(r);
            if (lane == 0) {
#pragma unroll
                for (int k = 0; k < NR; k++) rs[w][s][k] = r[k];
            }
        }
    }
    if constexpr (RED != R_NONE) {
        __syncthreads();
        for (int t = threadIdx.x; t < kMaxSys * NR; t += 64 * kMultiWaves) {
            const int s = t / NR, k = t - s * NR;
            if (live >> s & 1) A.s[s].partials[(size_t)k * A.ntiles + tile] = rs[0][s][k] + rs[1][s][k];
        }
    }
}

// Which form a launch takes.  1024 workgroups of k_mult_multi fit the device at
// once, so its time grows in steps of 1024 tiles, and below 1024 it is that of its
// longest workgroup; the workgroups of k_mult_mrhs are smaller and finish more
// evenly.  D-hat_ee, us, k_mult_mrhs -> k_mult_multi:
//   FP32: k_mult_multi is up to 1.5 times faster (2592 tiles: 3 fields 164 -> 108,
//   12 fields 399 -> 331), except for 2 fields, one wavefront a tile, in its second
//   round and a little beyond (1152 tiles 43 -> 48, 1732 57 -> 63, 2079 73 -> 76, but 1008
//   43 -> 35, 2376 82 -> 83, 2592 103 -> 89), for 4 fields just beyond 1024 tiles
//   (1152 63 -> 70, but 1408 faster), and for 4, 6 or 8 fields just beyond 512, from where on a workgroup takes all fields (640 tiles,
//   8 fields 62 -> 65, but 7 fields at 704 66 -> 60 and 8 at 768 no slower).
//   FP16, half the bytes and more arithmetic, needs full rounds: 384 tiles 12 | 16
//   fields 64 -> 60 | 66 -> 74, 512 tiles 12 | 16 fields 64 -> 62 | 72 -> 78, 640 tiles
//   6 | 8 | 16 fields 61 -> 58 | 64 -> 71 | 89 -> 127, 896 tiles 12 | 16 fields 91 -> 104 | 141 -> 134, 1008
//   tiles 8 | 12 | 16 fields 73 -> 76 | 105 -> 106 | 151 -> 136, 1260 tiles 8 fields 88
//   -> 113, 1732 tiles 8 | 12 fields 150 -> 139 | 182 -> 195, 2000 tiles 8 | 12 fields
//   155 -> 146 | 226 -> 202, 2048 tiles 6 fields 120 -> 135, 2592 tiles 8 fields 190 ->
//   197, 3024 tiles 8 | 12 fields 214 -> 212 | 330 -> 300, 5184 tiles 8 fields 383 ->
//   365.  Few fields beyond 1024 tiles stay with k_mult_mrhs (2 fields 5184 tiles 107
//   -> 138).  From 8192 tiles on a launch by itself loses 1-4% (16384 tiles, 12
//   fields 1500 -> 1550), while the iterations of a solve gain (6575 -> 6400 us each).
bool multi_by_tile(int prec, int ntiles, int nsys, int G, bool in_solve) {
    if (prec == P32) {
        if (G != 2) return true;
        if (nsys == 2) return ntiles <= 1024 || ntiles > 2304;
        if ((nsys == 4 || nsys == 6 || nsys == 8) && ntiles > 512 && ntiles <= 680) return false;
        return !(nsys == 4 && ntiles > 1024 && ntiles <= 1200);
    }
    if (ntiles <= 512) return nsys < 15 || ntiles <= 341;
    if (ntiles <= 1024) return nsys < 8 || (nsys >= 12 && ntiles >= 960) || (nsys >= 14 && ntiles >= 850);
    if (nsys < 6) return false;
    if (ntiles < 2700) return nsys <= 8 ? ntiles >= 1580 && ntiles <= 2010 : ntiles >= 1850 && ntiles <= 2030;
    return in_solve || ntiles < 8192;
}

template <int P, int MODE, int RED, int LR> void launch_mrhs_lr(const MrhsArgs &A, hipStream_t s, int G) {
    if (multi_by_tile(P, A.ntiles, A.nsys, G, A.loop)) {
        MrhsArgs B = A;
        // four workgroups fit a compute unit: fill them once, whole systems each
        // (two rounds of half as many systems: 16^3x32, 12 fields 50 -> 65 us)
        B.ngroups = std::max(1, std::min(A.nsys, 1024 / A.ntiles));
        B.chunk = A.chunk * B.ngroups;
        hipLaunchKernelGGL((k_mult_multi<P, MODE, RED, LR>), dim3(A.ntiles * B.ngroups), dim3(64 * kMultiWaves), 0, s, B);
        return;
    }
    MrhsArgs B = A;
    B.ngroups = (A.nsys + G - 1) / G;
    if constexpr (P == P16) {
        if (G != 2) {
            hipLaunchKernelGGL((k_mult_mrhs<P, MODE, RED, LR, 4>), dim3(A.ntiles), dim3(64 * B.ngroups), 0, s, B);
            return;
        }
    }
    hipLaunchKernelGGL((k_mult_mrhs<P, MODE, RED, LR, 2>), dim3(A.ntiles), dim3(64 * B.ngroups), 0, s, B);
}

template <int P, int MODE, int RED> void launch_mrhs_mode(const MrhsArgs &A, hipStream_t s, int lr, int G) {
    if constexpr (P == P32) {
        if (lr == 8) return launch_mrhs_lr<P, MODE, RED, 8>(A, s, G);
        if (lr == 18) return launch_mrhs_lr<P, MODE, RED, 18>(A, s, G);
    }
    launch_mrhs_lr<P, MODE, RED, 12>(A, s, G);
}

template <int P> void dispatch_mrhs(const MrhsArgs &A, int mode, int red, hipStream_t s, int lr, int G) {
    if (mode == M_HOPINV) launch_mrhs_mode<P, M_HOPINV, R_NONE>(A, s, lr, G);
    else if (red == R_DOT) launch_mrhs_mode<P, M_DHAT, R_DOT>(A, s, lr, G);
    else if (red == R_STEP) launch_mrhs_mode<P, M_DHAT, R_STEP>(A, s, lr, G);
    else launch_mrhs_mode<P, M_DHAT, R_NONE>(A, s, lr, G);
}

// ---------------------------------------------------------------------------
// The whole inner loop (Algorithm 2) in one cooperative launch, for lattices
// small enough that every workgroup is resident at once.  Each phase of an
// iteration ends in a grid-wide barrier instead of a kernel boundary; every
// block then sums the reduction partials itself, all in one order, so all
// blocks take the same decisions and leave the loop together.  It sums rho =
// <r~, r> where the launched loop forms it from <r~, s> and <r~, t>, and notices
// each stop at once; the per-site arithmetic is the same otherwise.  The flags, and
// the scalars that the host's closing update reads, are left as the launched loop
// leaves them, so the host finishes the call the same way.  Partials alternate between two buffers: a buffer is written again
// only after a barrier that follows its last read.
// ---------------------------------------------------------------------------
struct PersistArgs {
    Geom g;
    const char *links;
    size_t link_slab;
    const void *clov_e, *clov_o;  // F_ee^-1, F_oo^-1
    void *r, *rt, *p, *q, *t, *tmp, *x;
    double *part[2];              // [kMaxRed][nblk] each
    double *sc;
    int *fl;
    double kappa2;
    int maxit;
    int nblk;
    unsigned long long *bar;  // the kernel's own barrier words (OWN instances)
    unsigned long long tag0;  // call number << 32; barrier k of the call has tag tag0 + k
    unsigned long long epoch; // written to the abort word when a wait runs out
    long long limit;          // wall-clock ticks a wait may take
};

// from this many blocks up the kernel's own barrier beats the runtime's
constexpr int kOwnBarrierMinBlocks = 16;

__device__ __forceinline__ unsigned long long ld_agent(const unsigned long long *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_agent(unsigned long long *p, unsigned long long v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Grid-wide barrier of the one-launch loop.  The runtime's barrier fences
// every wave of every block, which costs about 0.13 us per block; here every
// wave only waits for its own stores to reach L2, and one wave per block
// writes the L2 back (release) and, on the way out, invalidates the caches
// (acquire) before its block reads again.  Each block posts its arrival in a
// word of its own (no contended atomics); one wave of block 0 gathers them
// and posts the release.  Tags grow from barrier to barrier and from call to
// call (the host clears the words when its call counter wraps).  Every
// wait is bounded in wall-clock time: a wait that runs out posts the abort
// word, every other waiter sees it, and the function returns false in every
// block, so the kernel always ends.
template <bool OWN> __device__ __forceinline__ bool grid_barrier(const PersistArgs &A, unsigned long long &tag, int lb) {
    __shared__ int ok;
    ++tag;
    if constexpr (!OWN) {
        cooperative_groups::this_grid().sync();
        return true;
    }
    unsigned long long *w = A.bar;
    unsigned long long *rel = w + A.nblk, *abort = w + A.nblk + 1;
    __builtin_amdgcn_s_waitcnt(0);  // this wave's stores have reached L2
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        st_agent(&w[lb], tag);
    }
    const long long t0 = wall_clock64();
    if (lb == 0 && threadIdx.x < 64) {
        int all = 0;
        for (;;) {
            int mine = 1;
            for (int j = threadIdx.x; j < A.nblk; j += 64) mine &= ld_agent(&w[j]) >= tag;
            all = __all(mine);
            if (all || ld_agent(abort) == A.epoch || wall_clock64() - t0 > A.limit) break;
            __builtin_amdgcn_s_sleep(1);
        }
        if (threadIdx.x == 0) {
            __threadfence();
            if (all) st_agent(rel, tag);
            else st_agent(abort, A.epoch);
        }
    }
    if (threadIdx.x == 0) {
        int good = 1;
        while (ld_agent(rel) < tag) {
            if (ld_agent(abort) == A.epoch || wall_clock64() - t0 > A.limit) {
                st_agent(abort, A.epoch);
                good = 0;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        __threadfence();
        ok = good;
    }
    __syncthreads();
    return ok;
}

// out = F^-1 H in (one parity), the MULT of the launched path
template <int P, int LR>
__device__ __forceinline__ Spinor<typename Real<P>::T> mult_site(const PersistArgs &A, const void *in, int out_par,
                                                                     const void *clov, int i) {
    using R = typename Real<P>::T;
    MultKArgs a;
    a.g = A.g;
    a.out_par = out_par;
    a.in = in;
    a.links = A.links;
    a.link_slab = A.link_slab;
    Spinor<R> acc, out;
#pragma unroll
    for (int k = 0; k < 12; k++) acc.c[k] = {R(0), R(0)};
    const SiteCoord c = eo_coords(A.g, i, out_par);
    hop_dir<P, 0, false, LR>(a, c, i, acc);
    hop_dir<P, 1, false, LR>(a, c, i, acc);
    hop_dir<P, 2, false, LR>(a, c, i, acc);
    hop_dir<P, 3, false, LR>(a, c, i, acc);
    clover_apply<P, R, false>(clov, A.g.Vh, i, acc, out);
    return out;
}

template <class R> __device__ __forceinline__ cx<R> to_r(cx<double> a) { return {(R)a.re, (R)a.im}; }

// The loop runs as four stages per iteration, each opening with the one
// stencil instance of the kernel:
//   0: tmp = F_oo^-1 H_oe p               2: tmp = F_oo^-1 H_oe s
//   1: q = p - kappa^2 F_ee^-1 H_eo tmp   3: t = s - kappa^2 F_ee^-1 H_eo tmp
// followed by the vector updates and reductions of that half-iteration.  A
// single instance keeps the register allocation that of one stencil launch;
// the scalars every thread needs (rho, alpha) stay in registers, the ones
// only the final write-out needs sit in LDS.
template <int P, int LR, bool OWN>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(P == P64 ? 1 : 2))) void k_inner_persistent(PersistArgs A) {
    using R = typename Real<P>::T;
    constexpr int XP = P == P64 ? P64 : P32;
    using RX = typename Real<XP>::T;
    enum { K_RQ = 0, K_N = 2 };
    __shared__ double kept[K_N];  // last <r~, q>, for the write-out by block 0
    const int Vh = A.g.Vh;
    const int lb = xcd_block(blockIdx.x, gridDim.x);  // neighbouring sites share an XCD's L2
    const int i = lb * kBlock + threadIdx.x;
    const bool active = i < Vh;
    const double tol2 = A.sc[S_TOL2];
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < K_N; k++) kept[k] = 0.0;
    }
    cx<double> rho = ld_c(A.sc, S_RHO0), al = {0.0, 0.0};
    int it = 0, stage = 0, done = DONE_NO, stopph = 0;
    unsigned long long tag = A.tag0;
    bool timed_out = false;
    while (it < A.maxit) {
        const bool mult = !(stage & 1);
        const bool second = stage >= 2;
        const void *v = second ? A.r : A.p;  // p, or s (held in r)
        Spinor<R> h;
        if (active) h = mult_site<P, LR>(A, mult ? v : A.tmp, mult ? 1 : 0, mult ? A.clov_o : A.clov_e, i);
        if (mult) {
            if (active) SpinorIO<P>::store(A.tmp, Vh, i, h);
            if (!grid_barrier<OWN>(A, tag, lb)) {
                timed_out = true;
                break;
            }
            stage++;
            continue;
        }
        // D-hat v = v - kappa^2 h into q or t, with <r~, q> or <s, t>, ||t||^2
        Spinor<R> out;
        {
            double d[3] = {0.0, 0.0, 0.0};
            if (active) {
                const Spinor<R> cen = SpinorIO<P>::load(v, Vh, i);
                const R coef = (R)(-A.kappa2);
#pragma unroll
                for (int k = 0; k < 12; k++) out.c[k] = cen.c[k] + coef * h.c[k];
                SpinorIO<P>::store(second ? A.t : A.q, Vh, i, out);
                const Spinor<R> ax = second ? cen : SpinorIO<P>::load(A.rt, Vh, i);
#pragma unroll
                for (int k = 0; k < 12; k++) {
                    const double ar = ax.c[k].re, ai = ax.c[k].im, orr = out.c[k].re, oi = out.c[k].im;
                    d[0] += ar * orr + ai * oi;
                    d[1] += ar * oi - ai * orr;
                    d[2] += orr * orr + oi * oi;
                }
            }
            if (second) {
                block_partials<3>(d, A.part[0], A.nblk, lb);
            } else {
                double d2[2] = {d[0], d[1]};
                block_partials<2>(d2, A.part[0], A.nblk, lb);
            }
            // the updates below use q or t as stored (FP16 storage rounds)
            if constexpr (P == P16) {
                if (active) out = SpinorIO<P>::load(second ? A.t : A.q, Vh, i);
            }
        }
        if (!grid_barrier<OWN>(A, tag, lb)) {
            timed_out = true;
            break;
        }
        if (!second) {
            double sm[2];
            sum_partials<2, 0>(SumSource{A.part[0], A.nblk}, SumSource{nullptr, 0}, sm);
            const cx<double> rq = {sm[0], sm[1]};
            al = cdiv(rho, rq);
            // s = r - alpha q (in r) with ||s||^2; the half-step check
            double n[1] = {0.0};
            if (active) {
                const cx<R> alpha = to_r<R>(al);
                Spinor<R> rv = SpinorIO<P>::load(A.r, Vh, i);
#pragma unroll
                for (int k = 0; k < 12; k++) rv.c[k] = rv.c[k] - alpha * out.c[k];
                SpinorIO<P>::store(A.r, Vh, i, rv);
#pragma unroll
                for (int k = 0; k < 12; k++) n[0] += norm2(rv.c[k]);
            }
            block_partials<1>(n, A.part[1], A.nblk, lb);
            if (!grid_barrier<OWN>(A, tag, lb)) {
                timed_out = true;
                break;
            }
            sum_partials<1, 0>(SumSource{A.part[1], A.nblk}, SumSource{nullptr, 0}, n);
            if (threadIdx.x == 0) {
                kept[K_RQ] = rq.re;
                kept[K_RQ + 1] = rq.im;
            }
            if (!(isfinite(al.re) && isfinite(al.im)) || !isfinite(n[0])) {
                done = DONE_BREAK;
                stopph = 1;
                break;
            }
            if (n[0] < tol2) {
                done = DONE_HALF;
                stopph = 1;
                break;
            }
            stage = 2;
            continue;
        }
        double sm[3];
        sum_partials<3, 0>(SumSource{A.part[0], A.nblk}, SumSource{nullptr, 0}, sm);
        const cx<double> st = {sm[0], sm[1]};
        const double tt = sm[2];
        // x += alpha p + omega s; r = s - omega t with ||r||^2, <r~, r>
        const cx<double> om = {st.re / tt, -st.im / tt};
        double v3[3] = {0.0, 0.0, 0.0};
        if (active) {
            const cx<RX> alx = to_r<RX>(al), omx = to_r<RX>(om);
            const cx<R> omega = to_r<R>(om);
            Spinor<R> sv = SpinorIO<P>::load(A.r, Vh, i);
            const Spinor<R> pv = SpinorIO<P>::load(A.p, Vh, i);
            Spinor<RX> xv = SpinorIO<XP>::load(A.x, Vh, i);
#pragma unroll
            for (int k = 0; k < 12; k++) {
                const cx<RX> pk = {(RX)pv.c[k].re, (RX)pv.c[k].im}, sk = {(RX)sv.c[k].re, (RX)sv.c[k].im};
                xv.c[k] = xv.c[k] + alx * pk + omx * sk;
            }
            SpinorIO<XP>::store(A.x, Vh, i, xv);
#pragma unroll
            for (int k = 0; k < 12; k++) sv.c[k] = sv.c[k] - omega * out.c[k];
            SpinorIO<P>::store(A.r, Vh, i, sv);
            const Spinor<R> rtv = SpinorIO<P>::load(A.rt, Vh, i);
#pragma unroll
            for (int k = 0; k < 12; k++) {
                v3[0] += norm2(sv.c[k]);
                const double ar = rtv.c[k].re, ai = rtv.c[k].im, br = sv.c[k].re, bi = sv.c[k].im;
                v3[1] += ar * br + ai * bi;
                v3[2] += ar * bi - ai * br;
            }
        }
        block_partials<3>(v3, A.part[1], A.nblk, lb);
        if (!grid_barrier<OWN>(A, tag, lb)) {
            timed_out = true;
            break;
        }
        sum_partials<3, 0>(SumSource{A.part[1], A.nblk}, SumSource{nullptr, 0}, v3);
        const double rr = v3[0];
        const cx<double> rho1 = {v3[1], v3[2]};
        const bool bad = !(tt > 0.0) || !(isfinite(om.re) && isfinite(om.im)) || !isfinite(rr) ||
                         (rho1.re == 0.0 && rho1.im == 0.0);
        if (bad || rr < tol2) {
            done = (rr < tol2) ? DONE_FULL : DONE_BREAK;
            stopph = 2;
            it++;
            break;
        }
        // p = r + beta (p - omega q)
        if (active) {
            const cx<R> beta = to_r<R>(cdiv(rho1, rho) * cdiv(al, om)), omega = to_r<R>(om);
            Spinor<R> pv = SpinorIO<P>::load(A.p, Vh, i);
            const Spinor<R> rv = SpinorIO<P>::load(A.r, Vh, i);
            const Spinor<R> qv = SpinorIO<P>::load(A.q, Vh, i);
#pragma unroll
            for (int k = 0; k < 12; k++) pv.c[k] = rv.c[k] + beta * (pv.c[k] - omega * qv.c[k]);
            SpinorIO<P>::store(A.p, Vh, i, pv);
        }
        rho = rho1;
        if (!grid_barrier<OWN>(A, tag, lb)) {
            timed_out = true;
            break;
        }
        stage = 0;
        it++;
    }
    if (timed_out) {
        done = DONE_BREAK;
        stopph = 3;
    }
    // leave the flags as the launched path would, and the scalars the host's
    // closing update reads
    if (lb == 0 && threadIdx.x == 0) {
        double *sc = A.sc;
        sc[S_RHO1] = rho.re;  // with S_RQ, the alpha of a half-step exit
        sc[S_RHO1 + 1] = rho.im;
        sc[S_RQ] = kept[K_RQ];
        sc[S_RQ + 1] = kept[K_RQ + 1];
        A.fl[F_DONE] = done;
        A.fl[F_ITERS] = it;
        A.fl[F_STOPPH] = stopph;
        A.fl[F_RAN] = stopph == 1 ? 1 : 0;
    }
}

}  // namespace

// Several calls on one lattice through the multi-system stencil: G systems per
// thread, the operator loaded once per site for all of them.
static int launch_mult_mrhs(hipStream_t s, const MultCall *calls, int n, wc_lattice *tl, int G) {
    const MultCall &c0 = calls[0];
    wc_lattice *lat = c0.lat;
    const int lr = c0.prec == P32 ? lat->recon : 12;
    MrhsArgs A;
    A.g = lat->g;
    A.out_par = c0.out_par;
    A.links = (const char *)link_base(lat, c0.prec);
    A.link_slab = link_slab_for(lat, c0.prec);
    A.clov = (const char *)lat->clovinv[c0.prec] + (size_t)c0.out_par * clover_slab_bytes(c0.prec, lat->Vh);
    A.coef = c0.coef;
    A.nsys = n;
    A.ngroups = 0;  // set with the form
    A.loop = c0.loop;
    A.ntiles = blocks_of(lat->Vh, 64);
    A.chunk = lattice_chunk(lat, c0.prec);
    double bytes = mult_operator_bytes(c0.prec, c0.mode, lr, lat->Vh);
    for (int k = 0; k < n; k++) {
        const MultCall &c = calls[k];
        if (c.coef != c0.coef) return wc_fail(WC_EINVAL, "multi-system stencil calls must share the coefficient");
        A.s[k] = MrhsSys{c.out, c.in, c.center, c.aux, c.red_to.partials, c.done};
        bytes += mult_spinor_bytes(c.prec, c.mode, c.red, lat->Vh);
        lat->dslash_count++;
    }
    int slot = c0.mode == M_HOPINV ? KS_MULT_HOPINV_P64 + c0.prec : KS_MULT_DHAT_P64 + c0.prec;
    TimedLaunch t;
    if (tl->timing) {
        timing_begin(tl, slot, bytes, t);
        t.iter = tl->tag_iter;
        t.phase = tl->tag_phase;
        TimedPart op{{}, mult_operator_bytes(c0.prec, c0.mode, lr, lat->Vh)};
        for (int k = 0; k < n; k++) {
            const MultCall &c = calls[k];
            t.parts.push_back(TimedPart{{c.done}, mult_spinor_bytes(c.prec, c.mode, c.red, lat->Vh)});
            op.owners.push_back(c.done);
        }
        t.parts.push_back(op);
    }
    if (c0.prec == P32) dispatch_mrhs<P32>(A, c0.mode, c0.red, s, lr, G);
    else dispatch_mrhs<P16>(A, c0.mode, c0.red, s, 12, G);
    WC_HIP(hipGetLastError());
    if (tl->timing) timing_end(tl, t);
    if (c0.red != R_NONE && c0.red_to.result) {
        FinArgs f[kMaxSys];
        for (int k = 0; k < n; k++) {
            f[k] = FinArgs{};
            f[k].blocks = A.ntiles;  // one partial per 64-site tile
            f[k].op = FIN_STORE;
            f[k].partials = calls[k].red_to.partials;
            f[k].result = calls[k].red_to.result;
            f[k].guard = calls[k].done;
        }
        return launch_fin_batch(s, f, n, red_values(c0.red));
    }
    return WC_OK;
}

// the form that a launch of these calls takes
enum StencilForm { F_PLAIN, F_SPLIT, F_MULTI };
static StencilForm stencil_form(const MultCall *calls, int n) {
    const MultCall &c0 = calls[0];
    // several systems on one lattice in an inner-precision stencil: the
    // multi-system form, when the lattice has it switched on
    bool same = n > 1 && mrhs_for(c0.lat, c0.prec) > 0 && (c0.prec == P32 || c0.prec == P16) &&
                (c0.mode == M_HOPINV || c0.mode == M_DHAT);
    for (int k = 1; same && k < n; k++)
        same = calls[k].lat == c0.lat && calls[k].prec == c0.prec && calls[k].mode == c0.mode &&
               calls[k].red == c0.red && calls[k].out_par == c0.out_par && calls[k].coef == c0.coef;
    if (same) return F_MULTI;
    if (c0.mode == M_DCANON) return F_SPLIT;
    // systems interleaved on one lattice share the operator through the cache,
    // which the split form's non-temporal loads would undo
    bool split = c0.mode != M_CLOV && (c0.mode != M_DFULL || c0.prec == P64);  // (FP32: M_DCANON)
    for (int k = 0; split && k < n; k++)
        split = split_stencil(calls[k].lat, c0.prec) && (k == 0 || calls[k].lat != c0.lat);
    return split ? F_SPLIT : F_PLAIN;
}

int stencil_partials(const MultCall *calls, int n, int k) {
    return blocks_of(calls[k].lat->Vh, stencil_form(calls, n) == F_PLAIN ? launch_bs(calls[0].bs) : 64);
}

int launch_mult_batch(hipStream_t s, const MultCall *calls, int n, wc_lattice *timing_lat) {
    if (n <= 0) return WC_OK;
    if (n > kMaxSys) return wc_fail(WC_EINVAL, "too many systems in one batch");
    const MultCall &c0 = calls[0];
    const StencilForm form = stencil_form(calls, n);
    if (form == F_MULTI) return launch_mult_mrhs(s, calls, n, timing_lat ? timing_lat : c0.lat, mrhs_for(c0.lat, c0.prec));
    if (!valid_block_size(launch_bs(c0.bs))) return wc_fail(WC_EINVAL, "block size must be 64, 128 or 256");
    const bool split = form == F_SPLIT;
    const int bs = split ? 64 : launch_bs(c0.bs);  // sites per workgroup
    MultBatch B;
    B.h.S = n;
    B.h.off[0] = 0;
    bool same = true;
    double bytes = 0, link_bytes = 0;
    const int lr = c0.prec == P32 ? c0.lat->recon : 12;  // link form of the FP32 stencil
    for (int k = 0; k < n; k++) {
        const MultCall &c = calls[k];
        wc_lattice *lat = c.lat;
        if (c.prec != c0.prec || c.mode != c0.mode || c.red != c0.red ||
            (c.out_par != c0.out_par && c.mode != M_DCANON))
            return wc_fail(WC_EINVAL, "batched stencil calls must share precision, mode, reduction and parity");
        if (c.bs != c0.bs) return wc_fail(WC_EINVAL, "batched stencil calls must share the block size");
        same = same && (lat == c0.lat);
        MultKArgs &a = B.d[k];
        a.g = lat->g;
        a.out_par = c.out_par;
        a.out = c.out;
        a.in = c.in;
        a.center = c.center;
        a.aux = c.aux;
        if ((c.prec == P32 ? lat->recon : 12) != lr)
            return wc_fail(WC_EINVAL, "batched stencil calls must share the link reconstruction");
        a.links = (const char *)link_base(lat, c.prec);
        a.link_slab = link_slab_for(lat, c.prec);
        const bool use_inv = (c.mode == M_HOPINV || c.mode == M_DHAT || c.mode == M_INVSRC ||
                              (c.mode == M_CLOV && c.inverse));
        const char *cb = (const char *)(use_inv ? lat->clovinv[c.prec] : lat->clov[c.prec]);
        a.clov = cb + (size_t)c.out_par * clover_slab_bytes(c.prec, lat->Vh);
        a.coef = c.coef;
        a.red = c.red_to;
        a.done = c.done;
        a.nblk = blocks_of(lat->Vh, bs);
        B.h.off[k + 1] = B.h.off[k] + a.nblk;
        bytes += mult_spinor_bytes(c.prec, c.mode, c.red, lat->Vh);
        bool seen = false;
        for (int j = 0; j < k; j++) seen = seen || (calls[j].lat == lat);
        if (!seen) {
            bytes += mult_operator_bytes(c.prec, c.mode, lr, lat->Vh);
            link_bytes += 8 * (double)link_bytes_per_site(c.prec, lr) * lat->Vh;
        }
        if (c.mode != M_CLOV) lat->dslash_count++;
    }
    B.h.interleave = (same && n > 1) ? 1 : 0;
    // the lattice's chunk of sites per XCD, in blocks of this launch (with the
    // systems of one lattice interleaved block by block, every system's blocks)
    {
        const int tiles = lattice_chunk(c0.lat, c0.prec);
        B.h.chunk = tiles <= 0 ? 0 : std::max(1, tiles / (bs / 64)) * (B.h.interleave ? n : 1);
    }
    const int blocks = B.h.off[n];
    wc_lattice *tl = timing_lat ? timing_lat : c0.lat;
    int slot = KS_MULT_OTHER;
    if (c0.mode == M_HOPINV) slot = KS_MULT_HOPINV_P64 + c0.prec;
    if (c0.mode == M_DHAT) slot = KS_MULT_DHAT_P64 + c0.prec;
    TimedLaunch t;
    if (tl->timing) {
        timing_begin(tl, slot, bytes, t);
        // split by system, and the operator by the systems that share it
        t.iter = tl->tag_iter;
        t.phase = tl->tag_phase;
        for (int k = 0; k < n; k++) {
            const MultCall &c = calls[k];
            t.parts.push_back(TimedPart{{c.done}, mult_spinor_bytes(c.prec, c.mode, c.red, c.lat->Vh)});
            bool seen = false;
            for (int j = 0; j < k; j++) seen = seen || (calls[j].lat == c.lat);
            if (seen) continue;
            TimedPart op{{}, mult_operator_bytes(c.prec, c.mode, lr, c.lat->Vh)};
            for (int j = k; j < n; j++)
                if (calls[j].lat == c.lat) op.owners.push_back(calls[j].done);
            t.parts.push_back(op);
        }
    }
    const unsigned lds = B.h.interleave ? 0u : cap_lds_bytes(c0.lat, c0.prec, split ? 64 * kSplitWaves : bs, c0.mode);
    const int shape = split ? kSplitBlock : bs;
    const bool keep = link_bytes <= (lr == 8 && !c0.loop ? kKeepLinkBytes8 : kKeepLinkBytes);
    if (c0.prec == P64) dispatch_mode<P64>(B, c0.mode, c0.red, blocks, shape, lds, s, 12, keep);
    else if (c0.prec == P32) dispatch_mode<P32>(B, c0.mode, c0.red, blocks, shape, lds, s, lr, keep);
    else dispatch_mode<P16>(B, c0.mode, c0.red, blocks, shape, lds, s, 12, keep);
    WC_HIP(hipGetLastError());
    if (tl->timing) timing_end(tl, t);
    if (c0.red != R_NONE && c0.mode == M_DHAT && c0.red_to.result) {
        FinArgs f[kMaxSys];
        for (int k = 0; k < n; k++) {
            f[k] = FinArgs{};
            f[k].blocks = blocks_of(calls[k].lat->Vh, bs);
            f[k].op = FIN_STORE;
            f[k].partials = calls[k].red_to.partials;
            f[k].result = calls[k].red_to.result;
            f[k].guard = calls[k].done;
        }
        return launch_fin_batch(s, f, n, red_values(c0.red));
    }
    return WC_OK;
}

std::atomic<double> g_barrier_timeout_s{2.0};

// The inner loop as one cooperative launch; *ran = false (and WC_OK) when the
// lattice is too large for all its workgroups to be resident at once, so the
// caller uses the launched loop instead.
int launch_inner_persistent(const PersistCall &c, hipStream_t s, bool *ran) {
    *ran = false;
    wc_lattice *lat = c.lat;
    const int lr = c.prec == P32 ? lat->recon : 12;
    PersistArgs A;
    A.g = lat->g;
    A.links = (const char *)link_base(lat, c.prec);
    A.link_slab = link_slab_for(lat, c.prec);
    const char *ci = (const char *)lat->clovinv[c.prec];
    A.clov_e = ci;
    A.clov_o = ci + clover_slab_bytes(c.prec, lat->Vh);
    A.r = c.r;
    A.rt = c.rt;
    A.p = c.p;
    A.q = c.q;
    A.t = c.t;
    A.tmp = c.tmp;
    A.x = c.x;
    A.part[0] = c.part0;
    A.part[1] = c.part1;
    A.sc = c.sc;
    A.fl = c.fl;
    A.kappa2 = lat->kappa * lat->kappa;
    A.maxit = c.maxit;
    A.nblk = blocks_of(lat->Vh, kBlock);  // its own 256-thread layout
    // the runtime's barrier is the cheaper one for a handful of blocks only
    A.bar = A.nblk >= kOwnBarrierMinBlocks ? c.bar : nullptr;
    A.epoch = c.epoch;
    A.tag0 = (unsigned long long)c.epoch << 32;
    const bool own = A.bar != nullptr;
    const void *fn = c.prec == P64 ? (own ? (const void *)k_inner_persistent<P64, 12, true>
                                          : (const void *)k_inner_persistent<P64, 12, false>)
                     : c.prec == P16 ? (own ? (const void *)k_inner_persistent<P16, 12, true>
                                            : (const void *)k_inner_persistent<P16, 12, false>)
                     : lr == 8 ? (own ? (const void *)k_inner_persistent<P32, 8, true>
                                      : (const void *)k_inner_persistent<P32, 8, false>)
                     : lr == 18 ? (own ? (const void *)k_inner_persistent<P32, 18, true>
                                       : (const void *)k_inner_persistent<P32, 18, false>)
                                : (own ? (const void *)k_inner_persistent<P32, 12, true>
                                       : (const void *)k_inner_persistent<P32, 12, false>);
    int dev = 0, cus = 0, per_cu = 0, coop = 0, clock_khz = 0;
    WC_HIP(hipGetDevice(&dev));
    WC_HIP(hipDeviceGetAttribute(&clock_khz, hipDeviceAttributeWallClockRate, dev));
    A.limit = (long long)(g_barrier_timeout_s.load() * 1e3 * clock_khz);
    WC_HIP(hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev));
    WC_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    WC_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, kBlock, 0));
    if (!coop || (long)per_cu * cus < A.nblk) return WC_OK;
    void *args[] = {&A};
    const hipError_t e = hipLaunchCooperativeKernel(fn, dim3(A.nblk), dim3(kBlock), args, 0, s);
    if (e == hipErrorCooperativeLaunchTooLarge) {
        (void)hipGetLastError();  // not resident all at once after all: use the launched loop
        return WC_OK;
    }
    if (e != hipSuccess) return wc_fail(WC_EHIP, std::string("cooperative launch: ") + hipGetErrorString(e));
    *ran = true;
    return WC_OK;
}
