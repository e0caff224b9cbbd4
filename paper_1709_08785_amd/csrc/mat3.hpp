// FP64 3x3 complex matrices in registers, and the lattice steps, of the kernels
// that multiply links along closed paths (the clover build and the gradient).
#pragma once

#include "common.hpp"

using C = cx<double>;
using M3 = Mat3<double>;

// an anti-Hermitian matrix: its imaginary diagonal and the entries above the
// diagonal, 9 reals
struct AntiHerm {
    double d[3];
    C o[3];  // (0,1) (0,2) (1,2)
};

// entry (i, j), i != j
__device__ __forceinline__ C ah_off(const AntiHerm &x, int i, int j) {
    const C v = x.o[i + j - 1];
    return i < j ? v : C{-v.re, v.im};
}

// c += a b
__device__ __forceinline__ void mmac(M3 &c, const M3 &a, const M3 &b) {
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++)
#pragma unroll
            for (int k = 0; k < 3; k++) cmac(c.m[3 * i + j], a.m[3 * i + k], b.m[3 * k + j]);
}
// c += a b^dagger
__device__ __forceinline__ void mmac_d(M3 &c, const M3 &a, const M3 &b) {
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++)
#pragma unroll
            for (int k = 0; k < 3; k++) cmacc(c.m[3 * i + j], b.m[3 * j + k], a.m[3 * i + k]);
}
// c += a^dagger b
__device__ __forceinline__ void mdmac(M3 &c, const M3 &a, const M3 &b) {
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++)
#pragma unroll
            for (int k = 0; k < 3; k++) cmacc(c.m[3 * i + j], a.m[3 * k + i], b.m[3 * k + j]);
}
// c += x a
__device__ __forceinline__ void xmac(M3 &c, const AntiHerm &x, const M3 &a) {
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++)
#pragma unroll
            for (int k = 0; k < 3; k++) {
                C &t = c.m[3 * i + j];
                if (k == i) {
                    t.re = fmar(-x.d[i], a.m[3 * k + j].im, t.re);
                    t.im = fmar(x.d[i], a.m[3 * k + j].re, t.im);
                } else {
                    cmac(t, ah_off(x, i, k), a.m[3 * k + j]);
                }
            }
}
// c += a x
__device__ __forceinline__ void macx(M3 &c, const M3 &a, const AntiHerm &x) {
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++)
#pragma unroll
            for (int k = 0; k < 3; k++) {
                C &t = c.m[3 * i + j];
                if (k == j) {
                    t.re = fmar(-x.d[j], a.m[3 * i + k].im, t.re);
                    t.im = fmar(x.d[j], a.m[3 * i + k].re, t.im);
                } else {
                    cmac(t, a.m[3 * i + k], ah_off(x, k, j));
                }
            }
}
__device__ __forceinline__ M3 mzero() {
    M3 c;
#pragma unroll
    for (int k = 0; k < 9; k++) c.m[k] = {0.0, 0.0};
    return c;
}
__device__ __forceinline__ M3 mdag(const M3 &a) {
    M3 c;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) c.m[3 * i + j] = conjx(a.m[3 * j + i]);
    return c;
}

// lexicographic step of one site along a direction, with the periodic wrap
__device__ __forceinline__ int lex_step(const Geom &g, const SiteCoord &c, int mu, bool up) {
    const int x = mu == 0 ? c.x : mu == 1 ? c.y : mu == 2 ? c.z : c.t;
    const int stride = mu == 0 ? 1 : mu == 1 ? g.L[0] : mu == 2 ? g.L[0] * g.L[1] : g.L[0] * g.L[1] * g.L[2];
    const int L = g.L[mu];
    if (up) return x == L - 1 ? -(L - 1) * stride : stride;
    return x == 0 ? (L - 1) * stride : -stride;
}
