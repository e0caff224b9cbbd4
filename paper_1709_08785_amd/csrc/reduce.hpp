// Deterministic two-stage reductions for 64-wide wavefronts.
//
// Stage 1 (inside the producing kernel): each block folds its per-thread
// values over its wavefronts and an LDS pass in a fixed order and writes
// one partial per value with a plain store.  Stage 2 sums the partials in a
// fixed order and runs the scalar logic of the solver: in the inner loop in every
// block of the kernel that consumes them (sum_partials), elsewhere in a separate
// one-block kernel (k_finalize, blas.hip).  The kernel boundary makes the partials
// visible; no block ever waits on, or fences against, another block, so the
// per-XCD L2 caches keep the stencil's working set.  Accumulation is FP64 and
// the summation order is fixed, so results are bit-reproducible.
#pragma once

#include "common.hpp"
#include "internal.hpp"

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / 64;

// one step of the wave fold: the lanes that dpp control CTRL supplies with a
// neighbour's value add it, the rows not in ROWS add zero
template <int CTRL, int ROWS> __device__ __forceinline__ double dpp_add(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffff), CTRL, ROWS, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xf, true);
    return v + __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Sum over the wavefront, in every lane.  Rows of 16 lanes by shifts, then the
// rows by broadcasts of lanes 15 and 31; the total arrives in lane 63.  These
// are moves between registers: as shuffles the 12 exchanges of each value went
// through LDS, and the split stencil, with four wavefronts on 64 sites, spent
// 25 us of a 192 us D-hat half at 32^3x64 on them.
template <int N> __device__ __forceinline__ void wave_fold(double (&v)[N]) {
#pragma unroll
    for (int k = 0; k < N; k++) v[k] = dpp_add<0x111, 0xf>(v[k]);  // row_shr:1
#pragma unroll
    for (int k = 0; k < N; k++) v[k] = dpp_add<0x112, 0xf>(v[k]);  // row_shr:2
#pragma unroll
    for (int k = 0; k < N; k++) v[k] = dpp_add<0x114, 0xf>(v[k]);  // row_shr:4
#pragma unroll
    for (int k = 0; k < N; k++) v[k] = dpp_add<0x118, 0xf>(v[k]);  // row_shr:8
#pragma unroll
    for (int k = 0; k < N; k++) v[k] = dpp_add<0x142, 0xa>(v[k]);  // row_bcast:15
#pragma unroll
    for (int k = 0; k < N; k++) v[k] = dpp_add<0x143, 0xc>(v[k]);  // row_bcast:31
#pragma unroll
    for (int k = 0; k < N; k++) {
        const long long b = __double_as_longlong(v[k]);
        const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffff), 63);
        const int hi = __builtin_amdgcn_readlane((int)(b >> 32), 63);
        v[k] = __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
    }
}

// Block-wide fold; the total is valid in thread 0.
template <int N> __device__ __forceinline__ void block_fold(double (&v)[N], double (*sh)[kWaves]) {
    wave_fold<N>(v);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < N; k++) sh[k][wave] = v[k];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const int nw = blockDim.x >> 6;  // 1, 2 or 4 waves
#pragma unroll
        for (int k = 0; k < N; k++) {
            double s = 0.0;
            for (int w = 0; w < nw; w++) s += sh[k][w];
            v[k] = s;
        }
    }
}

// Stage 1: per-block partials of one system, laid out [k][G] with G the
// system's number of blocks and blk this block's index among them.  Every
// thread of the block must call this.
template <int N>
__device__ __forceinline__ void block_partials(double (&v)[N], double *partials, int G, int blk) {
    __shared__ double sh[N][kWaves];
    block_fold<N>(v, sh);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < N; k++) partials[(size_t)k * G + blk] = v[k];
    }
}

// a value every lane holds alike, read from lane 0 so the compiler knows it
// is uniform (branches on it stay scalar, pointers chosen by it stay in SGPRs)
__device__ __forceinline__ double uniform(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readfirstlane((int)(b & 0xffffffff));
    const int hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Every block: the NA + NB sums of two sets of partials, in one order for all
// blocks.  Every thread of the block must call this.
template <int NA, int NB>
__device__ __forceinline__ void sum_partials(SumSource a, SumSource b, double (&out)[NA + NB]) {
    constexpr int N = NA + NB;
    __shared__ double sh[N][kWaves];
    double v[N];
#pragma unroll
    for (int k = 0; k < N; k++) v[k] = 0.0;
#pragma unroll 4
    for (int j = threadIdx.x; j < a.n; j += blockDim.x) {
#pragma unroll
        for (int k = 0; k < NA; k++) v[k] += a.p[(size_t)k * a.n + j];
    }
#pragma unroll 4
    for (int j = threadIdx.x; j < b.n; j += blockDim.x) {
#pragma unroll
        for (int k = 0; k < NB; k++) v[NA + k] += b.p[(size_t)k * b.n + j];
    }
    wave_fold<N>(v);
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int k = 0; k < N; k++) sh[k][threadIdx.x >> 6] = v[k];
    }
    __syncthreads();
    const int nw = blockDim.x >> 6;
#pragma unroll
    for (int k = 0; k < N; k++) {
        double s = 0.0;
        for (int w = 0; w < nw; w++) s += sh[k][w];
        out[k] = uniform(s);
    }
    __syncthreads();
}

// A batched launch covers several systems.  Concatenated: system s owns the
// logical blocks [off[s], off[s+1]).  Interleaved (all systems on one lattice,
// equal block counts): logical block L belongs to system L mod S, block L / S.
struct BatchHdr {
    int S;
    int interleave;
    int chunk;  // blocks per XCD chunk of the stencil's block remap (xcd_block)
    int off[kMaxSys + 1];
};

__device__ __forceinline__ void batch_locate(const BatchHdr &h, int L, int &s, int &lb) {
    if (h.interleave) {
        s = L % h.S;
        lb = L / h.S;
    } else {
        s = 0;
        while (s + 1 < h.S && L >= h.off[s + 1]) s++;
        lb = L - h.off[s];
    }
}

// complex helpers on the device scalar block
__device__ __forceinline__ cx<double> ld_c(const double *s, int slot) { return {s[slot], s[slot + 1]}; }
__device__ __forceinline__ cx<double> cdiv(cx<double> a, cx<double> b) {
    double d = b.re * b.re + b.im * b.im;
    return {(a.re * b.re + a.im * b.im) / d, (a.im * b.re - a.re * b.im) / d};
}
