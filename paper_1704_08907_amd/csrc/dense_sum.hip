// Dense kernel sums of the RBF / Gaussian-process methods (Section 1 and the
// RBF and Kansa examples of Section 1.1): y_i = sum_j K(x_i, x_j) w_j over all
// sources, for the radial kernels K = phi(|x_i - x_j|^2) of those examples:
// the Gaussian exp(-q / (2 sigma^2)) and the multiquadric sqrt(q + c^2); and
// the adjoint of the sum: dL/dw = K^T gy (the same sum with targets and
// sources exchanged) and the position gradients sum_j w_j 2 phi'(q) (a - b).
//
// Each thread keeps TI targets in registers; the workgroup streams tiles of
// 256 sources (position and weight, 16 or 32 bytes each) through LDS, and every
// lane reads each source with one broadcast LDS load.  Gaussian coordinates are
// pre-scaled by sqrt(c) so that the squared scaled distance is directly the
// argument of one exp2 (float) or exp (double).  The source range is split over
// a second grid dimension so that the launch fills all compute units; the split
// partial sums are added in a fixed order by a second kernel (which also
// applies the gradient's per-row factor), and inside a split every tile's sum
// is formed separately before it is added (pairwise accumulation keeps the
// float32 error well below the tile length times u).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <type_traits>

#include "common.hpp"

namespace aboria {

constexpr int kDenseBlock = 256;
constexpr int kDenseTile = 256;  // sources staged in LDS at once
constexpr int kDenseStep = 64;   // the source splits' granularity

// Scratch of aboria_dense_sum_noalloc: its split partial sums live in this
// file-scope device array (each GPU holds its own copy until the process ends)
// instead of the context's grow-only buffer.  Host code never passes the
// array's name to a kernel: in host code it is only a stand-in, and the device
// address of each GPU's copy comes from hipGetSymbolAddress (noalloc_scratch).
constexpr size_t kNoAllocScratchBytes = size_t(16) << 20;
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

__device__ __forceinline__ float kexp(float a) { return __builtin_amdgcn_exp2f(-a); }
__device__ __forceinline__ double kexp(double a) { return ::exp(-a); }
__device__ __forceinline__ float kfma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double kfma(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float ksqrt(float a) { return __builtin_amdgcn_sqrtf(a); }
__device__ __forceinline__ double ksqrt(double a) { return ::sqrt(a); }
__device__ __forceinline__ float krsqrt(float a) { return __builtin_amdgcn_rsqf(a); }
__device__ __forceinline__ double krsqrt(double a) { return ::rsqrt(a); }

// The radial argument q of a pair (displacement dk on the working coordinates), phi(q)
// (value) and the factor of the gradient summand w_j * slope * (a - b) (the constant
// 2 phi' / slope is applied by the reduction): Gaussian q = |dk|^2 on coordinates scaled
// by sqrt(c), value = slope = exp(-q); multiquadric q = |dk|^2 + c^2 (c^2 starts the
// multiply-add chain, one addition less per pair), value = sqrt(q) and slope =
// 1/sqrt(q), each one transcendental instruction, so a pass needing both computes the
// value exactly as the forward does.
template <typename T, int D, int KERN>
struct Radial {
    __device__ __forceinline__ static T arg(const T* dk, T c2) {
        T q = KERN == ABORIA_K_GAUSSIAN ? dk[0] * dk[0] : kfma(dk[0], dk[0], c2);
        if constexpr (D >= 2) q = kfma(dk[1], dk[1], q);
        if constexpr (D >= 3) q = kfma(dk[2], dk[2], q);
        return q;
    }
    __device__ __forceinline__ static T value(T q) {
        if constexpr (KERN == ABORIA_K_GAUSSIAN) return kexp(q);
        else return ksqrt(q);
    }
    __device__ __forceinline__ static T slope(T q) {
        if constexpr (KERN == ABORIA_K_GAUSSIAN) return kexp(q);
        else return krsqrt(q);
    }
};

// What a pass sums per target t over the split's sources j:
//   kSum:     part[split][t]      = sum of K w
//   kGrad:    part[split][t][k]   = sum of w * slope * (xt_t - xs_j)_k
//   kSumGrad: part[split][t][0]   = sum of K w and part[split][t][1 + k] the kGrad sum
//             (one pass for two sums with the same targets, sources and weights:
//             the adjoint's K^T gy and source-position gradient)
enum DenseMode { kSum = 0, kGrad = 1, kSumGrad = 2 };

template <int MODE, int D>
constexpr int dense_out() { return MODE == kSum ? 1 : (MODE == kGrad ? D : D + 1); }

// One pass: targets, sources and weights, the sources of a split (a multiple of
// kDenseStep) and where the split partials go.
template <typename T>
struct DenseJob {
    const T* xt;
    const T* xs;
    const T* w;
    T* part;
    uint32_t nt, ns, jchunk, tblocks;
};

// Target block tb of the pass against the sources of split `split`: what bounds
// it is the issue of the per-pair VALU instructions (6.1 slots per pair for the
// 2-d Gaussian at 65536 points, 0.68 ms), so a source is read once per TI
// targets.  A split may be shorter than a tile: only the tile's filled part,
// rounded up to the unroll (zero weights), is walked.
template <typename T, int D, int TI, int KERN, int MODE>
__device__ __forceinline__ void dense_block(const DenseJob<T>& jb, T sc, T c2, uint32_t tb, uint32_t split,
                                            VecN<T, 4>* tile) {
    using R = Radial<T, D, KERN>;
    constexpr int OUT = dense_out<MODE, D>();
    const uint32_t nt = jb.nt;
    T xi[TI][D];
    T acc[TI][OUT];
#pragma unroll
    for (int q = 0; q < TI; ++q) {
        const uint32_t t = tb * (kDenseBlock * TI) + q * kDenseBlock + threadIdx.x;
        const uint32_t tc = t < nt ? t : nt - 1;
#pragma unroll
        for (int k = 0; k < D; ++k) xi[q][k] = jb.xt[(size_t)tc * D + k] * sc;
#pragma unroll
        for (int k = 0; k < OUT; ++k) acc[q][k] = T(0);
    }
    const uint32_t jbeg = split * jb.jchunk;
    const uint32_t jend = min(jb.ns, jbeg + jb.jchunk);
    for (uint32_t j0 = jbeg; j0 < jend; j0 += kDenseTile) {
        __syncthreads();
        {
            const uint32_t j = j0 + threadIdx.x;
            VecN<T, 4> v;
            v.v[0] = v.v[1] = v.v[2] = v.v[3] = T(0);
            if (j < jend) {
#pragma unroll
                for (int k = 0; k < D; ++k) v.v[k] = jb.xs[(size_t)j * D + k] * sc;
                v.v[3] = jb.w[j];
            }
            tile[threadIdx.x] = v;
        }
        __syncthreads();
        T part[TI][OUT];
#pragma unroll
        for (int q = 0; q < TI; ++q)
#pragma unroll
            for (int k = 0; k < OUT; ++k) part[q][k] = T(0);
        const int cnt = (int)((min(jend - j0, (uint32_t)kDenseTile) + 3u) & ~3u);
        for (int j4 = 0; j4 < cnt; j4 += 4) {
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                const VecN<T, 4> p = tile[j4 + jj];
#pragma unroll
                for (int q = 0; q < TI; ++q) {
                    T dk[D];
#pragma unroll
                    for (int k = 0; k < D; ++k) dk[k] = xi[q][k] - p.v[k];
                    const T q2 = R::arg(dk, c2);
                    if constexpr (MODE == kSum) {
                        part[q][0] = kfma(R::value(q2), p.v[3], part[q][0]);
                    } else {
                        constexpr int G = MODE == kSumGrad ? 1 : 0;  // first gradient component
                        const T slope = R::slope(q2);
                        if constexpr (MODE == kSumGrad)  // (the Gaussian's value is its slope)
                            part[q][0] = kfma(KERN == ABORIA_K_GAUSSIAN ? slope : R::value(q2), p.v[3], part[q][0]);
                        const T h = slope * p.v[3];
#pragma unroll
                        for (int k = 0; k < D; ++k) part[q][G + k] = kfma(h, dk[k], part[q][G + k]);
                    }
                }
            }
        }
#pragma unroll
        for (int q = 0; q < TI; ++q)
#pragma unroll
            for (int k = 0; k < OUT; ++k) acc[q][k] += part[q][k];
    }
#pragma unroll
    for (int q = 0; q < TI; ++q) {
        const uint32_t t = tb * (kDenseBlock * TI) + q * kDenseBlock + threadIdx.x;
        if (t < nt)
#pragma unroll
            for (int k = 0; k < OUT; ++k) jb.part[((size_t)split * nt + t) * OUT + k] = acc[q][k];
    }
}

template <typename T, int D, int TI, int KERN, int MODE>
__global__ __launch_bounds__(kDenseBlock) void k_dense(DenseJob<T> jb, T sc, T c2) {
    __shared__ VecN<T, 4> tile[kDenseTile];
    dense_block<T, D, TI, KERN, MODE>(jb, sc, c2, xcd_tile(blockIdx.x, gridDim.x), blockIdx.y, tile);
}

// The adjoint's two passes in one launch: workgroups below n1 take the source
// pass js (kSumGrad), the others the target pass jt (kGrad).  Two launches of
// a small problem leave most of the chip idle twice.
template <typename T, int D, int TI, int KERN>
__global__ __launch_bounds__(kDenseBlock) void k_dense_adjoint(DenseJob<T> js, DenseJob<T> jt, uint32_t n1, T sc, T c2) {
    __shared__ VecN<T, 4> tile[kDenseTile];
    const uint32_t b = blockIdx.x;
    if (b < n1) dense_block<T, D, TI, KERN, kSumGrad>(js, sc, c2, b % js.tblocks, b / js.tblocks, tile);
    else dense_block<T, D, TI, KERN, kGrad>(jt, sc, c2, (b - n1) % jt.tblocks, (b - n1) / jt.tblocks, tile);
}

// The lane's value from the next lane of the wave (lane 63: from lane 0).
__device__ __forceinline__ float from_next_lane(float v) {
    return __builtin_bit_cast(
        float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x134 /* wave_rol:1 */, 0xF, 0xF, false));
}
__device__ __forceinline__ double from_next_lane(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, 0x134, 0xF, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), 0x134, 0xF, 0xF, false);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// The whole adjoint of a pair at once: targets, sources, weights w and gy, the targets'
// partials pt[split][target][D] (kGrad's) and the sources' ps[target block][source][D + 1]
// (kSumGrad's, with targets and sources exchanged).
template <typename T>
struct DensePairJob {
    const T *xt, *xs, *w, *gy;
    T *pt, *ps;
    uint32_t nt, ns, jchunk, tblocks;
};

// Two passes form every pair's displacement, q and transcendental twice: 26 VALU slots a
// pair for the 3-d multiquadric, and issue bounds them.  Here a pair is formed once.  A
// wave keeps TI targets per lane and takes 64 sources at a time, each lane starting with
// its own and going round: at step s, lane l has source (l + s) mod 64, read from LDS (the
// 64 rows twice, so that no index wraps), whose sums come from the next lane, by one move
// per sum and TI pairs.  After 64 steps every lane has its own source's sums over the
// wave's targets; the four waves' are added in order.  22 slots a pair: 20011 x 30011 in
// 3-d, multiquadric, 366 -> 335 us; 40000^2 in 2-d, Gaussian, 655 -> 502; 12000^2 in 3-d,
// float64, Gaussian, 280 -> 187.
template <typename T, int D, int TI, int KERN>
__global__ __launch_bounds__(kDenseBlock) void k_dense_pairs(DensePairJob<T> jb, T sc, T c2) {
    using R = Radial<T, D, KERN>;
    __shared__ VecN<T, 4> tile[128];
    __shared__ T sums[4][D + 1][64];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint32_t tb = xcd_tile(blockIdx.x, gridDim.x), split = blockIdx.y;
    T xi[TI][D], gi[TI], acc[TI][D];
    // Lanes past the last target stand on it with a gradient of zero.  That leaves a sum as
    // it is unless their kernel value overflows, where the multiquadric's is left out.
    const bool whole = (uint64_t)(tb + 1) * (kDenseBlock * TI) <= jb.nt;
    bool there[TI];
#pragma unroll
    for (int q = 0; q < TI; ++q) {
        const uint32_t t = tb * (kDenseBlock * TI) + q * kDenseBlock + threadIdx.x;
        const uint32_t tc = t < jb.nt ? t : jb.nt - 1;
        there[q] = t < jb.nt;
        gi[q] = t < jb.nt ? jb.gy[tc] : T(0);
#pragma unroll
        for (int k = 0; k < D; ++k) {
            xi[q][k] = jb.xt[(size_t)tc * D + k] * sc;
            acc[q][k] = T(0);
        }
    }
    const uint32_t jbeg = split * jb.jchunk;
    const uint32_t jend = min(jb.ns, jbeg + jb.jchunk);
    for (uint32_t j0 = jbeg; j0 < jend; j0 += 64) {
        if (wave < 2) {  // two waves, one copy each
            const uint32_t j = j0 + lane;
            VecN<T, 4> v;
            v.v[0] = v.v[1] = v.v[2] = v.v[3] = T(0);
            if (j < jend) {
#pragma unroll
                for (int k = 0; k < D; ++k) v.v[k] = jb.xs[(size_t)j * D + k] * sc;
                v.v[3] = jb.w[j];
            }
            tile[threadIdx.x] = v;
        }
        __syncthreads();
        T part[TI][D], own[D + 1];
#pragma unroll
        for (int k = 0; k < D + 1; ++k) own[k] = T(0);
#pragma unroll
        for (int q = 0; q < TI; ++q)
#pragma unroll
            for (int k = 0; k < D; ++k) part[q][k] = T(0);
        auto walk = [&](auto mask_tag) {
            constexpr bool MASK = decltype(mask_tag)::value;
#pragma unroll 2
            for (uint32_t step = 0; step < 64; ++step) {
                const VecN<T, 4> p = tile[lane + step];
                T add[D + 1];
#pragma unroll
                for (int q = 0; q < TI; ++q) {
                    T dk[D];
#pragma unroll
                    for (int k = 0; k < D; ++k) dk[k] = xi[q][k] - p.v[k];
                    const T q2 = R::arg(dk, c2);
                    const T slope = R::slope(q2);
                    T value = KERN == ABORIA_K_GAUSSIAN ? slope : R::value(q2);
                    if constexpr (MASK) value = there[q] ? value : T(0);
                    const T ht = slope * p.v[3], hs = slope * gi[q];
                    add[0] = q == 0 ? value * gi[q] : kfma(value, gi[q], add[0]);
#pragma unroll
                    for (int k = 0; k < D; ++k) {
                        part[q][k] = kfma(ht, dk[k], part[q][k]);
                        add[1 + k] = q == 0 ? hs * dk[k] : kfma(hs, dk[k], add[1 + k]);
                    }
                }
#pragma unroll
                for (int k = 0; k < D + 1; ++k) own[k] = from_next_lane(own[k]) + add[k];
            }
        };
        if (KERN == ABORIA_K_GAUSSIAN || whole) walk(std::integral_constant<bool, false>());
        else walk(std::integral_constant<bool, true>());
#pragma unroll
        for (int q = 0; q < TI; ++q)
#pragma unroll
            for (int k = 0; k < D; ++k) acc[q][k] += part[q][k];
#pragma unroll
        for (int k = 0; k < D + 1; ++k) sums[wave][k][lane] = from_next_lane(own[k]);
        __syncthreads();
        // (the source's displacement is seen from the source: its gradient's sign turns)
        for (uint32_t e = threadIdx.x; e < 64u * (D + 1); e += kDenseBlock) {
            const uint32_t i = e / (D + 1), k = e - i * (D + 1);
            T v = sums[0][k][i] + sums[1][k][i];
            v += sums[2][k][i];
            v += sums[3][k][i];
            if (j0 + i < jend) jb.ps[((size_t)tb * jb.ns + j0) * (D + 1) + e] = k == 0 ? v : -v;
        }
    }
#pragma unroll
    for (int q = 0; q < TI; ++q) {
        const uint32_t t = tb * (kDenseBlock * TI) + q * kDenseBlock + threadIdx.x;
        if (t < jb.nt)
#pragma unroll
            for (int k = 0; k < D; ++k) jb.pt[((size_t)split * jb.nt + t) * D + k] = acc[q][k];
    }
}

// Reduction of one pass's split partials: out[e] = sum over splits of part[split][e]
// for the nt * OUT values e = (target, component).  Component 0 of a kSumGrad pass
// goes to y, every other one to g after the factor mult[target] * C (mult given).
template <typename T>
struct DenseReduceJob {
    const T* part;
    const T* mult;
    T* y;
    T* g;
    uint32_t nt, nsplit;
};

// 64 consecutive values per workgroup and four waves, each wave adding a quarter of
// the splits in split order, the quarters then added in order: every load is a
// contiguous 256-byte run.  (A thread per target walking its components and all
// splits read each line OUT times and kept one load in flight: 30 us for 59 splits
// of 20011 x 3 values; this form 8 us.)
template <typename T, int D, int MODE>
__device__ __forceinline__ void dense_reduce(const DenseReduceJob<T>& jb, T C, uint32_t block, T (*quarter)[64]) {
    constexpr uint32_t OUT = dense_out<MODE, D>();
    const size_t nel = (size_t)jb.nt * OUT;
    const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const size_t e = (size_t)block * 64 + lane;
    const uint32_t per = (jb.nsplit + 3u) / 4u;
    const uint32_t q0 = min(w * per, jb.nsplit), q1 = min(q0 + per, jb.nsplit);
    T s = T(0);
    if (e < nel) {
        const T* p = jb.part + (size_t)q0 * nel + e;
        uint32_t q = q0;
        for (; q + 4 <= q1; q += 4, p += 4 * nel) {
            const T a = p[0], b = p[nel], c = p[2 * nel], d = p[3 * nel];
            s += a;
            s += b;
            s += c;
            s += d;
        }
        for (; q < q1; ++q, p += nel) s += p[0];
    }
    quarter[w][lane] = s;
    __syncthreads();
    if (w != 0 || e >= nel) return;
    s = quarter[0][lane] + quarter[1][lane];
    s += quarter[2][lane];
    s += quarter[3][lane];
    const size_t t = e / OUT;
    const uint32_t k = (uint32_t)(e - t * OUT);
    if (MODE == kSum) jb.y[t] = s;
    else if (MODE == kGrad) jb.g[e] = (jb.mult[t] * C) * s;
    else if (k == 0) jb.y[t] = s;
    else jb.g[t * D + (k - 1)] = (jb.mult[t] * C) * s;
}

template <typename T, int D, int MODE>
__global__ __launch_bounds__(256) void k_dense_reduce(DenseReduceJob<T> jb, T C) {
    __shared__ T quarter[4][64];
    dense_reduce<T, D, MODE>(jb, C, blockIdx.x, quarter);
}

// The reductions of k_dense_adjoint's two passes.
template <typename T, int D>
__global__ __launch_bounds__(256) void k_dense_adjoint_reduce(DenseReduceJob<T> js, DenseReduceJob<T> jt, uint32_t n1,
                                                              T C) {
    __shared__ T quarter[4][64];
    if (blockIdx.x < n1) dense_reduce<T, D, kSumGrad>(js, C, blockIdx.x, quarter);
    else dense_reduce<T, D, kGrad>(jt, C, blockIdx.x - n1, quarter);
}

namespace {

// Launch shapes of the dense sum: targets kept per lane and the number of
// workgroups the source split aims for (the split count is that over the
// target blocks, at most one per kDenseStep sources).  Eight targets per lane are
// float only (float64 would hold twice the registers).  aboria_autotune_dense
// times them; default_plan picks one of the 2048-workgroup plans untuned.
struct DensePlan {
    int32_t ti;
    int32_t wg;
    const char* name;
};
constexpr DensePlan kDensePlans[] = {
    {4, 2048, "4 targets per lane, 2048 workgroups"}, {2, 2048, "2 targets per lane, 2048 workgroups"},
    {8, 2048, "8 targets per lane, 2048 workgroups"}, {4, 4096, "4 targets per lane, 4096 workgroups"},
    {8, 4096, "8 targets per lane, 4096 workgroups"}, {2, 1024, "2 targets per lane, 1024 workgroups"},
    {4, 1024, "4 targets per lane, 1024 workgroups"}, {8, 1024, "8 targets per lane, 1024 workgroups"},
    {1, 2048, "1 targets per lane, 2048 workgroups"},
};
constexpr int32_t kNumDensePlans = sizeof(kDensePlans) / sizeof(kDensePlans[0]);

bool dense_plan_ok(int32_t p, int dtype) {
    return p >= 0 && p < kNumDensePlans && (dtype == ABORIA_F32 || kDensePlans[p].ti <= 4);
}

// From this many pairs on the adjoint forms each pair once (k_dense_pairs); below, its two
// passes side by side keep more workgroups in flight.  Two passes / once, us: 6000^2 in 2-d
// 24.7 / 23.7, 8000^2 in 3-d 47.7 / 41.9, 40000 x 1500 in 1-d 33 / 25; float64 6000^2 73.9 /
// 64.9, 12000 x 3000 in 3-d 79 / 60.
constexpr uint64_t kPairsOnce = uint64_t(1) << 25;

// Tuning key: direction with the adjoint's form (a plan that suits one form of it does not
// suit the other, and both occur in one pair of size buckets), kernel, dtype, d and the size
// buckets (floor log2) of the targets and sources.  Directions count from 4: plans that were
// saved under 0 and 1 were timed on kernels that split the sources by 256 and formed the
// adjoint's pairs twice.
uint64_t dense_key(bool backward, int kernel, int dtype, int d, int64_t nt, int64_t ns) {
    uint64_t k = 4u + (!backward ? 0u : ((uint64_t)nt * (uint64_t)ns < kPairsOnce ? 1u : 2u));
    k = k * 4 + (uint64_t)kernel;
    k = k * 4 + (uint64_t)dtype;
    k = k * 4 + (uint64_t)d;
    k = k * 64 + (uint64_t)std::floor(std::log2((double)nt + 1.0));
    k = k * 64 + (uint64_t)std::floor(std::log2((double)ns + 1.0));
    return k;
}

// The plan of a pass without a tuned or forced choice: two targets per lane when that
// leaves 8192 workgroups of kDenseStep sources (2.7e8 pairs), else one: below, the
// chip holds all workgroups at once and more of them hide more latency; above, half the
// LDS reads per pair count.  Measured with 1 / 2 / 4 targets per lane, us: Gaussian sums
// 5003 x 4099 float64 24 / 27 / 33, 8000^2 19.6 / 21.0 / 22.6, multiquadric 3000 x 40000
// 32 / 36 / 43, 65536^2 720 / 668 / 674, multiquadric adjoint 20011 x 30011 400 / 388 / 404.
int32_t default_plan(uint32_t nt, uint32_t ns) {
    const uint64_t steps = ((uint64_t)ns + kDenseStep - 1) / kDenseStep;
    const uint64_t tblocks = ((uint64_t)nt + 2 * kDenseBlock - 1) / (2 * kDenseBlock);
    return tblocks * steps >= 8192 ? 1 : 8;
}

// The plan a call uses: the tuner's current trial, else the cached choice for
// its key, else -1 (default_plan).
int32_t dense_plan_for(const aboria_ctx* ctx, uint64_t key, int dtype) {
    if (ctx->dense_plan_forced >= 0) return ctx->dense_plan_forced;
    for (const auto& kv : ctx->dense_cache) {
        if (kv.first != key) continue;
        for (int32_t p = 0; p < kNumDensePlans; ++p)
            if (kDensePlans[p].ti == kv.second.ti && kDensePlans[p].wg == kv.second.wg && dense_plan_ok(p, dtype))
                return p;
    }
    return -1;
}

// Kernel constants: Gaussian prm = sigma, multiquadric prm = c.
struct KernelPlan {
    double sc;   // coordinate scale
    double c2;   // multiquadric c^2
    double C;    // gradient constant: 2 phi'(q) (a - b) = C * slope * (scaled a - scaled b)
};

template <typename T>
KernelPlan plan_kernel(int kernel, double prm) {
    KernelPlan k{1.0, 0.0, 1.0};
    if (kernel == ABORIA_K_GAUSSIAN) {
        // float: exp2(-c d^2) with c = log2(e) / (2 sigma^2); double: exp(-d^2 / (2 sigma^2))
        const double c = (sizeof(T) == 4 ? 1.4426950408889634 : 1.0) / (2.0 * prm * prm);
        k.sc = std::sqrt(c);
        k.C = -1.0 / (prm * prm * (double)(T)k.sc);  // 2 phi' = -phi / sigma^2, and d = d' / sc
    } else {
        k.c2 = prm * prm;
    }
    return k;
}

// Gives the context's scratch need bytes.  UNSUPPORTED where it has fewer and a capture is
// in progress (nothing is allocated then), OUT_OF_MEMORY where the device has none left; no
// message, since a caller may have a form that needs less.  A graph may hold scratch that
// was there when it was captured: that is kept until the context goes.
aboria_status grow_scratch(aboria_ctx* ctx, size_t need) {
    if (ctx->scratch_bytes < need) {
        if (ctx->capturing) return ABORIA_ERR_UNSUPPORTED;
        if (ctx->scratch) {
            if (ctx->scratch_in_graph) {
                ctx->scratch_held.push_back(ctx->scratch);
            } else {
                ABORIA_HIP(ctx, hipStreamSynchronize(ctx->stream));
                (void)hipFree(ctx->scratch);
            }
            ctx->scratch = nullptr;
            ctx->scratch_bytes = 0;
            ctx->scratch_in_graph = false;
        }
        if (hipMalloc(&ctx->scratch, need) != hipSuccess) {
            (void)hipGetLastError();
            ctx->scratch = nullptr;
            return ABORIA_ERR_OUT_OF_MEMORY;
        }
        ctx->scratch_bytes = need;
    }
    ctx->scratch_in_graph |= ctx->capturing;
    return ABORIA_OK;
}

aboria_status ensure_scratch(aboria_ctx* ctx, size_t need) {
    const aboria_status st = grow_scratch(ctx, need);
    if (st == ABORIA_ERR_UNSUPPORTED)
        return fail(ctx, st, "dense scratch must be sized by an uncaptured call first");
    if (st == ABORIA_ERR_OUT_OF_MEMORY) return fail(ctx, st, "dense scratch allocation failed");
    return st;
}

// Device address of this GPU's copy of the no-allocation scratch array, looked
// up once per device with that device current and kept for the process.
constexpr int kMaxDevices = 64;
std::mutex g_noalloc_mu;
void* g_noalloc_ptr[kMaxDevices] = {};

aboria_status noalloc_scratch(aboria_ctx* ctx, void** out) {
    if (ctx->device < 0 || ctx->device >= kMaxDevices)
        return fail(ctx, ABORIA_ERR_UNSUPPORTED, "device index beyond the no-allocation scratch table");
    std::lock_guard<std::mutex> lock(g_noalloc_mu);
    if (!g_noalloc_ptr[ctx->device]) {
        int cur = 0;
        ABORIA_HIP(ctx, hipGetDevice(&cur));
        if (cur != ctx->device) ABORIA_HIP(ctx, hipSetDevice(ctx->device));
        void* ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (cur != ctx->device) (void)hipSetDevice(cur);
        if (e != hipSuccess || !ptr) {
            (void)hipGetLastError();
            return fail(ctx, ABORIA_ERR_DEVICE, std::string("hipGetSymbolAddress of the scratch array: ") +
                                                    hipGetErrorString(e));
        }
        g_noalloc_ptr[ctx->device] = ptr;
    }
    *out = g_noalloc_ptr[ctx->device];
    return ABORIA_OK;
}

// Launch shape of one pass under a plan (-1, or one not usable with the type: default_plan).
struct PassShape {
    int32_t ti;
    uint32_t tblocks, nsplit, jchunk;
    size_t split_bytes;  // partials of one split
};

template <typename T, int D, int MODE>
PassShape pass_shape(uint32_t nt, uint32_t ns, int32_t plan, size_t max_splits) {
    const int32_t p =
        dense_plan_ok(plan, sizeof(T) == 4 ? ABORIA_F32 : ABORIA_F64) ? plan : (plan < 0 ? default_plan(nt, ns) : 0);
    PassShape sh;
    sh.ti = kDensePlans[p].ti;
    const uint32_t per_block = kDenseBlock * (uint32_t)sh.ti;
    sh.tblocks = (nt + per_block - 1) / per_block;
    const uint32_t steps = std::max<uint32_t>((ns + kDenseStep - 1) / kDenseStep, 1);
    // enough workgroups to fill 256 CUs several times over
    uint32_t nsplit = std::max<uint32_t>(1, ((uint32_t)kDensePlans[p].wg + sh.tblocks - 1) / sh.tblocks);
    nsplit = (uint32_t)std::min<size_t>(std::min(nsplit, steps), std::max<size_t>(max_splits, 1));
    const uint32_t per_split = (steps + nsplit - 1) / nsplit;
    sh.nsplit = (steps + per_split - 1) / per_split;
    sh.jchunk = per_split * kDenseStep;
    sh.split_bytes = sizeof(T) * (size_t)nt * dense_out<MODE, D>();
    return sh;
}

uint32_t reduce_blocks(uint32_t nt, int out) { return (uint32_t)(((uint64_t)nt * out + 63) / 64); }

// kSum: out = sum_j K(xt_i, xs_j) w_j; kGrad: out = mult_i * C * sum_j w_j slope (xt_i - xs_j);
// kSumGrad: out = the kSum sum and out2 = the kGrad sum, from one pass.  The split
// partials go to the context's grow-only scratch, or, when part is given, to the
// part_cap bytes at part (fewer splits when they would not fit; an error when even
// one split's partials do not).  Every partial entry the reduction reads is
// written by k_dense, so the scratch needs no clearing.
template <typename T, int D, int KERN, int MODE>
aboria_status launch_dense(aboria_ctx* ctx, uint32_t nt, const void* xt, uint32_t ns, const void* xs, const void* w,
                           const KernelPlan& kp, const void* mult, void* out, void* out2, void* part,
                           size_t part_cap, int32_t plan) {
    constexpr int OUT = dense_out<MODE, D>();
    size_t max_splits = SIZE_MAX;
    if (part) {
        max_splits = part_cap / (sizeof(T) * (size_t)nt * OUT);
        if (max_splits == 0)
            return fail(ctx, ABORIA_ERR_INVALID_ARG, "n_target too large for the no-allocation scratch (" +
                                                         std::to_string(part_cap / (sizeof(T) * OUT)) +
                                                         " targets at most)");
    }
    const PassShape sh = pass_shape<T, D, MODE>(nt, ns, plan, max_splits);
    if (!part) {
        aboria_status st = ensure_scratch(ctx, sh.split_bytes * sh.nsplit);
        if (st != ABORIA_OK) return st;
        part = ctx->scratch;
    }
    const DenseJob<T> jb{(const T*)xt, (const T*)xs, (const T*)w, (T*)part, nt, ns, sh.jchunk, sh.tblocks};
#define ABORIA_DENSE_LAUNCH(TI)                                                                                   \
    hipLaunchKernelGGL((k_dense<T, D, TI, KERN, MODE>), dim3(sh.tblocks, sh.nsplit), dim3(kDenseBlock), 0, ctx->stream, \
                       jb, (T)kp.sc, (T)kp.c2)
    switch (sh.ti) {
        case 1: ABORIA_DENSE_LAUNCH(1); break;
        case 2: ABORIA_DENSE_LAUNCH(2); break;
        case 8:
            if constexpr (sizeof(T) == 4) ABORIA_DENSE_LAUNCH(8);
            break;
        default: ABORIA_DENSE_LAUNCH(4); break;
    }
#undef ABORIA_DENSE_LAUNCH
    const DenseReduceJob<T> rj{(const T*)part, (const T*)mult, (T*)out, (T*)(MODE == kGrad ? out : out2), nt, sh.nsplit};
    hipLaunchKernelGGL((k_dense_reduce<T, D, MODE>), dim3(reduce_blocks(nt, OUT)), dim3(256), 0, ctx->stream, rj, (T)kp.C);
    ABORIA_HIP(ctx, hipGetLastError());
    return ABORIA_OK;
}

// Partials of both adjoint passes that one launch may keep at once; above it the passes
// run one after the other in the same scratch.
constexpr size_t kAdjointScratch = size_t(256) << 20;

// Where that scratch leaves it fewer splits than it wants, the fewest workgroups it still
// pays with.  Once / two passes, us: 91000^2 in 3-d, multiquadric, 1424 workgroups 4442 /
// 4650, 91400^2 1074 5082 / 4670, 92000^2 540 6695 / 4720; float64 64200^2 756 6672 / 7520,
// 64400^2 630 8244 / 7560.
template <typename T>
constexpr uint32_t kPairsOnceBlocks = sizeof(T) == 4 ? 1280 : 704;

// The whole adjoint (gw and gxs from the source pass, gxt from the target pass) in one
// launch and one reduction; *done = false when the passes have to run apart.  Both forms
// here take more scratch than either pass: they are left where it cannot be had (a capture
// after uncaptured calls for one gradient at a time, a full device), and an uncaptured call
// leaves scratch for either pass too, so that a capture may ask for fewer gradients.
template <typename T, int D, int KERN>
aboria_status launch_adjoint(aboria_ctx* ctx, uint32_t nt, const void* xt, uint32_t ns, const void* xs, const void* w,
                             const void* gy, const KernelPlan& kp, void* gxt, void* gxs, void* gw, int32_t plan,
                             bool* done) {
    const PassShape a = pass_shape<T, D, kSumGrad>(ns, nt, plan, SIZE_MAX);
    const PassShape b = pass_shape<T, D, kGrad>(nt, ns, plan, SIZE_MAX);
    if ((uint64_t)nt * ns >= kPairsOnce) {
        // (a float-only plan is plan 0 in float64, as in the passes)
        const int32_t p = dense_plan_ok(plan, sizeof(T) == 4 ? ABORIA_F32 : ABORIA_F64) ? plan : std::min(plan, 0);
        const bool given = p >= 0;
        // Two targets per lane: the waves that eight leave hide less in 3-d (20011 x 30011
        // with 2 / 4 / 8: 335 / 351 / 369 us) and are too few for smaller sums; in 1-d and
        // 2-d float32 eight from 2^30 pairs (40000^2 575 / 614 / 502).
        const int32_t ti = given ? kDensePlans[p].ti
                                 : (sizeof(T) == 4 && D <= 2 && (uint64_t)nt * ns >= (uint64_t(1) << 30) ? 8 : 2);
        const uint32_t wg = given ? (uint32_t)kDensePlans[p].wg : 2048u;
        const uint32_t per_block = kDenseBlock * (uint32_t)ti;
        const uint32_t tblocks = (nt + per_block - 1) / per_block, steps = (ns + kDenseStep - 1) / kDenseStep;
        const size_t bytes_s = (sizeof(T) * (size_t)tblocks * ns * (D + 1) + 255) & ~(size_t)255;
        const size_t split_bytes = sizeof(T) * (size_t)nt * D;
        // (at most 384 splits: their sums are read again; 1500 x 40000 with 625 56 us, 342 51)
        uint32_t nsplit = std::min({steps, 384u, std::max<uint32_t>(1, (wg + tblocks - 1) / tblocks)});
        // fewer splits where their partials would not fit
        const size_t left = bytes_s < kAdjointScratch ? (kAdjointScratch - bytes_s) / split_bytes : 0;
        const bool fits = left >= nsplit || tblocks * left >= kPairsOnceBlocks<T>;
        nsplit = (uint32_t)std::min<size_t>(nsplit, std::max<size_t>(left, 1));
        const uint32_t per_split = (steps + nsplit - 1) / nsplit;
        nsplit = (steps + per_split - 1) / per_split;
        const size_t need = bytes_s + split_bytes * nsplit;
        const size_t passes = std::max(a.split_bytes * a.nsplit, b.split_bytes * b.nsplit);
        if (fits && grow_scratch(ctx, ctx->capturing ? need : std::max(need, passes)) == ABORIA_OK) {
            T* ps = (T*)ctx->scratch;
            T* pt = (T*)((char*)ctx->scratch + bytes_s);
            const DensePairJob<T> jb{(const T*)xt, (const T*)xs, (const T*)w, (const T*)gy, pt, ps, nt, ns,
                                     per_split * kDenseStep, tblocks};
#define ABORIA_DENSE_LAUNCH(TI)                                                                                   \
    hipLaunchKernelGGL((k_dense_pairs<T, D, TI, KERN>), dim3(tblocks, nsplit), dim3(kDenseBlock), 0, ctx->stream, \
                       jb, (T)kp.sc, (T)kp.c2)
            switch (ti) {
                case 1: ABORIA_DENSE_LAUNCH(1); break;
                case 2: ABORIA_DENSE_LAUNCH(2); break;
                case 8:
                    if constexpr (sizeof(T) == 4) ABORIA_DENSE_LAUNCH(8);
                    break;
                default: ABORIA_DENSE_LAUNCH(4); break;
            }
#undef ABORIA_DENSE_LAUNCH
            const DenseReduceJob<T> rs{ps, (const T*)w, (T*)gw, (T*)gxs, ns, tblocks};
            const DenseReduceJob<T> rt{pt, (const T*)gy, nullptr, (T*)gxt, nt, nsplit};
            const uint32_t r1 = reduce_blocks(ns, D + 1), r2 = reduce_blocks(nt, D);
            hipLaunchKernelGGL((k_dense_adjoint_reduce<T, D>), dim3(r1 + r2), dim3(256), 0, ctx->stream, rs, rt, r1,
                               (T)kp.C);
            ABORIA_HIP(ctx, hipGetLastError());
            *done = true;
            return ABORIA_OK;
        }
    }
    const size_t bytes_a = (a.split_bytes * a.nsplit + 255) & ~(size_t)255;
    const size_t need = bytes_a + b.split_bytes * b.nsplit;
    // one kernel holds one target count per lane
    *done = a.ti == b.ti && need <= kAdjointScratch && grow_scratch(ctx, need) == ABORIA_OK;
    if (!*done) return ABORIA_OK;
    T* pa = (T*)ctx->scratch;
    T* pb = (T*)((char*)ctx->scratch + bytes_a);
    const DenseJob<T> js{(const T*)xs, (const T*)xt, (const T*)gy, pa, ns, nt, a.jchunk, a.tblocks};
    const DenseJob<T> jt{(const T*)xt, (const T*)xs, (const T*)w, pb, nt, ns, b.jchunk, b.tblocks};
    const uint32_t n1 = a.tblocks * a.nsplit, n2 = b.tblocks * b.nsplit;
#define ABORIA_DENSE_LAUNCH(TI)                                                                                 \
    hipLaunchKernelGGL((k_dense_adjoint<T, D, TI, KERN>), dim3(n1 + n2), dim3(kDenseBlock), 0, ctx->stream, js, jt, n1, \
                       (T)kp.sc, (T)kp.c2)
    switch (a.ti) {
        case 1: ABORIA_DENSE_LAUNCH(1); break;
        case 2: ABORIA_DENSE_LAUNCH(2); break;
        case 8:
            if constexpr (sizeof(T) == 4) ABORIA_DENSE_LAUNCH(8);
            break;
        default: ABORIA_DENSE_LAUNCH(4); break;
    }
#undef ABORIA_DENSE_LAUNCH
    const DenseReduceJob<T> rs{pa, (const T*)w, (T*)gw, (T*)gxs, ns, a.nsplit};
    const DenseReduceJob<T> rt{pb, (const T*)gy, nullptr, (T*)gxt, nt, b.nsplit};
    const uint32_t r1 = reduce_blocks(ns, D + 1), r2 = reduce_blocks(nt, D);
    hipLaunchKernelGGL((k_dense_adjoint_reduce<T, D>), dim3(r1 + r2), dim3(256), 0, ctx->stream, rs, rt, r1, (T)kp.C);
    ABORIA_HIP(ctx, hipGetLastError());
    return ABORIA_OK;
}

template <typename T, int D, int MODE>
aboria_status launch_kernel(aboria_ctx* ctx, int kernel, uint32_t nt, const void* xt, uint32_t ns, const void* xs,
                            const void* w, double prm, const void* mult, void* out, void* out2, void* part,
                            size_t part_cap, int32_t plan) {
    const KernelPlan kp = plan_kernel<T>(kernel, prm);
    if (kernel == ABORIA_K_GAUSSIAN)
        return launch_dense<T, D, ABORIA_K_GAUSSIAN, MODE>(ctx, nt, xt, ns, xs, w, kp, mult, out, out2, part,
                                                            part_cap, plan);
    return launch_dense<T, D, ABORIA_K_MULTIQUADRIC, MODE>(ctx, nt, xt, ns, xs, w, kp, mult, out, out2, part,
                                                            part_cap, plan);
}

template <int MODE>
aboria_status dispatch(aboria_ctx* ctx, int dtype, int d, int kernel, uint32_t nt, const void* xt, uint32_t ns,
                       const void* xs, const void* w, double prm, const void* mult, void* out,
                       void* out2 = nullptr, void* part = nullptr, size_t part_cap = 0, int32_t plan = 0) {
    if (dtype == ABORIA_F32) {
        switch (d) {
            case 1:
                return launch_kernel<float, 1, MODE>(ctx, kernel, nt, xt, ns, xs, w, prm, mult, out, out2, part,
                                                     part_cap, plan);
            case 2:
                return launch_kernel<float, 2, MODE>(ctx, kernel, nt, xt, ns, xs, w, prm, mult, out, out2, part,
                                                     part_cap, plan);
            default:
                return launch_kernel<float, 3, MODE>(ctx, kernel, nt, xt, ns, xs, w, prm, mult, out, out2, part,
                                                     part_cap, plan);
        }
    }
    switch (d) {
        case 1:
            return launch_kernel<double, 1, MODE>(ctx, kernel, nt, xt, ns, xs, w, prm, mult, out, out2, part,
                                                  part_cap, plan);
        case 2:
            return launch_kernel<double, 2, MODE>(ctx, kernel, nt, xt, ns, xs, w, prm, mult, out, out2, part,
                                                  part_cap, plan);
        default:
            return launch_kernel<double, 3, MODE>(ctx, kernel, nt, xt, ns, xs, w, prm, mult, out, out2, part,
                                                  part_cap, plan);
    }
}

template <typename T, int D>
aboria_status adjoint_kernel(aboria_ctx* ctx, int kernel, uint32_t nt, const void* xt, uint32_t ns, const void* xs,
                             const void* w, const void* gy, double prm, void* gxt, void* gxs, void* gw, int32_t plan,
                             bool* done) {
    const KernelPlan kp = plan_kernel<T>(kernel, prm);
    return kernel == ABORIA_K_GAUSSIAN
               ? launch_adjoint<T, D, ABORIA_K_GAUSSIAN>(ctx, nt, xt, ns, xs, w, gy, kp, gxt, gxs, gw, plan, done)
               : launch_adjoint<T, D, ABORIA_K_MULTIQUADRIC>(ctx, nt, xt, ns, xs, w, gy, kp, gxt, gxs, gw, plan, done);
}

template <typename T>
aboria_status dispatch_adjoint(aboria_ctx* ctx, int d, int kernel, uint32_t nt, const void* xt, uint32_t ns,
                               const void* xs, const void* w, const void* gy, double prm, void* gxt, void* gxs,
                               void* gw, int32_t plan, bool* done) {
    switch (d) {
        case 1: return adjoint_kernel<T, 1>(ctx, kernel, nt, xt, ns, xs, w, gy, prm, gxt, gxs, gw, plan, done);
        case 2: return adjoint_kernel<T, 2>(ctx, kernel, nt, xt, ns, xs, w, gy, prm, gxt, gxs, gw, plan, done);
        default: return adjoint_kernel<T, 3>(ctx, kernel, nt, xt, ns, xs, w, gy, prm, gxt, gxs, gw, plan, done);
    }
}

aboria_status check_common(aboria_ctx* ctx, aboria_dtype dtype, aboria_kernel kernel, const double* params_host,
                           int32_t nparams, int32_t d, int64_t n_target, int64_t n_source) {
    if (kernel != ABORIA_K_GAUSSIAN && kernel != ABORIA_K_MULTIQUADRIC)
        return fail(ctx, ABORIA_ERR_INVALID_ARG, "unknown kernel");
    if (dtype != ABORIA_F32 && dtype != ABORIA_F64) return fail(ctx, ABORIA_ERR_INVALID_ARG, "unknown dtype");
    if (nparams != 1 || !params_host) return fail(ctx, ABORIA_ERR_INVALID_ARG, "the kernel takes one parameter");
    const double prm = params_host[0];
    if (!(prm > 0.0) || !std::isfinite(prm))
        return fail(ctx, ABORIA_ERR_INVALID_ARG, "the kernel parameter (sigma or c) must be positive");
    if (d < 1 || d > 3) return fail(ctx, ABORIA_ERR_INVALID_ARG, "d must be 1, 2 or 3");
    if (n_target < 0 || n_source < 0 || n_target >= ((int64_t)1 << 31) || n_source >= ((int64_t)1 << 31))
        return fail(ctx, ABORIA_ERR_INVALID_ARG, "sizes must lie in [0, 2^31)");
    return ABORIA_OK;
}

}  // namespace

}  // namespace aboria

using namespace aboria;

namespace {

// The forward's argument checks, shared by the two entry points.
aboria_status check_dense_sum(aboria_ctx* ctx, aboria_dtype dtype, aboria_kernel kernel, const double* params_host,
                              int32_t nparams, int32_t d, int64_t n_target, const void* xt, int64_t n_source,
                              const void* xs, const void* w, void* y) {
    aboria_status st = check_common(ctx, dtype, kernel, params_host, nparams, d, n_target, n_source);
    if (st != ABORIA_OK) return st;
    if (n_target == 0) return ABORIA_OK;
    if (!xt || !y || (n_source > 0 && (!xs || !w))) return fail(ctx, ABORIA_ERR_INVALID_ARG, "NULL array");
    const size_t tsz = dtype == ABORIA_F32 ? 4 : 8;
    const size_t ny = tsz * (size_t)n_target;
    if (overlaps(y, ny, xt, tsz * d * (size_t)n_target) || overlaps(y, ny, xs, tsz * d * (size_t)n_source) ||
        overlaps(y, ny, w, tsz * (size_t)n_source))
        return fail(ctx, ABORIA_ERR_INVALID_ARG, "y overlaps an input");
    return ABORIA_OK;
}

}  // namespace

extern "C" aboria_status aboria_dense_sum(aboria_ctx* ctx, aboria_dtype dtype, aboria_kernel kernel,
                                          const double* params_host, int32_t nparams, int32_t d, int64_t n_target,
                                          const void* xt, int64_t n_source, const void* xs, const void* w, void* y) {
    if (!ctx) return ABORIA_ERR_INVALID_ARG;
    try {
        aboria_status st =
            check_dense_sum(ctx, dtype, kernel, params_host, nparams, d, n_target, xt, n_source, xs, w, y);
        if (st != ABORIA_OK || n_target == 0) return st;
        const int32_t plan = dense_plan_for(ctx, dense_key(false, kernel, dtype, d, n_target, n_source), dtype);
        return dispatch<kSum>(ctx, dtype, d, kernel, (uint32_t)n_target, xt, (uint32_t)n_source, xs, w,
                              params_host[0], nullptr, y, nullptr, nullptr, 0, plan);
    } catch (...) {
        return fail(ctx, ABORIA_ERR_OUT_OF_MEMORY, "host exception in dense_sum");
    }
}

extern "C" aboria_status aboria_dense_sum_noalloc(aboria_ctx* ctx, aboria_dtype dtype, aboria_kernel kernel,
                                                  const double* params_host, int32_t nparams, int32_t d,
                                                  int64_t n_target, const void* xt, int64_t n_source,
                                                  const void* xs, const void* w, void* y) {
    if (!ctx) return ABORIA_ERR_INVALID_ARG;
    try {
        aboria_status st =
            check_dense_sum(ctx, dtype, kernel, params_host, nparams, d, n_target, xt, n_source, xs, w, y);
        if (st != ABORIA_OK || n_target == 0) return st;
        const size_t tsz = dtype == ABORIA_F32 ? 4 : 8;
        if ((size_t)n_target * tsz > kNoAllocScratchBytes)
            return fail(ctx, ABORIA_ERR_INVALID_ARG,
                        "n_target too large for the no-allocation scratch (" +
                            std::to_string(kNoAllocScratchBytes / tsz) + " targets at most)");
        void* part = nullptr;
        if ((st = noalloc_scratch(ctx, &part)) != ABORIA_OK) return st;
        const int32_t plan = dense_plan_for(ctx, dense_key(false, kernel, dtype, d, n_target, n_source), dtype);
        return dispatch<kSum>(ctx, dtype, d, kernel, (uint32_t)n_target, xt, (uint32_t)n_source, xs, w,
                              params_host[0], nullptr, y, nullptr, part, kNoAllocScratchBytes, plan);
    } catch (...) {
        return fail(ctx, ABORIA_ERR_OUT_OF_MEMORY, "host exception in dense_sum_noalloc");
    }
}

extern "C" aboria_status aboria_dense_sum_backward(aboria_ctx* ctx, aboria_dtype dtype, aboria_kernel kernel,
                                                   const double* params_host, int32_t nparams, int32_t d,
                                                   int64_t n_target, const void* xt, int64_t n_source,
                                                   const void* xs, const void* w, const void* gy, void* gxt,
                                                   void* gxs, void* gw) {
    if (!ctx) return ABORIA_ERR_INVALID_ARG;
    try {
        aboria_status st = check_common(ctx, dtype, kernel, params_host, nparams, d, n_target, n_source);
        if (st != ABORIA_OK) return st;
        if (n_target == 0 || n_source == 0) {
            // no pairs: every requested gradient is zero (a fill kernel, so the call stays capturable)
            const int64_t words = dtype == ABORIA_F32 ? 1 : 2;
            if (gxt && n_target > 0 && (st = fill_u32(ctx, (uint32_t*)gxt, 0u, words * d * n_target)) != ABORIA_OK)
                return st;
            if (gxs && n_source > 0 && (st = fill_u32(ctx, (uint32_t*)gxs, 0u, words * d * n_source)) != ABORIA_OK)
                return st;
            if (gw && n_source > 0 && (st = fill_u32(ctx, (uint32_t*)gw, 0u, words * n_source)) != ABORIA_OK)
                return st;
            return ABORIA_OK;
        }
        if (!xt || !xs || !w || !gy) return fail(ctx, ABORIA_ERR_INVALID_ARG, "NULL input array");
        const size_t tsz = dtype == ABORIA_F32 ? 4 : 8;
        const size_t nt = (size_t)n_target, ns = (size_t)n_source;
        struct Span { const void* p; size_t bytes; };
        const Span ins[] = {{xt, tsz * d * nt}, {xs, tsz * d * ns}, {w, tsz * ns}, {gy, tsz * nt}};
        const Span outs[] = {{gxt, tsz * d * nt}, {gxs, tsz * d * ns}, {gw, tsz * ns}};
        for (const Span& o : outs) {
            if (!o.p) continue;
            for (const Span& i : ins)
                if (overlaps(o.p, o.bytes, i.p, i.bytes))
                    return fail(ctx, ABORIA_ERR_INVALID_ARG, "an output overlaps an input");
            for (const Span& o2 : outs)
                if (&o2 != &o && o2.p && overlaps(o.p, o.bytes, o2.p, o2.bytes))
                    return fail(ctx, ABORIA_ERR_INVALID_ARG, "outputs overlap");
        }
        const double prm = params_host[0];
        const uint32_t t32 = (uint32_t)n_target, s32 = (uint32_t)n_source;
        const int32_t plan = dense_plan_for(ctx, dense_key(true, kernel, dtype, d, n_target, n_source), dtype);
        // dL/dw = K^T gy (the forward sum over the targets, seen from the sources) and the
        // source-position gradient sum over the same pairs with the same weights gy: one
        // pass when both are requested
        if (gw && gxs && gxt) {
            bool done = false;
            st = dtype == ABORIA_F32 ? dispatch_adjoint<float>(ctx, d, kernel, t32, xt, s32, xs, w, gy, prm, gxt, gxs,
                                                               gw, plan, &done)
                                     : dispatch_adjoint<double>(ctx, d, kernel, t32, xt, s32, xs, w, gy, prm, gxt, gxs,
                                                                gw, plan, &done);
            if (st != ABORIA_OK || done) return st;
        }
        if (gw && gxs) {
            if ((st = dispatch<kSumGrad>(ctx, dtype, d, kernel, s32, xs, t32, xt, gy, prm, w, gw, gxs, nullptr, 0,
                                         plan)) != ABORIA_OK)
                return st;
        } else if (gw) {
            if ((st = dispatch<kSum>(ctx, dtype, d, kernel, s32, xs, t32, xt, gy, prm, nullptr, gw, nullptr, nullptr,
                                     0, plan)) != ABORIA_OK)
                return st;
        } else if (gxs) {
            if ((st = dispatch<kGrad>(ctx, dtype, d, kernel, s32, xs, t32, xt, gy, prm, w, gxs, nullptr, nullptr, 0,
                                      plan)) != ABORIA_OK)
                return st;
        }
        if (gxt && (st = dispatch<kGrad>(ctx, dtype, d, kernel, t32, xt, s32, xs, w, prm, gy, gxt, nullptr, nullptr,
                                         0, plan)) != ABORIA_OK)
            return st;
        return ABORIA_OK;
    } catch (...) {
        return fail(ctx, ABORIA_ERR_OUT_OF_MEMORY, "host exception in dense_sum_backward");
    }
}

extern "C" aboria_status aboria_set_dense_plan(aboria_ctx* ctx, int32_t plan) {
    if (!ctx) return ABORIA_ERR_INVALID_ARG;
    if (plan < -1 || plan >= kNumDensePlans) return fail(ctx, ABORIA_ERR_INVALID_ARG, "no such dense plan");
    ctx->dense_plan_forced = plan;
    return ABORIA_OK;
}

extern "C" const char* aboria_dense_plan_name(int32_t plan) {
    return plan >= 0 && plan < kNumDensePlans ? kDensePlans[plan].name : "";
}

extern "C" aboria_status aboria_autotune_dense(aboria_ctx* ctx, aboria_dtype dtype, aboria_kernel kernel,
                                               const double* params_host, int32_t nparams, int32_t d,
                                               int64_t n_target, const void* xt, int64_t n_source, const void* xs,
                                               const void* w, const void* gy, void* scratch, int32_t* choice_host) {
    if (!ctx) return ABORIA_ERR_INVALID_ARG;
    if (ctx->capturing) return fail(ctx, ABORIA_ERR_UNSUPPORTED, "autotune cannot be captured");
    try {
        aboria_status st = check_common(ctx, dtype, kernel, params_host, nparams, d, n_target, n_source);
        if (st != ABORIA_OK) return st;
        if (n_target == 0 || n_source == 0) return fail(ctx, ABORIA_ERR_INVALID_ARG, "nothing to time: no pairs");
        if (!xt || !xs || !w || !scratch) return fail(ctx, ABORIA_ERR_INVALID_ARG, "NULL array");
        const bool backward = gy != nullptr;
        const size_t tsz = dtype == ABORIA_F32 ? 4 : 8;
        char* sc = static_cast<char*>(scratch);
        void* gxt = sc;
        void* gxs = sc + tsz * (size_t)d * (size_t)n_target;
        void* gw = sc + tsz * (size_t)d * (size_t)(n_target + n_source);
        auto run = [&]() {
            return backward ? aboria_dense_sum_backward(ctx, dtype, kernel, params_host, nparams, d, n_target, xt,
                                                        n_source, xs, w, gy, gxt, gxs, gw)
                            : aboria_dense_sum(ctx, dtype, kernel, params_host, nparams, d, n_target, xt, n_source,
                                               xs, w, scratch);
        };
        ABORIA_HIP(ctx, hipSetDevice(ctx->device));
        hipEvent_t e0 = nullptr, e1 = nullptr;
        if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
            if (e0) (void)hipEventDestroy(e0);
            return hip_fail(ctx, hipGetLastError(), "hipEventCreate");
        }
        double best_ms = INFINITY;
        int32_t best = 0;
        const int32_t forced_before = ctx->dense_plan_forced;
        for (int32_t p = 0; p < kNumDensePlans && st == ABORIA_OK; ++p) {
            if (!dense_plan_ok(p, dtype)) continue;
            ctx->dense_plan_forced = p;
            if ((st = run()) != ABORIA_OK) break;  // warm-up
            (void)hipEventRecord(e0, ctx->stream);
            for (int rep = 0; rep < 3 && st == ABORIA_OK; ++rep) st = run();
            (void)hipEventRecord(e1, ctx->stream);
            if (hipEventSynchronize(e1) != hipSuccess) {
                st = hip_fail(ctx, hipGetLastError(), "timing a dense plan");
                break;
            }
            float ms = 0.f;
            (void)hipEventElapsedTime(&ms, e0, e1);
            log_msg("autotune_dense: %s %.4f ms", kDensePlans[p].name, ms / 3.0);
            if (ms < best_ms) {
                best_ms = ms;
                best = p;
            }
        }
        ctx->dense_plan_forced = forced_before;
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
        if (st != ABORIA_OK) return st;
        const uint64_t key = dense_key(backward, kernel, dtype, d, n_target, n_source);
        const aboria_ctx::DenseChoice ch{kDensePlans[best].ti, kDensePlans[best].wg};
        bool found = false;
        for (auto& kv : ctx->dense_cache)
            if (kv.first == key) {
                kv.second = ch;
                found = true;
            }
        if (!found) ctx->dense_cache.emplace_back(key, ch);
        tune_cache_save(ctx);
        log_msg("autotune_dense: %s chosen", kDensePlans[best].name);
        if (choice_host) *choice_host = best;
        return ABORIA_OK;
    } catch (...) {
        ctx->dense_plan_forced = -1;
        return fail(ctx, ABORIA_ERR_OUT_OF_MEMORY, "host exception in autotune_dense");
    }
}
