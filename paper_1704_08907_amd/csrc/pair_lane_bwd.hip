// Lane-per-particle neighbour-sum adjoint (gather form: no atomics, no stored
// pair list between calls).
//
// The row-search adjoint defers the summands of vector operators: it tests up
// to 32 candidates into a per-lane bit mask, then pops the bits, reloads each
// accepted pair's position and gradient row, recomputes its displacement
// exactly and evaluates the summand, so a wave runs the summand as often as
// its busiest lane has pairs instead of for every candidate that any lane
// accepted.  The pairs and their order are those of the box search.
#include "pair_common.hpp"

namespace aboria {

// Elements of a gradient row in the windows, beside the positions (the count needs none).
// (Gathered from HBM for each accepted pair, the soft sphere's one element cost 15 us of
// 180 at 2^20 particles.)
template <int OP, int D>
constexpr int kWinGrad = OP == ABORIA_OP_COUNT ? 0 : GyPitch<OpShape<OP, D>::NY>::value;

// The adjoint, or with FUSED the forward and the adjoint in one box search (the
// upstream gradient is known before the forward): each accepted pair adds its
// forward summand to y_i and its adjoint contribution to gx_i (and ga_i), in the
// order of the separate kernels.
template <typename T, int D, int OP, bool BATCH, bool OFF32, bool FUSED, bool SPLIT>
__global__ __launch_bounds__(SPLIT ? kSearchThreads : 256) void k_lane_bwd(const T* __restrict__ xs, const uint32_t* __restrict__ off,
                                                  const uint32_t* __restrict__ perm, uint32_t n,
                                                  const SysParams<T>* __restrict__ sp,
                                                  const uint32_t* __restrict__ sys_part, int nsys,
                                                  const T* __restrict__ a_s, const T* __restrict__ gy_s,
                                                  OpArgs<T> q, T* __restrict__ y, T* __restrict__ gx,
                                                  T* __restrict__ ga, int32_t split) {
    using Op = PairOp<T, D, OP>;
    constexpr int NY = Op::NY, NA = OpShape<OP, D>::NA;
    constexpr int F = FUSED ? NY : 0;  // the sums: y (fused), gx, ga
    constexpr uint32_t WB = WindowBytes<T, D, kWinGrad<OP, D>>::value;
    extern __shared__ __align__(32) char lds[];
    const WaveRows w = wave_rows<D, SPLIT>(split);
    const uint32_t s = w.s;
    const int b = system_of_row<BATCH>(sys_part, nsys, w.first, s);
    WaveSums<T, D, F + D + NA, SPLIT> ws(split, w.wave, part_lds(lds, WB));
    auto& sums = ws.sums;
    if (s < n) {
        const SysParams<T> P = sp[b];
        T xi[D];
        load_point<T, D>(xs, s, xi);
        const T ai = NA ? a_s[s] : T(0);
        T gyi[NY];
        load_gy<T, NY, OFF32>(gy_s, s, gyi);
        const T r = P.r;
        T* const acc = sums.acc;
        auto pair = [&](uint32_t j, const T* dx, T d2, const T* gyj) {
            const T aj = NA ? load_row<T, 1, OFF32>(a_s, j).v[0] : T(0);
            if constexpr (FUSED) Op::fwd(q, r, dx, d2, ai, aj, acc);
            Op::bwd(q, r, dx, d2, ai, aj, gyi, gyj, acc + F, acc + F + (NA ? D : 0));
        };
        auto row_done = [&](int32_t row) { ws.row_done(row); };
        char* const wb = wave_window(lds, w.wave, WB);
        // accepted pairs first, then their summands, where those cost several pair tests;
        // the neighbour's gradient row comes with its position
        auto visit = [&](uint32_t j, const T* dx, T d2, bool, const T* gyj) { pair(j, dx, d2, gyj); };
        if constexpr (OP == ABORIA_OP_COUNT) {
            const T none[1] = {T(0)};
            neighbour_loop_staged<T, D, OFF32, 0>(P, xs, (const T*)nullptr, off, n, xi,
                                                  [&](uint32_t j, const T* dx, T d2, bool) { pair(j, dx, d2, none); },
                                                  row_done, w.range, wb);
        } else {
            neighbour_loop_staged<T, D, OFF32, NY, kDeferAdjoint<OP>>(P, xs, gy_s, off, n, xi, visit, row_done, w.range,
                                                                     wb);
        }
    }
    if (!ws.finish(w, n)) return;
    const uint32_t o = perm[s];
    if constexpr (FUSED) {
#pragma unroll
        for (int k = 0; k < NY; ++k) y[(size_t)o * NY + k] = sums.tot[k];
    }
#pragma unroll
    for (int k = 0; k < D; ++k) gx[(size_t)o * D + k] = sums.tot[F + k];
    if (NA && ga) ga[o] = sums.tot[F + D + NA - 1];
}

template <typename T, int D, int OP, bool BATCH, bool FUSED>
void launch_bwd_kernel(aboria_ctx* ctx, const aboria_cells* c, const OpArgs<T>& q, const T* a_s, const T* gy_s, T* y,
                       T* gx, T* ga) {
    const uint32_t n = (uint32_t)c->n;
    const SysParams<T>* sp = reinterpret_cast<const SysParams<T>*>(c->params_dev);
    constexpr int NV = (FUSED ? OpShape<OP, D>::NY : 0) + D + OpShape<OP, D>::NA;
    const SearchShape sh =
        search_shape(ctx, c, WindowBytes<T, D, kWinGrad<OP, D>>::value, WaveSums<T, D, NV, true>::part_bytes);
#define LB(O, S)                                                                                              \
    hipLaunchKernelGGL((k_lane_bwd<T, D, OP, BATCH, O, FUSED, S>), dim3(sh.blocks), dim3(sh.threads), sh.lds, \
                       ctx->stream, (const T*)c->xs, c->off, c->perm, n, sp, c->sys_part_dev, c->nsys, a_s,   \
                       gy_s, q, y, gx, ga, sh.split)
    if (sh.split > 0) LB(true, (D > 1));
    else if (off32_rows<T>(n)) LB(true, false);
    else LB(false, false);
#undef LB
}

template <typename T, int D, int OP, bool BATCH>
void launch_lane_fused(aboria_ctx* ctx, const aboria_cells* c, const OpArgs<T>& q, const T* a_s, const T* gy_s,
                       T* y, T* gx, T* ga) {
    launch_bwd_kernel<T, D, OP, BATCH, true>(ctx, c, q, a_s, gy_s, y, gx, ga);
}

template <typename T, int D, int OP, bool BATCH>
void launch_lane_bwd(aboria_ctx* ctx, const aboria_cells* c, const OpArgs<T>& q, const T* a_s, const T* gy_s, T* gx,
                     T* ga) {
    launch_bwd_kernel<T, D, OP, BATCH, false>(ctx, c, q, a_s, gy_s, nullptr, gx, ga);
}

#define ABORIA_INST(T, D, OP, BATCH)                                                                          \
    template void launch_lane_bwd<T, D, OP, BATCH>(aboria_ctx*, const aboria_cells*, const OpArgs<T>&, const T*,   \
                                                   const T*, T*, T*);                                   \
    template void launch_lane_fused<T, D, OP, BATCH>(aboria_ctx*, const aboria_cells*, const OpArgs<T>&, const T*, \
                                                     const T*, T*, T*, T*);
ABORIA_FOR_EACH_PAIR_INSTANCE(ABORIA_INST)
#undef ABORIA_INST

}  // namespace aboria
