// Lane-per-particle neighbour-sum forward: one lane per particle in cell
// order, so the lanes of a wave share home cells and therefore candidate
// cells, and their candidate loads hit the same cache lines.
#include "pair_common.hpp"

namespace aboria {

template <typename T, int D, int OP, bool BATCH, bool OFF32, bool SPLIT>
__global__ __launch_bounds__(SPLIT ? kSearchThreads : 256) void k_lane_fwd(const T* __restrict__ xs, const uint32_t* __restrict__ off,
                                                  const uint32_t* __restrict__ perm, uint32_t n,
                                                  const SysParams<T>* __restrict__ sp,
                                                  const uint32_t* __restrict__ sys_part, int nsys,
                                                  const T* __restrict__ a_s, OpArgs<T> q, T* __restrict__ y,
                                                  int32_t split) {
    using Op = PairOp<T, D, OP>;
    constexpr int NY = Op::NY;
    constexpr uint32_t WB = WindowBytes<T, D, 0>::value;
    extern __shared__ __align__(32) char lds[];
    const WaveRows w = wave_rows<D, SPLIT>(split);
    const uint32_t s = w.s;
    const int b = system_of_row<BATCH>(sys_part, nsys, w.first, s);
    WaveSums<T, D, NY, SPLIT> ws(split, w.wave, part_lds(lds, WB));
    auto& sums = ws.sums;
    if (s < n) {
        const SysParams<T> P = sp[b];
        T xi[D];
        load_point<T, D>(xs, s, xi);
        const T ai = OpShape<OP, D>::NA ? a_s[s] : T(0);
        const T r = P.r;
        auto visit = [&](uint32_t j, const T* dx, T d2, bool) {
            const T aj = OpShape<OP, D>::NA ? load_row<T, 1, OFF32>(a_s, j).v[0] : T(0);
            Op::fwd(q, r, dx, d2, ai, aj, sums.acc);
        };
        neighbour_loop_staged<T, D, OFF32, 0, kDeferForward<T, OP>>(P, xs, (const T*)nullptr, off, n, xi, visit,
                                              [&](int32_t row) { ws.row_done(row); }, w.range,
                                              wave_window(lds, w.wave, WB));
    }
    if (!ws.finish(w, n)) return;
    const uint32_t o = perm[s];
#pragma unroll
    for (int k = 0; k < NY; ++k) y[(size_t)o * NY + k] = sums.tot[k];
}

template <typename T, int D, int OP, bool BATCH>
void launch_lane_fwd(aboria_ctx* ctx, const aboria_cells* c, const OpArgs<T>& q, const T* a_s, T* y) {
    const uint32_t n = (uint32_t)c->n;
    const SysParams<T>* sp = reinterpret_cast<const SysParams<T>*>(c->params_dev);
    const SearchShape sh =
        search_shape(ctx, c, WindowBytes<T, D, 0>::value, WaveSums<T, D, PairOp<T, D, OP>::NY, true>::part_bytes);
#define LF(O, S)                                                                                                    \
    hipLaunchKernelGGL((k_lane_fwd<T, D, OP, BATCH, O, S>), dim3(sh.blocks), dim3(sh.threads), sh.lds, ctx->stream, \
                       (const T*)c->xs, c->off, c->perm, n, sp, c->sys_part_dev, c->nsys, a_s, q, y, sh.split)
    // (rows are split below a size whose offsets are far below 32 bits)
    if (sh.split > 0) LF(true, (D > 1));
    else if (off32_rows<T>(n)) LF(true, false);
    else LF(false, false);
#undef LF
}

#define ABORIA_INST(T, D, OP, BATCH)                                                                   \
    template void launch_lane_fwd<T, D, OP, BATCH>(aboria_ctx*, const aboria_cells*, const OpArgs<T>&, \
                                                   const T*, T*);
ABORIA_FOR_EACH_PAIR_INSTANCE(ABORIA_INST)
#undef ABORIA_INST

}  // namespace aboria
