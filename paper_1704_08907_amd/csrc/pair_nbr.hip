// Recorded neighbour lists: one box search per build that keeps each
// particle's accepted neighbours, so that the forward sums and the adjoints
// that follow on the same cell list evaluate accepted pairs only instead of
// repeating the pair test on every candidate of the 3^d cells (about 6.7
// candidates per accepted pair at 30 neighbours in 3-d).
//
// Layout: entry k of slot s at nbr[k * n + s] (a wave reads 64 consecutive
// words per entry), the neighbour's slot with kNbrShift set when the search
// reached it through an image shift and the row flag (nbr_entry.hpp) on the first neighbour
// of a stencil row, in box-search order, so a replayed sum adds its summands, row by
// row, in the same order as the search kernels.  nbr_count[s] is
// the slot's neighbour count, or kNbrOverflow where the list does not hold them all: such a
// slot is summed by the box search when replayed, also by a graph that was captured when
// the list held more.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "pair_common.hpp"

namespace aboria {

namespace {

constexpr uint32_t kMaxNbrCap = 4096;

// One lane per particle, the rows read through the wave's LDS window.  With SPLIT and
// split > 1 the rows of 64 particles are shared by that many waves, as in the sums.  A
// wave then keeps what it finds in LDS ([entry][lane]), and writes it after the entries of
// the waves before it; a wave with a lane of more entries than it can keep searches its
// rows once more for the rest, unless the list has no room for that particle's anyway.
template <typename T, int D, bool BATCH, bool OFF32, bool SPLIT>
__global__ __launch_bounds__(SPLIT ? kSearchThreads : 256) void k_nbr_build(const T* __restrict__ xs, const uint32_t* __restrict__ off,
                                                   uint32_t n, const SysParams<T>* __restrict__ sp,
                                                   const uint32_t* __restrict__ sys_part, int nsys,
                                                   uint32_t* __restrict__ nbr, uint32_t* __restrict__ nbr_count,
                                                   uint32_t cap, uint32_t* __restrict__ gen, int32_t split) {
    constexpr uint32_t WB = WindowBytes<T, D, 0>::value;
    extern __shared__ __align__(32) char lds[];
    const WaveRows w = wave_rows<D, SPLIT>(split);
    const uint32_t s = w.s;
    const int b = system_of_row<BATCH>(sys_part, nsys, w.first, s);
    const bool shared_rows = SPLIT && split > 1;
    const uint32_t lane = threadIdx.x & 63u;
    // after the windows: the waves' entries, and their counts
    const uint32_t kept = stash_of(split);
    uint32_t* const stash = reinterpret_cast<uint32_t*>(part_lds(lds, WB)) + (uint32_t)w.wave * kept * 64u + lane;
    uint32_t* const counts = reinterpret_cast<uint32_t*>(part_lds(lds, WB)) + (blockDim.x >> 6) * kept * 64u + lane;
    SysParams<T> P;
    T xi[D];
    uint32_t cnt = 0;
    const uint32_t row_flag = nbr_row_flag(n);
    uint32_t row = row_flag;  // set until the row's first neighbour
    auto search = [&](auto&& put) {
        cnt = 0;
        row = row_flag;
        auto visit = [&](uint32_t j, const T*, T, bool shifted) {
            put(cnt, j | (shifted ? kNbrShift : 0u) | row);
            row = 0u;
            ++cnt;
        };
        neighbour_loop_staged<T, D, OFF32, 0>(P, xs, (const T*)nullptr, off, n, xi, visit,
                                              [&](int32_t) { row = row_flag; }, w.range, wave_window(lds, w.wave, WB));
    };
    if (s < n) {
        if (s == 0 && w.wave == 0) gen[1] = gen[0];  // the list now belongs to the latest build
        P = sp[b];
        load_point<T, D>(xs, s, xi);
        if (shared_rows) {
            search([&](uint32_t k, uint32_t e) {
                if (k < kept) stash[k * 64u] = e;
            });
        } else {
            uint32_t* p = nbr + s;
            search([&](uint32_t k, uint32_t e) {
                if (k < cap) {
                    *p = e;
                    p += n;
                }
            });
            nbr_count[s] = cnt <= cap ? cnt : kNbrOverflow;
        }
    }
    if (!shared_rows) return;
    counts[(uint32_t)w.wave * 64u] = cnt;
    __syncthreads();
    if (s >= n) return;
    uint32_t base = 0, total = 0;
    for (int32_t q = 0; q < split; ++q) {
        const uint32_t found = counts[(uint32_t)q * 64u];
        base += q < w.wave ? found : 0u;
        total += found;
    }
    const uint32_t mine = cnt;
    const bool listed = total <= cap;
    if (w.wave == 0) nbr_count[s] = listed ? total : kNbrOverflow;
    if (listed)
        for (uint32_t k = 0; k < min(mine, kept); ++k) nbr[(size_t)(base + k) * n + s] = stash[k * 64u];
    if (__ballot(listed && mine > kept) != 0ull)
        search([&](uint32_t k, uint32_t e) {
            if (k >= kept && listed) nbr[(size_t)(base + k) * n + s] = e;
        });
}

// Mean neighbour count of the densest system: its density times the volume of the cutoff
// ball.
double mean_neighbours(const aboria_cells* c) {
    double mu = 0.0;
    for (int32_t b = 0; b < c->nsys; ++b) {
        const aboria_box& bx = c->boxes[(size_t)b];
        const double nb = (double)(c->sys_off[(size_t)b + 1] - c->sys_off[(size_t)b]);
        double vol = 1.0;
        for (int k = 0; k < c->d; ++k) vol *= bx.hi[k] - bx.lo[k];
        const double r = bx.cutoff;
        const double ball = c->d == 1 ? 2.0 * r : (c->d == 2 ? M_PI * r * r : 4.0 / 3.0 * M_PI * r * r * r);
        if (vol > 0.0) mu = std::max(mu, nb / vol * ball);
    }
    return mu;
}

// Entries per particle: the mean neighbour count mu of a uniform system plus six standard
// deviations of a Poisson count and a margin.
uint32_t auto_capacity(const aboria_cells* c) {
    const double mu = mean_neighbours(c);
    const double want = std::ceil(mu + 6.0 * std::sqrt(mu) + 8.0);
    uint32_t cap = (uint32_t)std::min<double>(want, (double)kMaxNbrCap);
    cap = (cap + 7u) & ~7u;
    return std::max<uint32_t>(cap, 8u);
}

// Most waves of particles whose rows the recording shares: where the search waits more than
// it computes.  One wave / shared, us: 3000 particles in 2-d 16.3 / 8.6, 20000 in 3-d 58 /
// 19, 100003 64 / 50; 224000 in 2-d with 12 neighbours 23.5 / 21.4, with 100 233 / 148;
// 300007 in 2-d 33.5 / 34.6.  Of many neighbours in 3-d three waves find more than they
// keep and search twice (48 neighbours, 100003 particles 93 / 93, 150000 96 / 107, in
// float64 103 / 134; 224000 113 / 146); of few there is little to wait for (5 neighbours,
// 224000 in 2-d 13.0 / 15.9, in 3-d 29.5 / 31.9).
uint64_t shared_waves(const aboria_cells* c) {
    const double mu = mean_neighbours(c);
    return c->d == 3 && mu > 40.0 ? 1600 : (mu < 10.0 ? 2400 : 3500);
}

template <typename T, int D>
void launch_build_nbr(aboria_ctx* ctx, aboria_cells* c) {
    const uint32_t n = (uint32_t)c->n;
    const SysParams<T>* sp = reinterpret_cast<const SysParams<T>*>(c->params_dev);
    const int32_t split = ((uint64_t)n + 63) / 64 <= shared_waves(c) ? row_waves(c) : 0;
    const SearchShape sh = settle_search(
        n, split, [](int32_t sp) { return WindowBytes<T, D, 0>::value + stash_bytes(sp); },
        [](int32_t) { return 0u; }, lds_limit(ctx));
#define NB(B, O, S)                                                                                             \
    hipLaunchKernelGGL((k_nbr_build<T, D, B, O, S>), dim3(sh.blocks), dim3(sh.threads), sh.lds, ctx->stream,     \
                       (const T*)c->xs, c->off, n, sp, c->sys_part_dev, c->nsys, c->nbr, c->nbr_count, c->nbr_cap, \
                       c->gen, sh.split)
    const bool o32 = off32_rows<T>(n);
    if (c->nsys == 1) {
        if (sh.split > 0) NB(false, true, (D > 1)); else if (o32) NB(false, true, false); else NB(false, false, false);
    } else {
        if (sh.split > 0) NB(true, true, (D > 1)); else if (o32) NB(true, true, false); else NB(true, false, false);
    }
#undef NB
}

}  // namespace

}  // namespace aboria

using namespace aboria;

extern "C" aboria_status aboria_build_neighbours(aboria_ctx* ctx, aboria_cells* c, int32_t capacity) {
    if (!ctx) return ABORIA_ERR_INVALID_ARG;
    if (!c) return fail(ctx, ABORIA_ERR_INVALID_ARG, "cells is NULL");
    if (c->device != ctx->device) return fail(ctx, ABORIA_ERR_INVALID_ARG, "cells belong to another device");
    if (capacity < 0 || capacity > (int32_t)kMaxNbrCap)
        return fail(ctx, ABORIA_ERR_INVALID_ARG, "capacity must be in 0..4096");
    try {
        uint32_t cap = capacity > 0 ? (uint32_t)capacity : auto_capacity(c);
        if (c->nbr_count) {
            // the buffers are fixed once allocated (graphs may hold them)
            if (cap > (uint32_t)c->nbr_alloc) {
                if (capacity > 0)
                    return fail(ctx, ABORIA_ERR_INVALID_ARG,
                                "capacity exceeds the one the list of these cells was allocated with");
                cap = (uint32_t)c->nbr_alloc;
            }
        } else {
            if (ctx->capturing)
                return fail(ctx, ABORIA_ERR_UNSUPPORTED, "a first neighbour list allocates and cannot be captured");
            ABORIA_HIP(ctx, hipSetDevice(ctx->device));
            const size_t nn = (size_t)std::max<int64_t>(c->n, 1);
            if (hipMalloc((void**)&c->nbr, sizeof(uint32_t) * nn * cap) != hipSuccess ||
                hipMalloc((void**)&c->nbr_count, sizeof(uint32_t) * nn) != hipSuccess) {
                (void)hipGetLastError();
                if (c->nbr) (void)hipFree(c->nbr);
                if (c->nbr_count) (void)hipFree(c->nbr_count);
                c->nbr = c->nbr_count = nullptr;
                return fail(ctx, ABORIA_ERR_OUT_OF_MEMORY, "device allocation for the neighbour list failed");
            }
            c->nbr_alloc = cap;
        }
        c->nbr_cap = cap;
        if (c->n > 0) {
            if (c->dtype == ABORIA_F32) {
                switch (c->d) {
                    case 1: launch_build_nbr<float, 1>(ctx, c); break;
                    case 2: launch_build_nbr<float, 2>(ctx, c); break;
                    default: launch_build_nbr<float, 3>(ctx, c); break;
                }
            } else {
                switch (c->d) {
                    case 1: launch_build_nbr<double, 1>(ctx, c); break;
                    case 2: launch_build_nbr<double, 2>(ctx, c); break;
                    default: launch_build_nbr<double, 3>(ctx, c); break;
                }
            }
            ABORIA_HIP(ctx, hipGetLastError());
        }
        c->nbr_recorded = true;
        return ABORIA_OK;
    } catch (...) {
        return fail(ctx, ABORIA_ERR_OUT_OF_MEMORY, "host exception in build_neighbours");
    }
}

extern "C" int32_t aboria_neighbour_capacity(const aboria_cells* c) {
    return (c && c->nbr_recorded) ? (int32_t)c->nbr_cap : 0;
}
