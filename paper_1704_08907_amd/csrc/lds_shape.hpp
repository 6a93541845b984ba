// Launch shapes that a device's LDS limit decides, as the host settles them before it
// launches.  Kernels lay their LDS out from the settled values alone (the split a search
// was launched with, a bucket's cap).  Plain C++, so that it can be checked without a GPU.
#pragma once

#include <stdint.h>

namespace aboria {

// A box search: `split` waves share the rows of 64 particles (0: a running sum, 1: row sums
// by one wave), in workgroups of `threads` with `lds` bytes.
struct SearchShape {
    int32_t split;
    uint32_t blocks, threads, lds;
};

// The shape of a search of n particles by at most `split` waves per 64, where a wave of a
// search split s ways needs wave_bytes(s) of LDS and its workgroup part_bytes(s) beside:
// fewer waves (the same sums) where theirs would not fit a workgroup's limit.
template <typename WaveBytes, typename PartBytes>
constexpr SearchShape settle_search(uint64_t n, int32_t split, WaveBytes wave_bytes, PartBytes part_bytes,
                                    uint32_t limit) {
    const uint32_t waves = (uint32_t)((n + 63) / 64);
    auto lds = [=](int32_t s) { return (uint32_t)s * wave_bytes(s) + part_bytes(s); };
    if (split > 3 && lds(split) > limit) split = 3;
    if (split > 1 && lds(split) > limit) split = 1;
    if (split <= 1) return SearchShape{split, (waves + 3) / 4, 256, 4 * wave_bytes(split)};
    return SearchShape{split, waves, 64u * (uint32_t)split, lds(split)};
}

// Neighbour list recording with shared rows: entries of its rows that a lane keeps in LDS
// before it knows their place in the list (a row of the 3-d stencil has a ninth of the
// neighbours, three have a third), and a wave's bytes for them and their counts.
constexpr uint32_t stash_of(int32_t split) { return split > 3 ? 16u : 32u; }
constexpr uint32_t stash_bytes(int32_t split) { return split > 1 ? (stash_of(split) + 1u) * 256u : 0u; }

// Small builds: the 16 waves' counts of 2^low_bits cells, beside a wave's total each.
constexpr uint32_t small_build_lds(int32_t low_bits) { return 16u * (4u << low_bits); }
constexpr bool small_build_fits(int32_t low_bits, uint32_t limit) { return small_build_lds(low_bits) + 64u <= limit; }

// Counts of a bucket pass of 2^low_bits cells by `threads` threads.
constexpr uint32_t bucket_counts(int32_t low_bits, uint32_t threads) { return (2u + threads / 64u) * (4u << low_bits); }

}  // namespace aboria
