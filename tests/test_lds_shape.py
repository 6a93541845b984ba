"""The launch shapes that depend on a device's LDS limit, compiled by the host compiler:
whatever a search is settled to, its LDS holds what its kernel lays out, under any limit."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1704_08907_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "lds_shape.hpp"
using namespace aboria;
int bad = 0;
static void need(bool ok, const char* what, int a, unsigned b, unsigned c) {
    if (!ok) { std::printf("%s %d %u %u\n", what, a, b, c); bad = 1; }
}
int main() {
    const uint32_t limits[] = {32768u, 65536u, 98304u, 163840u};
    const uint32_t windows[] = {512u, 1024u, 2048u, 4096u, 8192u};  // 128 rows of 4 to 64 bytes
    for (uint32_t limit : limits)
        for (uint32_t w : windows)
            for (int split : {0, 1, 3, 9}) {
                // list recording: a window, the stash and the counts of each wave, laid out by the settled split
                const SearchShape r = settle_search(40000, split, [=](int32_t s) { return w + stash_bytes(s); },
                                                    [](int32_t) { return 0u; }, limit);
                const uint32_t waves = r.threads / 64u;
                const uint32_t kernel = waves * w + (r.split > 1 ? waves * stash_of(r.split) * 256u + waves * 256u : 0u);
                need(r.split <= 1 || (int)waves == r.split, "waves", split, w, limit);
                need(kernel <= r.lds, "recording", split, w, limit);
                need(r.lds <= limit || r.split <= 1, "recording limit", split, w, limit);
                // sums: windows and the rows' sums of all waves but the first (256 to 3584 bytes a row)
                for (uint32_t row : {256u, 512u, 1792u, 3584u}) {
                    auto part = [=](int32_t s) { return s > 1 ? (9u - 9u / s) * row : 0u; };
                    const SearchShape s = settle_search(40000, split, [=](int32_t) { return w; }, part, limit);
                    need(s.lds >= (s.threads / 64u) * w + part(s.split), "sums", split, w, limit);
                    need(s.lds <= limit || s.split <= 1, "sums limit", split, w, limit);
                    need((uint64_t)s.blocks * (s.split > 1 ? 64u : 256u) >= 40000u, "blocks", split, w, limit);
                }
            }
    for (int bits = 1; bits <= 10; ++bits)
        for (uint32_t limit : limits)
            need(!small_build_fits(bits, limit) || 16u * (1u << bits) * 4u + 16u * 4u <= limit, "small", bits, limit, 0);
    need(!small_build_fits(10, 65536u) && small_build_fits(10, 163840u), "small edge", 10, 0, 0);
    need(bucket_counts(10, 1024) == 73728u && bucket_counts(10, 512) == 40960u, "bucket", 10, 0, 0);
    return bad;
}
"""


def test_settled_shapes_hold_what_kernels_lay_out(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src = tmp_path / "t.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "t"
    subprocess.run([cxx, "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
