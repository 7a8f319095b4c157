"""Launch sizes (launch_shape.h, host arithmetic) built with g++."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2207_05009_amd", "csrc")


def _run(tmp_path, program):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("needs g++")
    src, exe = tmp_path / "shape.cpp", tmp_path / "shape"
    src.write_text(program)
    subprocess.run([gxx, "-std=c++17", "-O2", "-Wall", "-Werror", f"-I{CSRC}", "-o", str(exe), str(src)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout == "ok\n", out.stdout


def test_streaming_launches_fit_a_grid_and_cover_every_word(tmp_path):
    """Every admitted tree (up to 2^30 leaves of 16 to 128 words): fewer than
    2^32 threads, all words reached, and a thread per word where that fits."""
    _run(tmp_path, r"""
#include "launch_shape.h"
#include <cstdio>
int main() {
    using namespace lq;
    const uint64_t leaves[] = {0, 1, 15, 16, 17, 882000, 33554431, 33554432, 56512728, 134217728, 1ull << 30};
    const uint64_t per_leaf[] = {1, 4, 13, 16, 28, 32, 64, 76, 128};
    for (uint64_t n : leaves)
        for (uint64_t words : per_leaf) {
            const uint64_t items = n * words, blocks = stream_blocks(items), threads = blocks * kStreamThreads;
            if (blocks < 1 || threads >= 1ull << 32) { std::printf("%llu items: %llu blocks\n", (unsigned long long)items, (unsigned long long)blocks); return 1; }
            if (items <= 1ull << 30 && threads < items) { std::printf("%llu items: not a thread each\n", (unsigned long long)items); return 1; }
            if (threads >= items + kStreamThreads && blocks > 1) { std::printf("%llu items: idle blocks\n", (unsigned long long)items); return 1; }
        }
    std::printf("ok\n");
    return 0;
}
""")


def test_slices_stay_within_their_bytes_and_cover_every_leaf(tmp_path):
    _run(tmp_path, r"""
#include "launch_shape.h"
#include <cstdio>
int main() {
    using namespace lq;
    const uint64_t leaves[] = {0, 1, 2, 100, 55188, 882000, 16777216, 16777217, 1ull << 30}, bytes[] = {4, 12, 108, 300, 304};
    for (uint64_t n : leaves)
        for (uint64_t b : bytes) {
            const uint64_t m = slice_leaves(n, b);
            if (m < 1 || m * b > kSliceBytes || (n && m > n) || (n * b <= kSliceBytes && n && m != n)) {
                std::printf("%llu leaves of %llu: %llu\n", (unsigned long long)n, (unsigned long long)b, (unsigned long long)m);
                return 1;
            }
        }
    std::printf("ok\n");
    return 0;
}
""")


def test_resident_blocks_are_a_kernels_own(tmp_path):
    """Kernels of one signature and of different occupancy, in either order, on
    two devices; each is asked for once."""
    _run(tmp_path, r"""
#include "launch_shape.h"
#include <cstdio>
static void a(int) {}
static void b(int) {}
int main() {
    using namespace lq;
    for (int order = 0; order < 2; ++order) {
        ResidentBlocks known;
        int asked = 0;
        for (int k = 0; k < 6; ++k) {
            const bool first = (k + order) % 2 == 0;
            const int device = k / 4, want = (first ? 1280 : 768) + device;
            const void *kern = reinterpret_cast<const void *>(first ? a : b);
            const int got = known.get(device, kern, [&] { ++asked; return want; });
            if (got != want) { std::printf("order %d, call %d: %d\n", order, k, got); return 1; }
        }
        if (asked != 4) { std::printf("asked %d times\n", asked); return 1; }
    }
    std::printf("ok\n");
    return 0;
}
""")


def test_camera_reservations_are_whole_tiles(tmp_path):
    """The ranges of a camera batch, reserved 64 positions at a time: they cover
    every position once, and each reservation starts on a tile, so that only the
    last one of the batch holds fewer than 64; and the ranges of other batches."""
    _run(tmp_path, r"""
#include "launch_shape.h"
#include <cstdio>
int main() {
    using namespace lq;
    const int64_t sizes[] = {1, 7, 63, 64, 65, 511, 512, 513, 1283 * 721, 2048 * 2048, 2147483647, (int64_t)1 << 40};
    for (int64_t n : sizes)
        for (int64_t unit = 1; unit <= 64; unit += 63) {
            int64_t at = 0;
            for (int x = 0; x < 8; ++x) {
                const int64_t a = range_begin(x, 8, n, unit), b = range_begin(x + 1, 8, n, unit);
                if (a != at || b < a || a % unit || b - a > n / 8 + 2 * unit) { std::printf("%lld, unit %lld, range %d\n", (long long)n, (long long)unit, x); return 1; }
                at = b;
            }
            if (at != n) { std::printf("%lld ends at %lld\n", (long long)n, (long long)at); return 1; }
        }
    std::printf("ok\n");
    return 0;
}
""")
