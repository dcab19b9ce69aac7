"""The launch-shape rules (csrc/shape.h) on the host, compiled with the host
compiler: chunks within the 32-bit counters, and the default segment length at
the largest series its tile numbers admit."""
import os
import subprocess


CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2208_09136_amd", "csrc")
PROGRAM = r"""
#include "shape.h"
#include <cstdio>
using namespace rqa;
int main()
{
    for (uint64_t T = 64; T <= 65536; T += 64) {
        const uint64_t most = chunk_tiles_limit((uint32_t)T);
        if (most < 16 || most * 64 * T > 0xFFFFFFFFull || (most + 1) * 64 * T <= 0xFFFFFFFFull) return std::printf("chunk %lu\n", T);
    }
    // tiles counted one by one
    for (uint64_t L0 : {1, 63, 64, 65, 1000, 5003})
        for (uint64_t T : {64, 192, 320, 1024}) {
            uint64_t n = 0;
            for (uint64_t t0 = 0; t0 < L0; t0 += T) n += (L0 - t0 + 63) / 64;
            if (n != tile_count(L0, (uint32_t)T)) return std::printf("tiles %lu %lu\n", L0, T);
        }
    // series are refused where 1024 steps per segment give too many tiles, and
    // nowhere below, whatever the walker's unit
    const uint64_t longest = 16776640;
    if (tile_count(longest, 1024) >= MAX_TILES || tile_count(longest + 64, 1024) < MAX_TILES) return std::printf("limit\n");
    for (uint32_t tiles : {6u, 9u})
    for (uint32_t unit : {64u, 192u, 320u})
        for (int cus : {1, 64, 256})
            for (uint64_t L0 = 1; L0 <= longest + 64; L0 += L0 < 16200000 ? L0 / 50 + 1 : 64) {
                const uint32_t T = default_segment(L0, L0 * (L0 + 1) / 2, cus, unit, tiles);
                if (T < 64 || T > 1024 || T % 64) return std::printf("segment %u of %lu\n", T, L0);
                if ((tile_count(L0, T) < MAX_TILES) != (L0 <= longest)) return std::printf("refused %lu unit %u\n", L0, unit);
                if (L0 > 450000 && L0 < 16200000 && T != 1024 / unit * unit) return std::printf("unit %u of %lu\n", unit, L0);
            }
    std::printf("ok\n");
}
"""


def test_shape_rules(tmp_path):
    src, exe = tmp_path / "shape.cpp", tmp_path / "shape"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-I", CSRC, "-o", str(exe), str(src)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True).stdout
    assert out == "ok\n", out
