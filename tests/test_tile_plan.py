"""The tile kernels' launch shapes (csrc/qsdp_tile_plan.hpp, plain C++) for every bucket size, compiled and checked
without a GPU: whole buckets fit the team, every bucket has lanes of its own, and the two multiplications that stand
for divisions are exact over the ranges the kernel uses them on."""
import subprocess

from paper_2302_02390_amd import build as lib_build

SOURCE = r"""
#include "qsdp_tile_plan.hpp"
#include <cstdio>
using namespace qsdp;
int main() {
    int bad = 0;
    for (int k = 1; k <= 256; ++k) {
        const TilePlan t = tile_plan(32 * k);
        const int groups = tile_groups(t.waves, t.rows), lanes = 1 << t.lanes_log2;
        const bool shape = (t.waves == 1 || t.waves == 4) && t.rows % 2 == 0 && t.rows >= 2 && t.rows <= kTileMaxRows;
        if (!shape || t.buckets < 1 || t.buckets * k > groups || (t.buckets + 1) * k <= groups) ++bad;
        if (t.buckets * lanes > 64 * t.waves || lanes > 64 || t.buckets > 64 * t.waves) ++bad;
        for (int i = 0; i < groups; ++i)
            if ((int)((uint32_t)i * t.group_magic >> 16) != i / k) ++bad;
    }
    for (int bits = 1; bits <= 8; ++bits)
        for (uint32_t w = 0; w < 2048u * bits / 8; ++w)
            if ((8 * w * word_magic(bits)) >> 18 != 8 * w / bits) ++bad;
    std::printf("%d\n", bad);
    return bad != 0;
}
"""


def test_every_bucket_size_has_an_exact_plan(tmp_path):
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", lib_build.CSRC, str(src), "-o", str(exe)], check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0 and run.stdout.strip() == "0"
