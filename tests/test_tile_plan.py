"""The tile kernels' launch shapes (csrc/qsdp_tile_plan.hpp, plain C++) for every bucket size, compiled and checked
without a GPU: whole buckets fit the team, every bucket has lanes of its own, and the two multiplications that stand
for divisions are exact over the ranges the kernel uses them on; small calls and tensors with tables of their own get
small tiles; the buckets of the GPU tests see every shape."""
import subprocess

from paper_2302_02390_amd import build as lib_build

SOURCE = r"""
#include "qsdp_tile_plan.hpp"
#include <cstdio>
#include <initializer_list>
using namespace qsdp;
static int bad = 0;
static void check(const TilePlan& t, int k, bool as_many_as_fit) {
    const int groups = tile_groups(t.waves, t.rows), lanes = 1 << t.lanes_log2;
    const bool shape = (t.waves == 1 || t.waves == 4) && t.rows % 2 == 0 && t.rows >= 2 && t.rows <= kTileMaxRows;
    if (!shape || t.buckets < 1 || t.buckets * k > groups) ++bad;
    if (as_many_as_fit && (t.buckets + 1) * k <= groups) ++bad;
    if (t.buckets * lanes > 64 * t.waves || lanes > 64 || t.buckets > 64 * t.waves) ++bad;
    for (int i = 0; i < groups; ++i)
        if ((int)((uint32_t)i * t.group_magic >> 16) != i / k) ++bad;
}
int main(int argc, char** argv) {
    const uint64_t any = ~0ull;
    for (int k = 1; k <= 256; ++k) {
        check(tile_plan(32 * k), k, true);
        const TilePlan s = tile_plan_small(32 * k);
        check(s, k, false);
        if (s.buckets > 1 && s.buckets * k > tile_groups(s.waves, 1)) ++bad;  // one row, or one bucket ...
        // ... or all that fit
        if (tile_groups(s.waves, 1) < k && (s.buckets + 1) * k <= tile_groups(s.waves, s.rows)) ++bad;
        for (const uint64_t mean : {0ull, 1ull, 2ull, 3ull, 7ull, 40ull, 1000ull}) {
            const TilePlan t = tile_plan_tensors(32 * k, mean);
            check(t, k, false);
            if ((uint64_t)t.buckets > (mean > 0 ? mean : 1)) ++bad;
        }
        // the line between small and large calls, and a launch that is capped
        const uint64_t most = 4095 / s.waves * (uint64_t)s.buckets;
        const TilePlan below = choose_tile(32 * k, most, 0, any);
        if (below.rows != s.rows || below.waves != s.waves || below.buckets != s.buckets) ++bad;
        const TilePlan f = tile_plan(32 * k), l = choose_tile(32 * k, most + 4 * (uint64_t)s.buckets, 0, any);
        if (l.rows != f.rows || l.waves != f.waves || l.buckets != f.buckets) ++bad;
        const TilePlan c = choose_tile(32 * k, 8 * (uint64_t)s.buckets, 0, 8);
        if (c.rows != f.rows || c.waves != f.waves || c.buckets != f.buckets) ++bad;
        // tables per tensor: never more buckets to a tile than to the mean tensor
        for (const uint64_t tensors : {1ull, 10ull, 999ull})
            if ((uint64_t)choose_tile(32 * k, 1000, tensors, any).buckets > 1000 / tensors) ++bad;
    }
    for (int bits = 1; bits <= 8; ++bits)
        for (uint32_t w = 0; w < 2048u * bits / 8; ++w)
            if ((8 * w * word_magic(bits)) >> 18 != 8 * w / bits) ++bad;
    std::printf("%d", bad);
    for (int i = 1; i < argc; ++i) {  // shapes of some buckets: large calls, small ones, tensors
        int b;
        std::sscanf(argv[i], "%d", &b);
        for (const TilePlan& t : {tile_plan(b), tile_plan_small(b), tile_plan_tensors(b, 1)})
            std::printf(" %d,%d", t.waves, t.rows);
    }
    return bad != 0;
}
"""


def test_every_bucket_size_has_an_exact_plan(tmp_path):
    from test_gpu_tile import BUCKETS, RECEIVE_BUCKETS
    from test_gpu_random_parity import TILE_BUCKETS
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", lib_build.CSRC, str(src), "-o", str(exe)], check=True)
    for buckets in (BUCKETS, RECEIVE_BUCKETS, TILE_BUCKETS):
        run = subprocess.run([str(exe)] + [str(b) for b in buckets], capture_output=True, text=True)
        bad, *shapes = run.stdout.split()
        assert run.returncode == 0 and bad == "0"
        assert set(shapes) == {f"{w},{r}" for w, r in lib_build.TILE_SHAPES}


CALL_SOURCE = r"""
#include "qsdp_tile_plan.hpp"
#include <cstdio>
using namespace qsdp;
int main() {
    int bad = 0, half = 0, six = 0;
    for (int k = 1; k <= 256; ++k)
        for (int work = 0; work < 3; ++work)
            for (uint64_t nb = 1; nb * k < (1u << 20); nb = nb * 5 / 4 + 1) {
                const TilePlan t = choose_step_tile(32 * k, nb, ~0ull, (TileWork)work, 0), f = tile_plan(32 * k);
                const int groups = tile_groups(t.waves, t.rows);
                if (t.buckets < 1 || t.buckets * k > groups || (t.buckets << t.lanes_log2) > 64 * t.waves) ++bad;
                for (int i = 0; i < groups; ++i)
                    if ((int)((uint32_t)i * t.group_magic >> 16) != i / k) ++bad;
                if (t.waves == 4 && t.rows == 2 && t.buckets == groups / k) ++half;
                if (work == TILE_INSTRUCTIONS && f.rows == 4 && t.rows == 6 && t.waves == 4) ++six;
                // few workgroups: the tiles of large calls
                const TilePlan c = choose_step_tile(32 * k, 1000000, 8, (TileWork)work, 0);
                if (work != TILE_INSTRUCTIONS && (c.rows != f.rows || c.waves != f.waves)) ++bad;
            }
    std::printf("%d %d", half, six);
    return bad != 0;
}
"""


def test_tile_plan_of_a_call(tmp_path):
    """Every tile of a call is a valid plan, the two that only some calls take among them."""
    src, exe = tmp_path / "call.cpp", tmp_path / "call"
    src.write_text(CALL_SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", lib_build.CSRC, str(src), "-o", str(exe)], check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    half, six = map(int, run.stdout.split())
    assert run.returncode == 0 and half > 100 and six > 100


TENSORS_SOURCE = r"""
#include "qsdp_tile_plan.hpp"
#include <cstdio>
using namespace qsdp;
int main() {
    int bad = 0, fewer = 0, six = 0;
    for (int k = 1; k <= 256; ++k)
        for (int work = 0; work < 3; ++work)
            for (uint64_t nb = 1; nb * k < (1u << 23); nb = nb * 5 / 4 + 1)
                for (uint64_t tensors = 1; tensors <= nb; tensors *= 4) {
                    const TilePlan t = choose_step_tile(32 * k, nb, ~0ull, (TileWork)work, tensors);
                    const TilePlan plain = choose_tile(32 * k, nb, 0, ~0ull);
                    const bool same = t.waves == plain.waves && t.rows == plain.rows && t.buckets == plain.buckets;
                    const bool large = nb / tensors >= 512 * (uint64_t)t.buckets && 32 * nb * k >= (24u << 20);
                    if (!same && t.buckets >= plain.buckets && !(work == TILE_INSTRUCTIONS && large)) ++bad;
                    fewer += t.buckets < plain.buckets;
                    six += t.buckets > plain.buckets;
                }
    std::printf("%d %d", fewer, six);
    return bad != 0;
}
"""


def test_tile_plan_of_a_multi_tensor_call(tmp_path):
    """Tiles that meet tensors' ends are slow: such calls take no tiles of more buckets than the general rule's, but for
    gradients of a few large tensors."""
    src, exe = tmp_path / "tensors.cpp", tmp_path / "tensors"
    src.write_text(TENSORS_SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", lib_build.CSRC, str(src), "-o", str(exe)], check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    fewer, six = map(int, run.stdout.split())
    assert run.returncode == 0 and fewer > 100 and six > 5


STREAM_SOURCE = r"""
#include "qsdp_tile_plan.hpp"
#include <initializer_list>
using namespace qsdp;
static bool three(int bucket, uint64_t n, bool tensors = false, bool half = false, int bits = 8, bool lattice = false) {
    const TilePlan t = tile_plan(bucket);
    return three_workgroups_stream(bucket, t.buckets, t.waves, t.rows, n, tensors, half, bits, lattice);
}
int main() {
    const uint64_t large = 3ull << 25;
    int bad = 0;
    for (int bucket : {384, 608, 768, 864, 1184, 1536, 2944, 3008, 3040, 5952, 6016, 6048, 6144}) {
        bad += !three(bucket, large) + three(bucket, large - 1) + three(bucket, large, true);
        bad += three(bucket, large, false, true) + three(bucket, large, false, false, 0);
        bad += three(bucket, large, false, false, 4) + three(bucket, large, false, false, 8, true);
    }
    for (int bucket : {736, 1472, 1504}) bad += three(bucket, (1ull << 27) - 1) + !three(bucket, 1ull << 27);
    for (int bucket : {32, 160, 224, 288, 416, 704, 800, 2016, 2080, 4128, 4992, 8192})
        bad += three(bucket, large) + three(bucket, 1ull << 28);
    return bad != 0;
}
"""


def test_large_steps_in_full_tiles_run_three_workgroups(tmp_path):
    """... and no others: not over tensors, in tiles that are less full, on smaller vectors or with other outputs."""
    src, exe = tmp_path / "stream.cpp", tmp_path / "stream"
    src.write_text(STREAM_SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", lib_build.CSRC, str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)]).returncode == 0


SIZES_SOURCE = r"""
#include "qsdp_tile_plan.hpp"
#include <initializer_list>
using namespace qsdp;
static bool takes(int waves, int rows, int bucket, uint64_t n, TileWork work, uint64_t tensors = 0) {
    const TilePlan t = choose_step_tile(bucket, (n + bucket - 1) / bucket, ~0ull, work, tensors);
    return t.waves == waves && t.rows == rows && t.buckets == tile_groups(waves, rows) / (bucket / 32);
}
int main() {
    int bad = 0;
    for (int bucket : {96, 160, 416, 768}) bad += !takes(4, 2, bucket, 1 << 19, TILE_MEMORY);
    for (int bucket : {32, 1504}) bad += !takes(4, 2, bucket, 5 << 18, TILE_MEMORY);
    for (int bucket : {96, 160, 416, 768, 1504}) bad += !takes(4, 2, bucket, 1 << 22, TILE_ADAMW);
    for (int bucket : {32, 160, 544}) bad += !takes(4, 6, bucket, 7 << 20, TILE_INSTRUCTIONS);
    bad += !takes(4, 2, 416, 1 << 21, TILE_MEMORY, 100);
    for (int bucket : {32, 160, 544}) bad += !takes(4, 6, bucket, 9 << 22, TILE_INSTRUCTIONS, 3);
    return bad;
}
"""


def test_sizes_that_take_the_tiles_of_their_own(tmp_path):
    """The calls of test_gpu_tile_calls.py are of these sizes (32 with 2^19 elements takes a smaller tile)."""
    src, exe = tmp_path / "sizes.cpp", tmp_path / "sizes"
    src.write_text(SIZES_SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", lib_build.CSRC, str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)]).returncode == 0
