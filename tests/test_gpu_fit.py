"""The level fit against the oracle, bit for bit, where its kernel can go wrong: the smallest and largest bucket of each
launch shape, every table width, rounds that are not full, a short last batch, one batch only; batches that leave the
boundary search (levels that coincide, values crowded into few cells by an outlier, constant buckets) and counts past the
table of powers."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2302_02390_amd import binding as qb
from gpu_util import DEV, np_f32, synth

pytestmark = pytest.mark.gpu


def _same(v, bits, B, lr, levels, cap=0):
    lv = torch.from_numpy(levels.copy()).to(DEV)
    qb.qsdp_fit_levels(torch.from_numpy(v).to(DEV), bits, B, lr, lv, cap)
    want = ref.fit_levels(v, bits, B, lr, levels.copy(), max_batches=cap)
    return np.array_equal(np_f32(lv).view(np.uint32), want.view(np.uint32))


@pytest.mark.parametrize("B", [32, 96, 128, 160, 256, 288, 512, 544, 1024, 1056, 2048, 2080, 4096, 4128, 8192])
@pytest.mark.parametrize("batches,cut", [(1, 0), (1, 31), (6, 0), (7, 3), (26, 17)])
def test_shapes(B, batches, cut):
    x, g = synth(batches * B - cut, B + batches)
    for bits in range(1, 9):
        for v in (x, g):
            assert _same(v, bits, B, 0.01, ref.levels_uniform(bits)), (bits, B)


@pytest.mark.parametrize("B", [64, 1024, 2048, 8192])
@pytest.mark.parametrize("bits", [1, 2, 4, 5, 6, 7, 8])
def test_batches_without_a_boundary_search(B, bits):
    rng = np.random.default_rng(B + bits)
    n, K = 9 * B - 5, 1 << bits
    x, _ = synth(n, B)
    outlier = (1.0 + 1e-4 * rng.standard_normal(n)).astype(np.float32)  # crowded: all but one value per bucket
    outlier[::B] = 1e3
    constant = np.repeat(rng.standard_normal(9).astype(np.float32), B)[:n]
    two = np.where(rng.random(n) < 0.97, 0.25, -4.0).astype(np.float32)  # two values: most of a bucket on one level
    equal = ref.levels_uniform(bits)
    equal[-2] = 1.0
    close = np.float32(0.5) + np.arange(K, dtype=np.float32) * np.float32(2.0 ** -22)  # gaps below the search's bound
    for v in (x, outlier, constant, two):
        for levels in (ref.levels_uniform(bits), equal, close):
            assert _same(v, bits, B, 0.02, levels), (B, bits)


@pytest.mark.parametrize("B", [96, 128, 512, 1024, 4096])
@pytest.mark.parametrize("bits", [1, 3, 5, 6, 8])
def test_boundaries_among_the_last_values_of_a_batch(B, bits):
    """The consumer reads on past the cells of a boundary and past the batch: boundaries in the last cell, batches that
    end at, before and after a multiple of what it reads at once, seven to a round and one more."""
    rng = np.random.default_rng(B + bits)
    for cut in (0, 1, 3, 4, 8, 15, 16, 17):
        x = rng.beta(8.0, 1.0, 8 * B - cut).astype(np.float32)  # most of a bucket next to its maximum
        x[B - 1 - cut::B] = 1.0
        assert _same(x, bits, B, 0.05, ref.levels_uniform(bits)), cut
        high = np.sort(rng.uniform(0.9, 1.0, 1 << bits)).astype(np.float32)
        assert _same(x, bits, B, 0.05, high), cut


def test_offset_data_and_tensors_that_start_anywhere():
    B, bits, sizes = 1024, 5, [8, 40 * 1024 + 8, 1024, 24, 13 * 1024 + 40]
    x, g = synth(sum(sizes), 5)
    for v in (x, (g + 3.0).astype(np.float32)):
        segs = qb.Segments(sizes, B, DEV)
        levels = qb.levels_uniform(bits, DEV).repeat(len(sizes), 1).contiguous()
        qb.qsdp_fit_levels_segmented(torch.from_numpy(v).to(DEV), segs, bits, 0.01, levels, 30)
        o = 0
        for t, s in enumerate(sizes):
            want = ref.fit_levels(v[o:o + s].copy(), bits, B, 0.01, ref.levels_uniform(bits), max_batches=30)
            assert np.array_equal(np_f32(levels[t]).view(np.uint32), want.view(np.uint32)), t
            o += s


@pytest.mark.parametrize("m", [1, 63, 64, 65, 127, 128, 129, 192, 193, 1023, 1024, 1025, 1039, 1040, 1041, 1279, 1280,
                               1296, 2047, 2048, 4095, 4096, 8191, 8192])
def test_counts_where_the_table_of_powers_grows(m):
    """All m values of a batch on one level, then fewer, then half of them: the table is extended, used as it is, and
    read at its ends."""
    B = -(-m // 32) * 32
    v = np.full(3 * B, 0.5, np.float32)
    v[m:B], v[2 * B: 2 * B + B // 2] = 3.0, -1.0
    for bits in (1, 4, 8):
        for n in (m, 3 * B, 2 * B - 1):
            assert _same(v[:n].copy(), bits, B, 0.01, ref.levels_uniform(bits)), (bits, n)


@pytest.mark.parametrize("bits", [1, 3, 5, 8])
@pytest.mark.parametrize("B", [64, 1024, 4096])
def test_levels_without_values_stay_as_they_are(B, bits):
    """Bit for bit: a negative zero beside another one, and past [0, 1], where tables are not checked, padding."""
    x, _ = synth(5 * B, B + bits)
    K = 1 << bits
    if K > 2:
        levels = ref.levels_uniform(bits)
        levels[:2] = -0.0  # the values at the minimum go to the first of the two
        assert _same(x, bits, B, 0.01, levels, 1)
    for fill in (np.inf, 3e38, 2.5):
        levels = ref.levels_uniform(bits)
        levels[K // 2:] = fill
        lv = torch.from_numpy(levels).to(DEV)
        qb.qsdp_fit_levels(torch.from_numpy(x).to(DEV), bits, B, 0.01, lv)
        got = np_f32(lv)
        assert np.array_equal(got[K // 2:], levels[K // 2:]) and (got[:K // 2] < 1.0).all(), fill


@pytest.mark.parametrize("B", [96, 128, 512, 1024, 1056, 2048])
@pytest.mark.parametrize("bits", [1, 4, 5, 6, 8])
def test_sums_before_the_groups_of_a_batch(B, bits):
    """The kernel keeps count and sum before every fourth value of the sorted batch, short by the values that are exactly
    1 except in the word of all: many of them, in several of its rows, in batches that end inside a group; and cells that
    an outlier outside the sample which places them makes so narrow that 1 is not in the last one."""
    rng = np.random.default_rng(B + bits)
    for cut in (0, 1, 2, 3, 30):
        n = 17 * B - cut
        top = rng.uniform(0.0, 1.0, n).astype(np.float32)
        top[rng.random(n) < 0.4] = 1.0
        top[::B] = 0.0
        crest = (1.0 - rng.random(n) * 1e-4).astype(np.float32)
        crest[70 % B::B] = -30.0
        crest[71 % B::B] = 1.0
        far = rng.uniform(0.0, 0.1, n).astype(np.float32)
        far[70 % B::B] = -2.0e4
        for v in (top, crest, far):
            assert _same(v, bits, B, 0.03, ref.levels_uniform(bits)), cut


def _steep_ranges(rng):
    """Ranges whose reciprocal is subnormal and rounds up, so that the largest normalised value is past 1."""
    r = rng.uniform(2.0 ** 126, 3.39e38, 4000).astype(np.float32)
    r = r[r * (np.float32(1.0) / r) > np.float32(1.0)]
    assert r.size > 400
    return r


@pytest.mark.parametrize("B", [32, 96, 128, 256, 512, 1024, 2048, 4096, 8192])
@pytest.mark.parametrize("bits", [1, 3, 4, 5, 6, 8])
def test_normalised_values_past_one(B, bits):
    """Finite buckets with a range above 2^126, where the largest normalised value can be 1 + 2^-23 or 1 + 2^-22: its
    excess enters the sums, on the way of the boundaries and value by value, and takes the last level past 1, from where
    later batches start."""
    rng = np.random.default_rng(B + bits)
    ranges = _steep_ranges(rng)
    K = 1 << bits
    close = (1.0 - 2.0 ** -22 * np.arange(K, dtype=np.float64)[::-1]).astype(np.float32)  # gaps below the search's bound
    past = False
    for cut in (0, 1, 30):
        n = 13 * B - cut
        v = np.empty(n, np.float32)
        for j in range(13):
            b = v[j * B: (j + 1) * B]
            r = ranges[rng.integers(ranges.size)]
            lo, hi = -r * np.float32(0.5), r * np.float32(0.5)  # exact, and so is their difference
            share = (0.3, 1.0, 0.02)[j % 3]
            b[:] = np.where(rng.random(b.size) < share, hi, (rng.random(b.size) * r + lo).astype(np.float32))
            b[0], b[-1] = lo, hi
            assert (hi - lo) * (np.float32(1.0) / (hi - lo)) > np.float32(1.0)
        ordinary = v.copy()
        ordinary[7 * B:] = rng.standard_normal(n - 7 * B).astype(np.float32)  # later batches within [0, 1]
        for x in (v, ordinary):
            for levels in (ref.levels_uniform(bits), close):
                past |= bool((ref.fit_levels(x, bits, B, 0.3, levels.copy(), max_batches=2) > 1.0).any())
                assert _same(x, bits, B, 0.3, levels), cut
    assert past
