"""The learned-level encoders against the oracle, bit for bit, on the tables that decide how a value is looked up: evenly spread,
denser in the middle, crowded (two bounds in one cell), runs of equal levels (inside, at both ends, all of them), gaps too
small for exact thresholds, tables that do not reach 0 or 1; values on the levels and on the midpoints themselves."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2302_02390_amd import binding as qb
from gpu_util import DEV, np_u32, synth

pytestmark = pytest.mark.gpu


def _tables(bits, rng):
    K = 1 << bits
    uniform = ref.levels_uniform(bits)
    u = 2 * uniform.astype(np.float64) - 1
    inside = uniform.copy()
    inside[K // 2 - 1:K // 2 + 1] = inside[K // 2]
    ends = uniform.copy()
    ends[:max(1, K // 4)] = 0.0
    ends[-max(1, K // 4):] = 1.0
    return [uniform, (0.5 + 0.5 * (0.4 * u + 0.6 * u ** 3)), 0.25 + 0.5 * uniform, np.sort(rng.random(K)) ** 6, inside, ends,
            np.full(K, 0.5), 0.5 + np.arange(K) * 2.0 ** -24, np.sort(rng.integers(0, max(2, K // 2), K)) / K]


def _values(n, B, table, rng):
    """Gaussian values; every other bucket spans exactly [0, 1] and holds levels, midpoints and their neighbours."""
    x, _ = synth(n, B)
    picks = np.concatenate([table, (table[1:] + table[:-1]) / 2]).astype(np.float32)
    picks = np.concatenate([picks, np.nextafter(picks, np.float32(2)), np.nextafter(picks, np.float32(-2))]).clip(0, 1)
    for o in range(0, n, 2 * B):
        m = min(B, n - o)
        x[o:o + m] = rng.choice(picks, m)
        x[o], x[o + m - 1] = 0.0, 1.0
    return x


@pytest.mark.parametrize("B", [32, 96, 128, 256, 512, 608, 1024, 2048, 2080, 4096, 8192])
@pytest.mark.parametrize("bits", range(1, 9))
def test_tables(bits, B):
    rng = np.random.default_rng(100 * bits + B)
    n = 7 * B + B // 2 + 3
    for table in _tables(bits, rng):
        table = np.ascontiguousarray(table, dtype=np.float32)
        x = _values(n, B, table, rng)
        xd, td = torch.from_numpy(x).to(DEV), torch.from_numpy(table).to(DEV)
        codes, meta = qb.alloc_packed(n, bits, B, DEV)
        qb.qsdp_quantize_levels(xd, bits, B, td, codes, meta.view(-1))
        wc, wm = ref.quantize_levels(x, bits, B, table)
        assert np.array_equal(np_u32(codes), wc) and np.array_equal(np_u32(meta), wm.view(np.uint32).reshape(-1))
        qb.qsdp_quantize_levels_stochastic(xd, bits, B, td, 3, 8, codes, meta.view(-1))
        wc, wm = ref.quantize_levels_stochastic(x, bits, B, table, 3, index_offset=8)
        assert np.array_equal(np_u32(codes), wc) and np.array_equal(np_u32(meta), wm.view(np.uint32).reshape(-1))


@pytest.mark.parametrize("grid", [None, "1", "7"])
@pytest.mark.parametrize("B", [96, 128, 512, 608, 1024, 2048, 2080, 4096])
@pytest.mark.parametrize("bits", [3, 5, 7])
def test_workgroups_that_cross_tensors(bits, B, grid, monkeypatch):
    """Runs of buckets with several tensors in them, each with another kind of table, also with few workgroups."""
    if grid is not None:
        monkeypatch.setenv("QSDP_DEBUG_MAXGRID", grid)
    rng = np.random.default_rng(bits + B)
    tables = [np.ascontiguousarray(t, dtype=np.float32) for t in _tables(bits, rng)]
    sizes = [B, 8, 5 * B + 16, 40, 33 * B, 2 * B + 8, 3 * B, 16, 19 * B + 24]
    segs = qb.Segments(sizes, B, DEV)
    xs = [_values(s, B, t, rng) for s, t in zip(sizes, tables)]
    xd, td = torch.from_numpy(np.concatenate(xs)).to(DEV), torch.from_numpy(np.stack(tables)).to(DEV)
    for coin in (False, True):
        codes, meta = segs.alloc_packed(bits)
        qb.qsdp_quantize_levels_segmented(xd, segs, bits, td, codes, meta.view(-1), coin, 4, 16)
        wc, wm, o = [], [], 0
        for x, t in zip(xs, tables):
            c, m = (ref.quantize_levels_stochastic(x, bits, B, t, 4, index_offset=16 + o) if coin
                    else ref.quantize_levels(x, bits, B, t))
            wc.append(c)
            wm.append(m.view(np.uint32).reshape(-1))
            o += x.size
        assert np.array_equal(np_u32(codes), np.concatenate(wc)) and np.array_equal(np_u32(meta), np.concatenate(wm))


def _same_bits(codes, want_codes, meta, want_meta):
    return (np.array_equal(np_u32(codes), want_codes)
            and np.array_equal(np_u32(meta), want_meta.view(np.uint32).reshape(-1)))


@pytest.mark.parametrize("B", [96, 128, 608, 1024, 2048, 2080, 4096])
@pytest.mark.parametrize("bits", [1, 2, 5, 6, 8])
def test_coin_flip_in_gaps_next_to_zero(bits, B):
    """The smallest gaps that binary32 has (only levels next to 0 can be that close): values all over such a gap."""
    rng = np.random.default_rng(bits + B)
    n = 4 * B
    for exponent in (100, 119, 121, 123, 125, 127, 129, 134):
        gap = np.float32(np.ldexp(1.0, -exponent))
        table = ref.levels_uniform(bits)
        table[1] = gap
        x = rng.random(n).astype(np.float32) * gap
        x[0::B], x[B - 1::B] = 0.0, 1.0
        codes, meta = qb.alloc_packed(n, bits, B, DEV)
        qb.qsdp_quantize_levels_stochastic(torch.from_numpy(x).to(DEV), bits, B, torch.from_numpy(table).to(DEV), 3, 8,
                                           codes, meta.view(-1))
        wc, wm = ref.quantize_levels_stochastic(x, bits, B, table, 3, index_offset=8)
        assert _same_bits(codes, wc, meta, wm), exponent


@pytest.mark.parametrize("B", [96, 128, 608, 1024, 2080, 4096])
@pytest.mark.parametrize("bits", [2, 4, 6, 8])
def test_nearest_level_among_close_levels(bits, B):
    """Two neighbours a few steps apart, anywhere in the table: values all over, on the pair and between."""
    K, n = 1 << bits, 6 * B
    for k, top in ((0, 1.0), (K // 2 - 1, 1.0), (K // 3, 1.0), (K - 2, 1.0), (K - 2, 0.5), (K - 2, 0.999)):
        for gap in (2.0 ** -19, 2.0 ** -21, 2.0 ** -23):
            rng = np.random.default_rng(bits + B + k)
            table = (ref.levels_uniform(bits) * np.float32(top)).astype(np.float32)
            if k == K - 2:
                table[k] = table[k + 1] - np.float32(gap)
            else:
                table[k + 1] = table[k] + np.float32(gap)
            x = rng.random(n).astype(np.float32)
            near = np.arange(n) % 3 == 0
            x[near] = np.clip(table[k] + (rng.integers(-6, 7, near.sum()) * gap / 4), 0, 1).astype(np.float32)
            x[0::B], x[B - 1::B] = 0.0, 1.0
            codes, meta = qb.alloc_packed(n, bits, B, DEV)
            qb.qsdp_quantize_levels(torch.from_numpy(x).to(DEV), bits, B, torch.from_numpy(table).to(DEV), codes,
                                    meta.view(-1))
            wc, wm = ref.quantize_levels(x, bits, B, table)
            assert _same_bits(codes, wc, meta, wm), (k, gap)


@pytest.mark.parametrize("stochastic", [False, True])
@pytest.mark.parametrize("B,tensors", [(32, 1500), (128, 40), (128, 1400), (512, 1400), (608, 300), (1024, 1300),
                                       (2080, 50), (4096, 20)])
def test_tensors_of_a_bucket_or_two(B, tensors, stochastic):
    """A table each: as many workgroups as tensors, small tiles, past 1280 small tensors the tile kernel for all."""
    rng = np.random.default_rng(B + tensors)
    for most, bits in ((1, 4), (2, 7)):
        sizes = [8 * int(v) for v in rng.integers(1, most * B // 8 + 1, tensors)]
        tables = np.sort(rng.random((tensors, 1 << bits)), axis=1).astype(np.float32)
        x = rng.standard_normal(sum(sizes)).astype(np.float32)
        segs = qb.Segments(sizes, B, DEV)
        codes, meta = segs.alloc_packed(bits)
        qb.qsdp_quantize_levels_segmented(torch.from_numpy(x).to(DEV), segs, bits, torch.from_numpy(tables).to(DEV),
                                          codes, meta.view(-1), stochastic, 3, 16)
        want, o = [[], []], 0
        for t, s in enumerate(sizes):
            v = x[o:o + s].copy()
            wc, wm = (ref.quantize_levels_stochastic(v, bits, B, tables[t], 3, 16 + o) if stochastic
                      else ref.quantize_levels(v, bits, B, tables[t]))
            want[0].append(wc); want[1].append(wm.view(np.uint32).reshape(-1))
            o += s
        assert np.array_equal(np_u32(codes), np.concatenate(want[0]))
        assert np.array_equal(np_u32(meta), np.concatenate(want[1]))
