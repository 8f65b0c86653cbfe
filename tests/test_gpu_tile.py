"""The tile kernels (bucket sizes without a wave kernel) against the oracle, bit for bit, at the bucket sizes where a
tile can go wrong: one group per bucket, buckets that fill a tile of each shape exactly, that leave one group over, that
only just fit; a last tile with few buckets, a short last bucket, one bucket only; tensors of a multi-tensor call that
start and end inside a tile."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2302_02390_amd import binding as qb
from gpu_util import DEV, bits_equal, np_f32, np_u32, synth

pytestmark = pytest.mark.gpu

# every shape of a tile, in small calls and in large ones (see test_tile_plan.py)
RECEIVE_BUCKETS = [32, 224, 288, 608, 768, 2016, 2080, 4064, 4128]
BUCKETS = [32, 64, 224, 288, 608, 768, 1056, 1504, 1536, 2016, 2080, 2720, 4064, 4128, 6144, 6176, 8160, 8192]


@pytest.fixture
def large(monkeypatch):
    """Few workgroups, so that the tiles of large calls are taken and every team works on several of them."""
    monkeypatch.setenv("QSDP_DEBUG_MAXGRID", "2")


def _dev(a):
    return torch.from_numpy(np.array(a)).to(DEV)


@pytest.mark.parametrize("B", BUCKETS)
@pytest.mark.parametrize("buckets,cut", [(1, 0), (1, 31), (2, 5), (97, 0), (131, 13)])
def test_single_tensor(B, buckets, cut):
    n = buckets * B - cut
    x, g = synth(n, B + buckets)
    for bits in (1, 3, 4, 7, 8):
        c, m = qb.alloc_packed(n, bits, B, DEV)
        qb.qsdp_quantize_grad(_dev(g), bits, B, 5, 24, c, m.view(-1))
        wc, wm = ref.quantize_grad(g, bits, B, 5, index_offset=24)
        assert np.array_equal(np_u32(c), wc) and np.array_equal(np_u32(m), wm.view(np.uint32).reshape(-1))
    for wbits, gbits, delta in ((8, 4, 0.0), (5, 8, 0.0), (6, 3, 2.0 ** -9)):
        xd, sat = _dev(x), torch.zeros(1, dtype=torch.int64, device=DEV)
        c, m = qb.alloc_packed(n, wbits, B, DEV)
        qb.qsdp_fused_step(xd, _dev(g), 1e-2, wbits, gbits, B, delta, 9, 8, c, m.view(-1), sat)
        want, wc, wm, ws = ref.fused_step(x, g, 1e-2, wbits, gbits, B, delta, 9, index_offset=8, emit_codes=True)
        assert bits_equal(np_f32(xd), want) and int(sat) == ws
        assert np.array_equal(np_u32(c), wc) and np.array_equal(np_u32(m), wm.view(np.uint32).reshape(-1))
        qb.qsdp_fused_step_codes(c, m.view(-1), _dev(g), 1e-2, wbits, gbits, B, delta, 10)
        wc, wm, _ = ref.fused_step_codes(wc, wm, g, 1e-2, wbits, gbits, B, delta, 10)
        assert np.array_equal(np_u32(c), wc) and np.array_equal(np_u32(m), wm.view(np.uint32).reshape(-1))


@pytest.mark.parametrize("B", RECEIVE_BUCKETS)
def test_receive_side(B):
    n, P, gbits = 41 * B - 9, 3, 5
    x, _ = synth(n, 3 * B)
    rng = np.random.default_rng(B)
    mom, var = (1e-4 * rng.standard_normal(n)).astype(np.float32), (1e-7 * rng.random(n)).astype(np.float32)
    cs, ms = zip(*(ref.quantize_grad(synth(n, 7 * B + p)[1], gbits, B, p) for p in range(P)))
    cs, ms = np.stack(cs), np.stack([m.reshape(-1) for m in ms])
    row = -(-cs.shape[1] // 4) * 4
    gc = torch.zeros((P, row), dtype=torch.int32, device=DEV)
    gc[:, :cs.shape[1]] = _dev(cs.view(np.int32))
    args = (1.0 / P, 1e-2, 0.9, 0.95, 1e-8, 0.01, 0.4, 0.3, 8, gbits, B, 0.0, 4)
    xd, md, vd = _dev(x), _dev(mom), _dev(var)
    c, m = qb.alloc_packed(n, 8, B, DEV)
    qb.qsdp_recv_adamw_step(xd, md, vd, gc, _dev(ms), P, *args, 0, c, m.view(-1))
    want = ref.recv_adamw_step(x, mom, var, cs, ms, P, *args, emit_codes=True)
    assert bits_equal(np_f32(xd), want[0]) and bits_equal(np_f32(md), want[1]) and bits_equal(np_f32(vd), want[2])
    assert np.array_equal(np_u32(c), want[3]) and np.array_equal(np_u32(m), want[4].view(np.uint32).reshape(-1))


@pytest.mark.parametrize("B", [32, 224, 608, 768, 2016, 2080, 4064, 4128])
def test_tensors_inside_a_tile(B):
    sizes = [B, 8, 3 * B + 16, 24 * B, 40, 97 * B + 8, 2 * B, 5 * B + 3]
    segs, n = qb.Segments(sizes, B, DEV), sum(sizes)
    x, g = synth(n, 11 * B)
    bits, K = 4, 16
    tables = np.sort(np.random.default_rng(B).random((len(sizes), K)), axis=1).astype(np.float32)
    tables[:, 0], tables[:, -1] = 0.0, 1.0
    c, m = segs.alloc_packed(bits)
    qb.qsdp_quantize_grad_segmented(_dev(g), segs, bits, 6, 16, c, m.view(-1))
    lc, lm = segs.alloc_packed(bits)
    qb.qsdp_quantize_levels_segmented(_dev(x), segs, bits, _dev(tables), lc, lm.view(-1))
    sc, sm = segs.alloc_packed(bits)
    qb.qsdp_quantize_levels_segmented(_dev(g), segs, bits, _dev(tables), sc, sm.view(-1), True, 6, 16)
    xd = _dev(x)
    qb.qsdp_fused_step_segmented(xd, _dev(g), segs, 1e-2, 8, 4, 0.0, 6, 16)
    o, want = 0, [[], [], [], [], [], [], []]
    for t, s in enumerate(sizes):
        xt, gt = x[o:o + s].copy(), g[o:o + s].copy()
        got = (*ref.quantize_grad(gt, bits, B, 6, index_offset=16 + o), *ref.quantize_levels(xt, bits, B, tables[t]),
               *ref.quantize_levels_stochastic(gt, bits, B, tables[t], 6, 16 + o),
               ref.fused_step(xt, gt, 1e-2, 8, 4, B, 0.0, 6, index_offset=16 + o)[0])
        for w, v in zip(want, got):
            w.append(np.ascontiguousarray(v).view(np.uint32).reshape(-1))
        o += s
    for got, w in zip((c, m, lc, lm, sc, sm, xd), want):
        assert np.array_equal(np_u32(got), np.concatenate(w))


@pytest.mark.parametrize("B", BUCKETS)
def test_large_tiles_single_tensor(B, large):
    test_single_tensor(B, 97, 0)
    test_single_tensor(B, 131, 13)


@pytest.mark.parametrize("B", RECEIVE_BUCKETS)
def test_large_tiles_receive_side(B, large):
    test_receive_side(B)


@pytest.mark.parametrize("B", [32, 224, 608, 768, 2016, 2080, 4064, 4128])
def test_large_tiles_tensors(B, large):
    test_tensors_inside_a_tile(B)


@pytest.mark.parametrize("B", [96, 224, 608, 768, 2016, 2080, 4064, 8192])
def test_more_tiles_than_a_small_call_has(B):
    n = 9 * 2 ** 20 - 27
    x, g = synth(n, B)
    c, m = qb.alloc_packed(n, 5, B, DEV)
    qb.qsdp_quantize_grad(_dev(g), 5, B, 5, 24, c, m.view(-1))
    wc, wm = ref.quantize_grad(g, 5, B, 5, index_offset=24)
    assert np.array_equal(np_u32(c), wc) and np.array_equal(np_u32(m), wm.view(np.uint32).reshape(-1))
    xd = _dev(x)
    qb.qsdp_fused_step(xd, _dev(g), 1e-2, 8, 4, B, 0.0, 9)
    assert bits_equal(np_f32(xd), ref.fused_step(x, g, 1e-2, 8, 4, B, 0.0, 9)[0])


@pytest.mark.parametrize("B", [32, 96, 416, 544, 1024 + 480, 2016])
def test_tiles_of_middling_and_large_calls(B):
    """Sizes at which a call takes tiles of two rows of four waves, and of six rows in the modes that instructions bind
    (test_tile_plan_of_a_call says which)."""
    for buckets, cut in (((1 << 19) // B, 5), ((7 << 20) // B + 7, 31)):
        n = buckets * B - cut
        x, g = synth(n, B)
        c, m = qb.alloc_packed(n, 3, B, DEV)
        qb.qsdp_quantize_grad(_dev(g), 3, B, 5, 24, c, m.view(-1))
        gc, gm = ref.quantize_grad(g, 3, B, 5, index_offset=24)
        assert np.array_equal(np_u32(c), gc) and np.array_equal(np_u32(m), gm.view(np.uint32).reshape(-1))
        for wbits, delta in ((8, 0.0), (5, 2.0 ** -8)):
            xd = _dev(x)
            c, m = qb.alloc_packed(n, wbits, B, DEV)
            qb.qsdp_quantize_weight(xd, wbits, B, delta, 9, c, m.view(-1))
            wc, wm, _ = ref.quantize_weight(x, wbits, B, delta, 9)
            assert np.array_equal(np_u32(c), wc) and np.array_equal(np_u32(m), wm.view(np.uint32).reshape(-1))
            qb.qsdp_fused_step_codes(c, m.view(-1), _dev(g), 1e-2, wbits, 4, B, delta, 10)
            wc, wm, _ = ref.fused_step_codes(wc, wm, g, 1e-2, wbits, 4, B, delta, 10)
            assert np.array_equal(np_u32(c), wc) and np.array_equal(np_u32(m), wm.view(np.uint32).reshape(-1))
        rows = torch.zeros((1, -(-gc.size // 4) * 4), dtype=torch.int32, device=DEV)  # 16-byte rows
        rows[0, :gc.size] = _dev(gc.view(np.int32))
        floats = torch.zeros((1, -(-gm.size // 4) * 4), dtype=torch.float32, device=DEV)
        floats[0, :gm.size] = _dev(gm.reshape(-1))
        qb.qsdp_recv_step(xd, rows, floats, 1, 0.5, 1e-2, 8, 3, B, 0.0, 11)
        want = ref.recv_step(x, gc[None], gm.reshape(1, -1), 1, 0.5, 1e-2, 8, 3, B, 0.0, 11)[0]
        assert bits_equal(np_f32(xd), want)
