"""The tile kernel against the oracle, bit for bit, in calls large enough for the tiles that only such calls take: two
rows of four waves with several buckets (from about 2^19 elements, AdamW up to 2^23), six rows in the gradient encoder
(from about 2^22.5, over a few large tensors 2^25), three workgroups to a compute unit (large steps with codes). Every
mode that is served, from 16-bit gradients, with 16-bit weights out, several peers, and over tensors that end inside
tiles."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2302_02390_amd import binding as qb
from paper_2302_02390_amd import workloads as wl
from gpu_util import DEV, ORACLE_THREADS, bits_equal, first_mismatch, np_f32, np_u32, synth

pytestmark = pytest.mark.gpu

ADAMW = (2e-4, 0.9, 0.95, 1e-8, 0.1, 0.3, 0.2)
HALVES = {torch.bfloat16: ref.BF16, torch.float16: ref.F16}


@pytest.fixture(autouse=True)
def threads():
    ref.set_threads(ORACLE_THREADS)
    yield
    ref.set_threads(1)


def _dev(a, dtype=None):
    t = torch.from_numpy(np.array(a)).to(DEV)
    return t if dtype is None else t.to(dtype)


def _moments(n, seed):
    rng = np.random.default_rng(seed)
    return (1e-4 * rng.standard_normal(n)).astype(np.float32), (1e-7 * rng.random(n)).astype(np.float32)


def _same(codes, meta, want_codes, want_meta):
    return np.array_equal(np_u32(codes), want_codes) and \
        np.array_equal(np_u32(meta).reshape(-1), want_meta.view(np.uint32).reshape(-1))


def _ragged(elements, B):
    return elements // B * B + B // 2 + 3


@pytest.mark.parametrize("B", [32, 96, 160, 416, 768, 1504])
@pytest.mark.parametrize("g_dtype,x_dtype", [(torch.bfloat16, torch.float16), (torch.float16, torch.bfloat16)])
def test_steps(B, g_dtype, x_dtype):
    n = _ragged(1 << 19 if 32 < B < 1024 else 5 << 18, B)
    x, g = synth(n, B)
    gd = _dev(g, g_dtype)
    g = gd.float().cpu().numpy()
    for wbits, gbits, delta, flags in ((8, 4, 0.0, 0), (5, 3, 2.0 ** -8, 0), (6, 4, 0.0, qb.QSDP_FLAG_GRAD_SHIFT),
                                       (8, 8, 0.0, qb.QSDP_FLAG_KEEP_MASTER)):
        xd, sat = _dev(x), torch.zeros(1, dtype=torch.int64, device=DEV)
        c, m = qb.alloc_packed(n, wbits, B, DEV)
        x16 = torch.empty(n, dtype=x_dtype, device=DEV)
        qb.qsdp_fused_step_mp(xd, gd, 1e-2, wbits, gbits, B, delta, 9, 8, flags, c, m.view(-1), x16, sat)
        want, wc, wm, ws = ref.fused_step(x, g, 1e-2, wbits, gbits, B, delta, 9, index_offset=8, emit_codes=True,
                                          flags=flags)
        assert bits_equal(np_f32(xd), want) and int(sat) == ws and _same(c, m, wc, wm), (wbits, delta, flags)
        half = ref.dequantize(wc, wm, n, wbits, B, HALVES[x_dtype])
        assert np.array_equal(x16.cpu().view(torch.int16).numpy(), half.view(np.int16)), (wbits, delta, flags)


@pytest.mark.parametrize("B", [96, 160, 416, 768, 1504])
@pytest.mark.parametrize("elements", [1 << 19, 1 << 22])
def test_adamw_steps(B, elements):
    n = _ragged(elements, B)
    x, g = synth(n, B)
    mom, var = _moments(n, B + 1)
    gd = _dev(g, torch.bfloat16)
    g = gd.float().cpu().numpy()
    for wbits, delta, flags in ((8, 0.0, 0), (5, 2.0 ** -8, qb.QSDP_FLAG_KEEP_MASTER)):
        xd, md, vd = _dev(x), _dev(mom), _dev(var)
        c, m = qb.alloc_packed(n, wbits, B, DEV)
        x16 = torch.empty(n, dtype=torch.float16, device=DEV)
        qb.qsdp_fused_adamw_step_mp(xd, gd, md, vd, *ADAMW, wbits, 4, B, delta, 9, 8, flags, c, m.view(-1), x16)
        wx, wmo, wvo, wc, wm, _ = ref.fused_adamw_step(x, g, mom, var, *ADAMW, wbits, 4, B, delta, 9, 8, flags, True)
        assert all(bits_equal(np_f32(t), a) for t, a in ((xd, wx), (md, wmo), (vd, wvo))), (wbits, delta)
        half = ref.dequantize(wc, wm, n, wbits, B, ref.F16)
        assert _same(c, m, wc, wm) and np.array_equal(x16.cpu().view(torch.int16).numpy(), half.view(np.int16))
        g32 = _dev(g)
        qb.qsdp_fused_adamw_step_codes(c, m.view(-1), g32, md, vd, *ADAMW, wbits, 4, B, delta, 10, 8)
        w = ref.dequantize(wc, wm, n, wbits, B)
        _, wmo, wvo, wc, wm, _ = ref.fused_adamw_step(w, g, wmo, wvo, *ADAMW, wbits, 4, B, delta, 10, 8, 0, True)
        assert _same(c, m, wc, wm) and bits_equal(np_f32(md), wmo) and bits_equal(np_f32(vd), wvo), (wbits, delta)


@pytest.mark.parametrize("B", [32, 160, 544])
def test_gradient_encoder(B):
    n = _ragged(7 << 20, B)
    _, g = synth(n, B, heavy=False)
    for dtype, bits, flags in ((torch.float32, 3, 0), (torch.bfloat16, 4, 0),
                               (torch.float16, 8, qb.QSDP_FLAG_GRAD_SHIFT)):
        gd = _dev(g, dtype)
        c, m = qb.alloc_packed(n, bits, B, DEV)
        if dtype == torch.float32:
            qb.qsdp_quantize_grad_ex(gd, bits, B, 5, 24, flags, c, m.view(-1))
        else:
            qb.qsdp_quantize_grad_g16(gd, bits, B, 5, 24, c, m.view(-1), flags)
        assert _same(c, m, *ref.quantize_grad(gd.float().cpu().numpy(), bits, B, 5, 24, flags)), (dtype, bits)


@pytest.mark.parametrize("B", [32, 160, 544])
def test_gradients_of_a_few_large_tensors(B):
    n = 9 << 22
    sizes = [12 * (1 << 20) + 24, 11 * (1 << 20) - 8]
    sizes.append(n - sum(sizes) + 5)
    g = wl.grads_student_t3(sum(sizes), 1252, DEV).cpu()
    segs = qb.Segments(sizes, B, DEV)
    c, m = segs.alloc_packed(4)
    qb.qsdp_quantize_grad_segmented(g.to(DEV), segs, 4, 6, 64, c, m.view(-1))
    offsets = np.concatenate([[0], np.cumsum(sizes)])
    wc, wm = zip(*(ref.quantize_grad(g.numpy()[a:b], 4, B, 6, index_offset=64 + int(a))
                   for a, b in zip(offsets[:-1], offsets[1:])))
    assert _same(c, m, np.concatenate(wc), np.concatenate(wm))


@pytest.mark.parametrize("B", [96, 160, 544, 768])
@pytest.mark.parametrize("elements,peers", [(1 << 19, 3), (1 << 19, 8), (7 << 20, 3)])
def test_receive_side(B, elements, peers):
    n, gbits = _ragged(elements, B), 3
    x, _ = synth(n, 3 * B)
    mom, var = _moments(n, B)
    cs, ms = zip(*(ref.quantize_grad(synth(n, 7 * B + p)[1], gbits, B, p) for p in range(peers)))
    cs, ms = np.stack(cs), np.stack([m.reshape(-1) for m in ms])
    rows = torch.zeros((peers, -(-cs.shape[1] // 4) * 4), dtype=torch.int32, device=DEV)  # rows of whole 16 bytes
    floats = torch.zeros((peers, -(-ms.shape[1] // 4) * 4), dtype=torch.float32, device=DEV)
    rows[:, :cs.shape[1]] = _dev(cs.view(np.int32))
    floats[:, :ms.shape[1]] = _dev(ms)
    for wbits, delta, flags in ((8, 0.0, 0), (6, 2.0 ** -9, qb.QSDP_FLAG_KEEP_MASTER)):
        xd = _dev(x)
        c, m = qb.alloc_packed(n, wbits, B, DEV)
        qb.qsdp_recv_step(xd, rows, floats, peers, 1.0 / peers, 1e-2, wbits, gbits, B, delta, 11, flags, c, m.view(-1))
        want, wc, wm, _ = ref.recv_step(x, cs, ms, peers, 1.0 / peers, 1e-2, wbits, gbits, B, delta, 11, flags, True)
        assert bits_equal(np_f32(xd), want) and _same(c, m, wc, wm), (wbits, delta)
        xd, md, vd = _dev(x), _dev(mom), _dev(var)
        qb.qsdp_recv_adamw_step(xd, md, vd, rows, floats, peers, 1.0 / peers, *ADAMW, wbits, gbits, B, delta, 11, flags,
                                c, m.view(-1))
        wx, wmo, wvo, wc, wm, _ = ref.recv_adamw_step(x, mom, var, cs, ms, peers, 1.0 / peers, *ADAMW, wbits, gbits, B,
                                                      delta, 11, flags, True)
        assert all(bits_equal(np_f32(t), a) for t, a in ((xd, wx), (md, wmo), (vd, wvo))), (wbits, delta)
        assert _same(c, m, wc, wm), (wbits, delta)


@pytest.mark.parametrize("B,elements,tensors", [(32, 1 << 19, 40), (96, 1 << 19, 200), (160, 1 << 20, 9),
                                                (416, 1 << 21, 100), (416, 1 << 21, 3), (768, 1 << 19, 25)])
def test_tensors_that_end_inside_tiles(B, elements, tensors):
    rng = np.random.default_rng(B + tensors)
    sizes = [8 * int(s) for s in rng.integers(1, elements // 4 // tensors, tensors - 1)]
    sizes.append(max(8, elements - sum(sizes)) + 5)
    n, offsets = sum(sizes), np.concatenate([[0], np.cumsum(sizes)])
    parts = [slice(a, b) for a, b in zip(offsets[:-1], offsets[1:])]
    x, g = synth(n, B)
    mom, var = _moments(n, B)
    segs = qb.Segments(sizes, B, DEV)

    c, m = segs.alloc_packed(3)
    qb.qsdp_quantize_grad_segmented(_dev(g), segs, 3, 6, 64, c, m.view(-1))
    wc, wm = zip(*(ref.quantize_grad(g[s], 3, B, 6, index_offset=64 + s.start) for s in parts))
    assert _same(c, m, np.concatenate(wc), np.concatenate(wm))

    for wbits, delta in ((8, 0.0), (5, 2.0 ** -8)):
        c, m = segs.alloc_packed(wbits)
        qb.qsdp_quantize_weight_segmented(_dev(x), segs, wbits, delta, 6, c, m.view(-1))
        codes = [ref.quantize_weight(x[s], wbits, B, delta, 6)[:2] for s in parts]
        assert _same(c, m, *map(np.concatenate, zip(*codes))), wbits
        qb.qsdp_fused_step_codes_segmented(c, m.view(-1), _dev(g), segs, 1e-2, wbits, 4, delta, 7, 64)
        codes = [ref.fused_step_codes(a, b, g[s], 1e-2, wbits, 4, B, delta, 7, index_offset=64 + s.start)[:2]
                 for (a, b), s in zip(codes, parts)]
        assert _same(c, m, *map(np.concatenate, zip(*codes))), wbits

        xd, gd = _dev(x), _dev(g, torch.bfloat16)
        x16 = torch.empty(n, dtype=torch.bfloat16, device=DEV)
        qb.qsdp_fused_step_segmented_mp(xd, gd, segs, 1e-2, wbits, 4, delta, 8, 64, 0, c, m.view(-1), x16)
        wide = gd.float().cpu().numpy()
        want = [ref.fused_step(x[s], wide[s], 1e-2, wbits, 4, B, delta, 8, index_offset=64 + s.start, emit_codes=True)
                for s in parts]
        new = np.concatenate([w[0] for w in want])
        assert bits_equal(np_f32(xd), new) and torch.equal(x16.cpu(), torch.from_numpy(new).bfloat16()), wbits
        assert _same(c, m, np.concatenate([w[1] for w in want]), np.concatenate([w[2] for w in want])), wbits

        xd, md, vd = _dev(x), _dev(mom), _dev(var)
        qb.qsdp_fused_adamw_step_segmented(xd, _dev(g), md, vd, segs, *ADAMW, wbits, 4, delta, 9, 64, 0, c, m.view(-1))
        want = [ref.fused_adamw_step(x[s], g[s], mom[s], var[s], *ADAMW, wbits, 4, B, delta, 9, 64 + s.start, 0, True)
                for s in parts]
        for t, a in zip((xd, md, vd), zip(*(w[:3] for w in want))):
            assert bits_equal(np_f32(t), np.concatenate(a)), wbits
        assert _same(c, m, np.concatenate([w[3] for w in want]), np.concatenate([w[4] for w in want])), wbits


def test_a_step_large_enough_for_three_workgroups():
    n, B = (3 << 25) + 100, 768
    x, g = wl.weights(n, 1250, DEV), wl.grads_student_t3(n, 1251, DEV)
    x_np, g_np = x.cpu().numpy(), g.cpu().numpy()
    c, m = qb.alloc_packed(n, 8, B, DEV)
    qb.qsdp_fused_step(x, g, 1e-3, 8, 8, B, 0.0, 3, 0, c, m.view(-1))
    wc, wm = np.zeros(c.numel(), np.uint32), np.zeros((m.shape[0], 2), np.float32)
    ref.fused_step_inplace(x_np, g_np, 1e-3, 8, 8, B, 0.0, 3, 0, wc, wm)
    assert first_mismatch(x, x_np) == -1 and first_mismatch(c, wc.view(np.int32)) == -1
    assert first_mismatch(m.view(-1), wm.reshape(-1)) == -1


@pytest.mark.parametrize("B", [32, 96, 320, 768, 2336, 4128, 6176])
@pytest.mark.parametrize("tail", [1, 2, 3, 4, 5, 30])  # elements of the last bucket, at its slots of four
@pytest.mark.parametrize("buckets", [0, 1, 37])        # full ones before it
def test_the_last_tile(B, tail, buckets):
    """A tile that the call's elements do not fill, down to less than one slot: what it computes, and that what follows
    the call's elements stays as it is."""
    n, room = buckets * B + tail, 64
    x, g = synth(n, B + tail)
    mom, var = _moments(n, B)
    guard = -7.0

    def dev(a, dtype=torch.float32):
        t = torch.full((n + room,), guard, dtype=dtype, device=DEV)
        t[:n] = _dev(a).to(dtype)
        return t

    for dtype, wbits, gbits, delta in ((torch.float32, 8, 4, 0.0), (torch.bfloat16, 5, 3, 2.0 ** -8),
                                       (torch.float16, 6, 8, 0.0)):
        gd = dev(g, dtype)
        wide = gd[:n].float().cpu().numpy()
        c, m = qb.alloc_packed(n, gbits, B, DEV)
        if dtype == torch.float32:
            qb.qsdp_quantize_grad(gd[:n], gbits, B, 5, 24, c, m.view(-1))
        else:
            qb.qsdp_quantize_grad_g16(gd[:n], gbits, B, 5, 24, c, m.view(-1))
        grads = ref.quantize_grad(wide, gbits, B, 5, 24)
        assert _same(c, m, *grads), dtype

        c, m = qb.alloc_packed(n, wbits, B, DEV)
        qb.qsdp_quantize_weight(dev(x)[:n], wbits, B, delta, 6, c, m.view(-1))
        codes = ref.quantize_weight(x, wbits, B, delta, 6)[:2]
        assert _same(c, m, *codes), dtype
        qb.qsdp_fused_step_codes(c, m.view(-1), dev(wide)[:n], 1e-2, wbits, gbits, B, delta, 7)
        assert _same(c, m, *ref.fused_step_codes(*codes, wide, 1e-2, wbits, gbits, B, delta, 7)[:2]), dtype

        xd, md, vd, x16 = dev(x), dev(mom), dev(var), dev(x, torch.float16)
        sat = torch.zeros(1, dtype=torch.int64, device=DEV)
        half = torch.float16 if dtype == torch.float32 else dtype
        gh = dev(wide, half)
        wide = gh[:n].float().cpu().numpy()
        qb.qsdp_fused_adamw_step_mp(xd[:n], gh[:n], md[:n], vd[:n], *ADAMW, wbits, gbits, B, delta, 9, 8, 0, c,
                                    m.view(-1), x16[:n], sat)
        wx, wmo, wvo, wc, wm, ws = ref.fused_adamw_step(x, wide, mom, var, *ADAMW, wbits, gbits, B, delta, 9, 8, 0,
                                                        True)
        assert _same(c, m, wc, wm) and int(sat) == ws, dtype
        for t, want in ((xd, wx), (md, wmo), (vd, wvo)):
            assert bits_equal(np_f32(t[:n]), want) and bool((t[n:] == guard).all()), dtype
        assert torch.equal(x16[:n].cpu(), torch.from_numpy(wx).half()) and bool((x16[n:] == guard).all()), dtype

        xd, rows = dev(x), torch.zeros((2, -(-grads[0].size // 4) * 4), dtype=torch.int32, device=DEV)
        rows[:, :grads[0].size] = _dev(grads[0].view(np.int32))
        floats = torch.zeros((2, -(-grads[1].size // 4) * 4), dtype=torch.float32, device=DEV)
        floats[:, :grads[1].size] = _dev(grads[1].reshape(-1))
        floats[1] *= 0.5
        qb.qsdp_recv_step(xd[:n], rows, floats, 2, 0.5, 1e-2, wbits, gbits, B, delta, 11, 0, c, m.view(-1))
        peer = grads[1].reshape(-1)
        want, wc, wm, _ = ref.recv_step(x, np.stack([grads[0]] * 2), np.stack([peer, peer * np.float32(0.5)]), 2, 0.5,
                                        1e-2, wbits, gbits, B, delta, 11, 0, True)
        assert bits_equal(np_f32(xd[:n]), want) and _same(c, m, wc, wm) and bool((xd[n:] == guard).all()), dtype


def _levels(bits, seed):
    """An ascending table over part of [0, 1], so that values lie below its first level and past its last."""
    rng = np.random.default_rng(seed)
    return np.sort(rng.uniform(0.05, 0.95, 1 << bits)).astype(np.float32)


# tiles of two rows, and of the smallest team that holds a bucket (small calls); of one wave with four, six and eight rows
# and of four with six (the others)
@pytest.mark.parametrize("B,elements", [(32, 0), (96, 0), (320, 0), (768, 0), (2336, 0), (4128, 0), (6176, 0),
                                        (32, 1 << 20), (96, 1 << 20), (768, 1 << 20), (2016, 1 << 22), (608, 1 << 20)])
@pytest.mark.parametrize("tail", [1, 2, 3, 4, 5, 30])
def test_the_last_tile_onto_levels(B, elements, tail):
    """As above, with one table and, in small calls, a table to each of several tensors that end inside tiles."""
    room = 64
    for buckets in ((0, 1, 37) if elements == 0 else (elements // B,)):
        n = buckets * B + tail
        _, v = synth(n, B + tail)
        vd = _dev(v)
        for bits, coin in ((4, False), (4, True), (5, False), (3, True), (8, False)):
            levels = _levels(bits, B + bits)
            c, m = qb.alloc_packed(n, bits, B, DEV)
            guarded = torch.full((c.numel() + room,), -7, dtype=torch.int32, device=DEV)
            metas = torch.full((m.numel() + room,), -7.0, dtype=torch.float32, device=DEV)
            c, m = guarded[:c.numel()], metas[:m.numel()]
            if coin:
                qb.qsdp_quantize_levels_stochastic(vd, bits, B, _dev(levels), 11, 16, c, m)
                want = ref.quantize_levels_stochastic(v, bits, B, levels, 11, 16)
            else:
                qb.qsdp_quantize_levels(vd, bits, B, _dev(levels), c, m)
                want = ref.quantize_levels(v, bits, B, levels)
            assert _same(c, m, *want), (buckets, bits, coin)
            assert bool((guarded[c.numel():] == -7).all()) and bool((metas[m.numel():] == -7.0).all()), (buckets, bits)
    if elements:
        return
    sizes = [8 * (tail // 8 + 1), 3 * B, B + 8, 5 * B + tail]
    segs = qb.Segments(sizes, B, DEV)
    _, v = synth(sum(sizes), B)
    for bits, coin in ((4, False), (3, True)):
        tables = np.stack([_levels(bits, B + t) for t in range(len(sizes))])
        c, m = segs.alloc_packed(bits)
        qb.qsdp_quantize_levels_segmented(_dev(v), segs, bits, _dev(tables), c, m.view(-1), coin, 11, 16)
        o = b = 0
        for t, size in enumerate(sizes):
            nb = -(-size // B)
            got = c[b * B * bits // 32:(b + nb) * B * bits // 32], m[b:b + nb]
            if coin:
                want = ref.quantize_levels_stochastic(v[o:o + size].copy(), bits, B, tables[t], 11, 16 + o)
            else:
                want = ref.quantize_levels(v[o:o + size].copy(), bits, B, tables[t])
            assert _same(*got, *want), (t, bits, coin)
            o, b = o + size, b + nb


@pytest.mark.parametrize("B", [96, 416, 768])
@pytest.mark.parametrize("bits", [5, 8])
@pytest.mark.parametrize("last", [-1, 0])  # buckets of the call against the number that makes 12 * 2^20 slots
def test_who_draws_the_shift_of_weights_over_tensors(B, bits, last):
    """From 12 * 2^20 code slots on the waves draw it at 8 bits in tiles of four rows, with less the host."""
    total = -(-(12 << 20) // B) + last
    sizes = [40 * B + 24, (total // 2) * B - 8, 8, B]
    sizes.append((total - sum(-(-n // B) for n in sizes)) * B - 16)
    segs = qb.Segments(sizes, B, DEV)
    assert segs.total_buckets == total
    x = torch.randn(segs.n, device=DEV)
    c, m = segs.alloc_packed(bits)
    for delta in (0.0, 2.0 ** -6):
        sat = torch.zeros(1, dtype=torch.int64, device=DEV)
        qb.qsdp_quantize_weight_segmented(x, segs, bits, delta, 12, c, m.view(-1), sat)
        o = b = saturated = 0
        for t, size in enumerate(sizes):
            nb = -(-size // B)
            wc, wm, ws = ref.quantize_weight(x[o:o + size].cpu().numpy(), bits, B, delta, 12)
            assert _same(c[b * B * bits // 32:(b + nb) * B * bits // 32], m[b:b + nb], wc, wm), (t, delta)
            o, b, saturated = o + size, b + nb, saturated + ws
        assert int(sat) == saturated, delta
