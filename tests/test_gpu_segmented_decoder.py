"""The multi-tensor decoder where a wave takes several tiles (large buffers): tensors that end inside a tile, inside a run of
tiles and on its edge, tensors smaller than a tile, every code width, tables and uniform levels, bit for bit against
one single-tensor decode per tensor."""
import pytest
import torch

from paper_2302_02390_amd import binding as qb
from gpu_util import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("B", [32, 768, 1024, 4096])
@pytest.mark.parametrize("bits", [1, 4, 5, 6, 7, 8])
def test_runs_of_tiles(bits, B, dtype):
    sizes = [8, 2048 - 8, 3 * 4096, 1024, 40, 5 * 1000 * 1000 + 24, 16, 7 * 1024, 12 * 1024 * 1024 + 8, 2 * B, 1024 - 8, 24]
    segs = qb.Segments(sizes, B, DEV)
    gen = torch.Generator(device=DEV).manual_seed(B + bits)
    codes, meta = segs.alloc_packed(bits)
    codes.random_(-2 ** 31, 2 ** 31, generator=gen)
    meta.normal_(generator=gen)
    levels = torch.rand((len(sizes), 1 << bits), device=DEV, generator=gen).sort(dim=1).values.contiguous()
    outs = [torch.empty(sum(sizes), dtype=dtype, device=DEV) for _ in range(2)]
    qb.qsdp_dequantize_segmented(codes, meta.view(-1), segs, bits, outs[0])
    qb.qsdp_dequantize_levels_segmented(codes, meta.view(-1), segs, bits, levels, outs[1])
    o = b = 0
    for t, n in enumerate(sizes):
        nb = -(-n // B)
        c = codes[b * B * bits // 32:(b + nb) * B * bits // 32].clone()
        m = meta.view(-1)[2 * b:2 * (b + nb)].clone()
        want = torch.empty(n, dtype=dtype, device=DEV)
        for i in range(2):
            if i == 0:
                qb.qsdp_dequantize(c, m, n, bits, B, want)
            else:
                qb.qsdp_dequantize_levels(c, m, n, bits, B, levels[t].contiguous(), want)
            kind = torch.int32 if dtype == torch.float32 else torch.int16
            assert torch.equal(outs[i][o:o + n].view(kind), want.view(kind)), (t, i)
        o, b = o + n, b + nb
