"""The multi-tensor decoder where a wave takes several tiles (large buffers): tensors that end inside a tile, inside a run of
tiles and on its edge, tensors smaller than a tile, every code width, tables and uniform levels, bit for bit against
one single-tensor decode per tensor."""
import numpy as np
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


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("B", [32, 64, 96, 608, 1024])
@pytest.mark.parametrize("bits", [4, 8])
def test_many_tensors_in_a_tile(bits, B, dtype):
    """Tensors of one to three buckets: a lane's rows lie in different tensors, often several apart."""
    gen = torch.Generator(device=DEV).manual_seed(B + bits)
    sizes = (8 * torch.randint(1, 3 * B // 8 + 1, (700,), generator=torch.Generator().manual_seed(B))).tolist()
    segs = qb.Segments(sizes, B, DEV)
    codes, meta = segs.alloc_packed(bits)
    codes.random_(-2 ** 31, 2 ** 31, generator=gen)
    meta.normal_(generator=gen)
    levels = torch.rand((len(sizes), 1 << bits), device=DEV, generator=gen).sort(dim=1).values.contiguous()
    outs = [torch.empty(sum(sizes), dtype=dtype, device=DEV) for _ in range(2)]
    qb.qsdp_dequantize_segmented(codes, meta.view(-1), segs, bits, outs[0])
    qb.qsdp_dequantize_levels_segmented(codes, meta.view(-1), segs, bits, levels, outs[1])
    # every slot decoded on its own: code * scale + base in 64 bits is exact before the rounding of the fma
    c = codes.cpu().numpy().view("uint32")
    shifts = 32 // bits
    code = torch.from_numpy(((c[:, None] >> (bits * np.arange(shifts))) & ((1 << bits) - 1)).reshape(-1).astype("int64"))
    m = meta.cpu().double()
    slot, tensor, b = [], [], 0
    for t, n in enumerate(sizes):
        slot.append(torch.arange(b * B, b * B + n)); tensor.append(torch.full((n,), t)); b += -(-n // B)
    slot, tensor = torch.cat(slot), torch.cat(tensor)
    base, scale = m[slot // B, 0], m[slot // B, 1]
    for out, level in ((outs[0], code[slot].double()), (outs[1], levels.cpu().double()[tensor, code[slot]])):
        want = (level * scale + base).float().to(dtype)
        kind = torch.int32 if dtype == torch.float32 else torch.int16
        assert ((out.cpu().view(kind) - want.view(kind)).abs() <= 1).all()  # rounded twice here, once there
