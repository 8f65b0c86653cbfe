"""The wave kernels' guarded path against the oracle, bit for bit: last buckets of every length that matters (one to five
elements, around the lanes' four and the waves' parts, one less than full), from fp32, bf16 and binary16, with memory
behind the vectors that must not change."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2302_02390_amd import binding as qb
from gpu_util import DEV, bits_equal, guarded, guards_intact, np_f32, np_u32, synth

pytestmark = pytest.mark.gpu


def _on_device(a, dtype, fill):
    full, t = guarded(a.size, dtype, fill)
    t.copy_(torch.from_numpy(np.array(a)).to(DEV).to(dtype))
    return full, t


@pytest.mark.parametrize("B", [128, 256, 512, 1024, 2048, 4096])
@pytest.mark.parametrize("whole", [0, 3])
def test_lengths_of_the_last_bucket(B, whole):
    lengths = {1, 2, 3, 4, 5, 7, 8, 31, 33, 63, 64, 65, 126, 127, B // 2 - 1, B // 2, B // 2 + 1, B - 5, B - 4, B - 1}
    lengths |= {1024 + d for d in (-1, 0, 1, 2, 3, 4, 5) if 1024 + d < B}
    for last in sorted(lengths):
        n = whole * B + last
        x, g = synth(n, B + last)
        for g_dtype in (torch.float32, torch.bfloat16, torch.float16):
            xf, xd = _on_device(x, torch.float32, 7.0)
            gf, gd = _on_device(g, g_dtype, 1e4)
            g32 = gd.float().cpu().numpy()
            c, m = qb.alloc_packed(n, 5, B, DEV)
            hf, h = guarded(n, torch.float16, 3.0)
            qb.qsdp_fused_step_mp(xd, gd, 1e-2, 5, 4, B, 2.0 ** -9 if last % 2 else 0.0, 3, wcodes=c, wmeta=m.view(-1), x16=h)
            want, wc, wm, _ = ref.fused_step(x, g32, 1e-2, 5, 4, B, 2.0 ** -9 if last % 2 else 0.0, 3, emit_codes=True)
            assert bits_equal(np_f32(xd), want) and guards_intact(xf, n, 7.0), (n, g_dtype)
            assert np.array_equal(np_u32(c), wc) and np.array_equal(np_u32(m), wm.view(np.uint32).reshape(-1))
            assert torch.equal(h.cpu(), torch.from_numpy(want).half()) and guards_intact(hf, n, 3.0), (n, g_dtype)
            c, m = qb.alloc_packed(n, 3, B, DEV)
            if g_dtype == torch.float32:
                qb.qsdp_quantize_grad(gd, 3, B, 5, 0, c, m.view(-1))
            else:
                qb.qsdp_quantize_grad_g16(gd, 3, B, 5, 0, c, m.view(-1))
            wc, wm = ref.quantize_grad(g32, 3, B, 5)
            assert np.array_equal(np_u32(c), wc) and np.array_equal(np_u32(m), wm.view(np.uint32).reshape(-1)), (n, g_dtype)
