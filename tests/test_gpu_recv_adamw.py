"""GPU parity of qsdp_recv_adamw_step (P workers' quantized gradient slices averaged, AdamW on
the owner's partition, Q^w of the result) against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2302_02390_amd import binding as qb
from gpu_util import DEV, bits_equal, np_f32, np_u32, synth

pytestmark = pytest.mark.gpu

CASES = [
    # n, P, wbits, gbits, B, delta, flags
    (300 * 1024 + 77, 8, 8, 4, 1024, 0.0, qb.QSDP_FLAG_KEEP_MASTER),
    (300 * 1024 + 77, 8, 8, 4, 1024, 0.0, 0),
    (17 * 128 + 5, 3, 5, 2, 128, 0.0, qb.QSDP_FLAG_KEEP_MASTER),
    (9 * 256 + 255, 5, 6, 3, 256, 0.0, 0),
    (33 * 512 + 8, 4, 3, 6, 512, 0.0, qb.QSDP_FLAG_SYMMETRIC | qb.QSDP_FLAG_KEEP_MASTER),
    (7 * 2048 + 1000, 9, 8, 4, 2048, 0.0, qb.QSDP_FLAG_KEEP_MASTER),
    (5 * 4096 + 4095, 2, 7, 8, 4096, 0.0, qb.QSDP_FLAG_NO_SHIFT),
    (20 * 1024 + 300, 6, 4, 4, 1024, 2.0 ** -10, qb.QSDP_FLAG_KEEP_MASTER),   # saturating lattice
    (11 * 96 + 40, 4, 5, 7, 96, 0.0, qb.QSDP_FLAG_KEEP_MASTER),               # generic bucket size: tile kernel
    (100, 2, 8, 1, 1024, 0.0, 0),
]


@pytest.mark.parametrize("n,P,wbits,gbits,B,delta,flags", CASES)
def test_recv_adamw_step_matches_oracle_over_three_steps(n, P, wbits, gbits, B, delta, flags):
    x, _ = synth(n, 41 + n % 101)
    m = np.zeros(n, np.float32)
    v = np.zeros(n, np.float32)
    xd = torch.from_numpy(x).to(DEV)
    md, vd = torch.zeros(n, device=DEV), torch.zeros(n, device=DEV)
    b1, b2, eps, wd, lr = 0.9, 0.95, 1e-8, 0.1, 2e-4
    for t in range(1, 4):
        cs, ms = [], []
        for p in range(P):
            _, g = synth(n, 1000 * t + 13 * p)
            c, mm = ref.quantize_grad(g, gbits, B, 200 + p)
            cs.append(c); ms.append(mm.reshape(-1))
        cs, ms = np.stack(cs), np.stack(ms)
        c1, c2 = 1 - b1 ** t, 1 - b2 ** t
        x, m, v, want_c, want_m, want_sat = ref.recv_adamw_step(x, m, v, cs, ms, P, 1.0 / P, lr, b1, b2, eps, wd, c1,
                                                                c2, wbits, gbits, B, delta, t, flags, emit_codes=True)
        row = -(-cs.shape[1] // 4) * 4
        gc = torch.zeros((P, row), dtype=torch.int32, device=DEV)
        gc[:, :cs.shape[1]] = torch.from_numpy(cs.view(np.int32)).to(DEV)
        gm = torch.from_numpy(ms).to(DEV)
        wc, wm = qb.alloc_packed(n, wbits, B, DEV)
        sat = torch.zeros(1, dtype=torch.int64, device=DEV)
        qb.qsdp_recv_adamw_step(xd, md, vd, gc[:, :cs.shape[1]], gm, P, 1.0 / P, lr, b1, b2, eps, wd, c1, c2, wbits,
                                gbits, B, delta, t, flags, wc, wm.reshape(-1), sat)
        assert bits_equal(np_f32(xd), x) and bits_equal(np_f32(md), m) and bits_equal(np_f32(vd), v), t
        assert np.array_equal(np_u32(wc), want_c), t
        assert np.array_equal(np_u32(wm).reshape(-1), want_m.view(np.uint32).reshape(-1)), t
        assert int(sat) == want_sat, t


def test_recv_adamw_step_rejects_bad_arguments():
    z = torch.zeros(2048, dtype=torch.float32, device=DEV)
    gc = torch.zeros((2, 256), dtype=torch.int32, device=DEV)
    gm = torch.zeros((2, 4), dtype=torch.float32, device=DEV)
    ok = dict(alpha=0.5, lr=1e-3, beta1=0.9, beta2=0.95, eps=1e-8, weight_decay=0.0, bias1=0.1, bias2=0.05, wbits=8,
              gbits=4, bucket=1024, delta=0.0, seed=0)
    for kw in (dict(beta2=1.0), dict(eps=0.0), dict(bias1=0.0), dict(flags=qb.QSDP_FLAG_GRAD_SHIFT), dict(gbits=9)):
        a = dict(ok)
        a.update(kw)
        with pytest.raises(qb.QsdpError):
            qb.qsdp_recv_adamw_step(z, z.clone(), z.clone(), gc, gm, 2, **a)
    qb.qsdp_recv_adamw_step(z, z.clone(), z.clone(), gc, gm, 2, **ok)
