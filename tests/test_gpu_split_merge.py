"""Split attention merged by a unit's last work-group: whatever the split
count, the output has to be the bits of the separate merge kernel, which runs
when the same tokens are given by the caller (no earlier kernel clears the
arrival counts then).  Many repetitions on one workspace (the counts start from
what the last call left), several calls in flight, empty splits, units from one
to more than the compute units."""
import pytest
import torch

import paper_2604_07815_amd as tls
import synth
from gpu_harness import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("splits", [2, 3, 7, 8, 9, 31, 64, 128])
@pytest.mark.parametrize("dtype,G,d,batch", [("bf16", 1, 64, 1), ("bf16", 4, 128, 5), ("bf16", 8, 64, 3),
                                              ("bf16", 8, 128, 2), ("bf16", 2, 128, 90), ("f32", 4, 128, 2),
                                              ("f32", 1, 64, 3)])
def test_same_bits_as_the_merge_kernel(dtype, G, d, batch, splits):
    cfg = synth.config("toy").replace(batch=batch, h_q=3 * G, h_kv=3, d_qk=d, d_v=d, dtype=dtype, ctx_lo=100,
                                      ctx_hi=900, clusters=1, k_b=9, k_t=200, seed=60 + G + d)
    c = Case(cfg, backend="host", pad="nan").build_index()
    ws = c.workspace()
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    outs = []
    for r in range(6):
        out = torch.empty((batch, cfg.h_q, d), dtype=dt, device="cuda")
        lse = torch.empty((batch, cfg.h_q), dtype=torch.float32, device="cuda")
        tids = torch.empty((batch, 3, cfg.k_t), dtype=torch.int32, device="cuda")
        tls.tls_sparse_decode(c.layout, c.q, c.kv(), c.ctx, c.kmax, c.kmin, c.codes, c.qparams, c.ch, cfg.k_b, cfg.k_t,
                              None, None, out, lse, None, tids, ws, attn_splits=splits)
        outs.append((out, lse, tids))
    torch.cuda.synchronize()
    ref = c.decode(token_ids_in=outs[0][2], attn_splits=splits)
    bits = torch.int16 if dtype == "bf16" else torch.int32
    for out, lse, tids in outs:
        assert torch.equal(tids, outs[0][2])
        assert torch.equal(out.view(bits), ref["out"].view(bits))
        assert torch.equal(lse.view(torch.int32), ref["lse"].view(torch.int32))
