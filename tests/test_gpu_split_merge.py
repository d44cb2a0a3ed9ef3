"""Split attention merged by a unit's last work-group: whatever the split
count, the output has to be the bits of the separate merge kernel, which runs
when the same tokens (or blocks) are given by the caller (no earlier kernel
clears the arrival counts then).  Many repetitions on one workspace (the counts
start from what the last call left), several calls in flight, empty splits,
units from one to more than the compute units.

Which of the two merged a call is read from the workspace: the arrival count of
every unit, its last region, is the split count after a merge in the attention
and 0 where the merge kernel followed."""
import pytest
import torch

import paper_2604_07815_amd as tls
import synth
from gpu_harness import Case

pytestmark = pytest.mark.gpu


def folds(dtype, G, d, units, k_t, splits):
    """Where the rule puts a call: True or False, None where it depends on how many work-groups share a compute unit."""
    if G * d > 512 or splits * G * d > 32768 or units * k_t > 2 ** 18:
        return False  # columns per thread, partials, tokens in flight
    if dtype == "f32" and -(-k_t // splits) > 64:
        return False  # only the fp32 kernel of one chunk merges
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    if units * splits <= cus:
        return True   # one round of work-groups whatever else fits
    if units * splits > cus * (2 if dtype == "f32" and d == 128 else 8):
        return False  # (64 KB of rows each: two fp32 work-groups of 128 dims; eight: the smallest, 20 KB)
    return None


def arrivals(ws, units):
    return ws[ws.numel() - (4 * units + 255) // 256 * 256:][:4 * units].view(torch.int32).cpu()


def check(cfg, splits, mode=tls.MODE_TWO_LEVEL, expect=None):
    c = Case(cfg, backend="host", pad="nan").build_index()
    units = cfg.batch * cfg.h_kv
    ws = c.workspace()
    assert ws.numel() == tls.tls_workspace_size(c.layout, cfg.k_b, cfg.k_t)
    dt = torch.bfloat16 if cfg.dtype == "bf16" else torch.float32
    blocks, tokens = mode != tls.MODE_TOKEN_SPARSE, mode != tls.MODE_BLOCK_SPARSE
    runs = []

    def call(bids_in, tids_in, bids, tids, w, op):
        out = torch.empty((cfg.batch, cfg.h_q, cfg.d_v), dtype=dt, device="cuda")
        lse = torch.empty((cfg.batch, cfg.h_q), dtype=torch.float32, device="cuda")
        given = bids_in is not None or tids_in is not None
        tls.tls_sparse_decode(c.layout, c.q, c.kv(), c.ctx, None if given or not blocks else c.kmax,
                              None if given or not blocks else c.kmin, None if given or not tokens else c.codes,
                              None if given or not tokens else c.qparams, None if given or not tokens else c.ch,
                              cfg.k_b, cfg.k_t, bids_in, tids_in, out, lse, bids, tids, w, attn_splits=splits, mode=op)
        return out, lse

    for r in range(6):
        bids = tids = None
        if tokens:
            tids = torch.empty((cfg.batch, cfg.h_kv, cfg.k_t), dtype=torch.int32, device="cuda")
        else:
            bids = torch.empty((cfg.batch, cfg.h_kv, cfg.k_b), dtype=torch.int32, device="cuda")
        runs.append((*call(None, None, bids, tids, ws, mode), tids if tokens else bids))
    torch.cuda.synchronize()
    if expect is not None:
        assert bool((arrivals(ws, units) == (splits if expect else 0)).all())
    ws2 = c.workspace()
    ids = runs[0][2]
    ref = call(None if tokens else ids, ids if tokens else None, None, None, ws2,
               tls.MODE_TWO_LEVEL if tokens else mode)
    bits = torch.int16 if cfg.dtype == "bf16" else torch.int32
    for out, lse, got in runs:
        assert torch.equal(got, ids)
        assert torch.equal(out.view(bits), ref[0].view(bits))
        assert torch.equal(lse.view(torch.int32), ref[1].view(torch.int32))


def config(dtype, G, d, batch, h_kv, k_b, k_t, ctx_hi, seed):
    return synth.config("toy").replace(batch=batch, h_q=h_kv * G, h_kv=h_kv, d_qk=d, d_v=d, dtype=dtype, ctx_lo=100,
                                       ctx_hi=ctx_hi, clusters=1, k_b=k_b, k_t=k_t, seed=seed)


@pytest.mark.parametrize("splits", [2, 3, 7, 8, 9, 31, 64, 128])
@pytest.mark.parametrize("dtype,G,d,batch", [("bf16", 1, 64, 1), ("bf16", 4, 128, 5), ("bf16", 8, 64, 3),
                                              ("bf16", 8, 128, 2), ("bf16", 2, 128, 90), ("f32", 4, 128, 2),
                                              ("f32", 1, 64, 3)])
def test_same_bits_as_the_merge_kernel(dtype, G, d, batch, splits):
    check(config(dtype, G, d, batch, 3, 9, 200, 900, 60 + G + d), splits,
          expect=folds(dtype, G, d, 3 * batch, 200, splits))


# one unit; few and many units on either side of the rule's lines
@pytest.mark.parametrize("dtype,G,d,batch,h_kv,k_t,splits,merged", [
    ("bf16", 4, 128, 1, 1, 200, 2, True), ("bf16", 8, 64, 1, 1, 200, 64, True), ("f32", 1, 64, 1, 1, 200, 128, True),
    ("bf16", 2, 128, 2, 8, 200, 16, True), ("bf16", 1, 128, 16, 8, 300, 2, True), ("f32", 4, 128, 8, 8, 200, 4, True),
    ("f32", 8, 64, 8, 4, 300, 7, True),
    ("bf16", 8, 128, 1, 1, 200, 2, False),   # 1024 columns
    ("bf16", 4, 128, 1, 1, 200, 65, False),  # 33280 floats of partials
    ("f32", 4, 128, 1, 1, 200, 3, False),    # two chunks per work-group
    ("f32", 4, 128, 12, 8, 400, 8, False),   # 768 work-groups of 64 KB: more than one round
    ("f32", 1, 128, 26, 8, 300, 5, False),
])
def test_which_kernel_merges(dtype, G, d, batch, h_kv, k_t, splits, merged):
    assert folds(dtype, G, d, batch * h_kv, k_t, splits) is merged
    check(config(dtype, G, d, batch, h_kv, 9, k_t, 900, 7 * G + d + batch), splits, expect=merged)


# work-groups of 12 waves (768 tokens or more each)
@pytest.mark.parametrize("G,d,batch,h_kv,k_t,splits", [(4, 128, 8, 4, 1700, 2), (1, 64, 3, 1, 2400, 3), (8, 64, 2, 4, 1540, 2)])
def test_wide_work_groups(G, d, batch, h_kv, k_t, splits):
    assert k_t >= 768 * splits
    check(config("bf16", G, d, batch, h_kv, 40, k_t, 2600, 5 + G), splits, expect=True)


# the counts cleared by the block top-k and by the token-level top-k
@pytest.mark.parametrize("splits", [2, 9])
@pytest.mark.parametrize("mode", [tls.MODE_BLOCK_SPARSE, tls.MODE_TOKEN_SPARSE])
@pytest.mark.parametrize("dtype,G,d,batch", [("bf16", 4, 128, 3), ("f32", 2, 64, 2)])
def test_single_level_operators(dtype, G, d, batch, mode, splits):
    cfg = config(dtype, G, d, batch, 2, 9, 400, 900, 31 + G)
    tokens = 576 if mode == tls.MODE_BLOCK_SPARSE else 400
    check(cfg, splits, mode, expect=folds(dtype, G, d, 2 * batch, tokens, splits))
