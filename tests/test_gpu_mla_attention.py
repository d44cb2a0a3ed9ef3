"""The absorbed-MLA attention on given token ids, at the edges of its chunks
(32 or 64 tokens), splits and work-groups: list lengths around one and two
chunks, empty entries (single ones, a whole chunk, the whole list), more
work-groups than compute units, both head counts, and logits that grow along
the list, so that the running maximum has to be raised after the first chunk.

Bound: bf16 has eight significant bits, so rounding to nearest is off by up to
2^-8 of a value.  The probabilities are rounded before the second product (the
normaliser is not) and the output once more, so an element may be off by
2^-8 (sum_j w_j |v_j| + |o|); 1e-4 sum_j w_j |v_j| covers the fp32
logits (576 products of magnitude ~1/576 each) and exponentials."""
import math

import pytest
import torch

import paper_2604_07815_amd as tls

pytestmark = pytest.mark.gpu

T = 1600


def _inputs(heads, batch, seed, growing):
    g = torch.Generator().manual_seed(seed)
    q = (torch.randn((batch, heads, 576), generator=g) / 24).to(torch.bfloat16)
    K = torch.randn((batch, 1, T, 576), generator=g)
    if growing:  # base-2 logits rising by about 12 per 64 tokens along the first head's query
        d = q[:, :1].float() / q[:, :1].float().norm(dim=-1, keepdim=True) ** 2
        K = 0.1 * K + d.reshape(batch, 1, 1, 576) * (torch.arange(T) * (12 / 64 * math.log(2) * 24)).reshape(1, 1, T, 1)
    assert K.shape == (batch, 1, T, 576)
    return q, K.to(torch.bfloat16)


def _check(q, K, ids, out, lse):
    b, H, _ = q.shape
    for s in range(b):
        sel = ids[s, 0][ids[s, 0] >= 0].long()
        if len(sel) == 0:
            assert bool((out[s] == 0).all()) and bool((lse[s] == -math.inf).all())
            continue
        k = K[s, 0][sel].double()
        v = k[:, :512]
        z = (q[s].double() @ k.T) / 24.0
        w = torch.softmax(z, -1)
        o, mag = w @ v, w @ v.abs()
        tol = 2.0 ** -8 * (mag + o.abs()) + 1e-4 * mag
        err = (out[s].double() - o).abs()
        assert bool((err <= tol).all()), (s, float((err / tol).max()))
        assert torch.allclose(lse[s].double(), torch.logsumexp(z, -1), rtol=1e-5, atol=1e-4)


def _decode(q, K, ids, splits):
    b, H, _ = q.shape
    layout = tls.make_layout(b, H, 1, 576, 512, T, index_channels=64, dtype=torch.bfloat16, mla_shared_kv=True)
    k_t = ids.shape[-1]
    ws = tls.alloc_workspace(layout, 1, k_t)
    out = torch.empty((b, H, 512), dtype=torch.bfloat16, device="cuda")
    lse = torch.empty((b, H), dtype=torch.float32, device="cuda")
    n = torch.full((b,), T, dtype=torch.int32, device="cuda")
    tls.tls_sparse_decode(layout, q.cuda(), tls.KV(K.cuda(), None), n, None, None, None, None, None, 1, k_t, None,
                          ids.cuda(), out, lse, None, None, ws, attn_splits=splits)
    assert tls.tls_check_device_error(ws) == 0
    return out.cpu(), lse.cpu()


@pytest.mark.parametrize("heads", [16, 32])
@pytest.mark.parametrize("k_t,splits", [(1, 0), (31, 1), (33, 1), (64, 0), (65, 1), (129, 2), (500, 0), (1025, 0),
                                        (1500, 128)])
def test_list_lengths_and_splits(heads, k_t, splits):
    q, K = _inputs(heads, 3, 100 + k_t, False)
    g = torch.Generator().manual_seed(k_t)
    ids = torch.stack([torch.randperm(T, generator=g)[:k_t].sort().values for _ in range(3)]).reshape(3, 1, k_t).int()
    ids[1, 0, torch.rand(k_t, generator=g) < 0.3] = -1  # single empty entries
    ids[2, 0, :64] = -1                                  # whole empty chunks
    _check(q, K, ids, *_decode(q, K, ids, splits))


@pytest.mark.parametrize("heads", [16, 32])
@pytest.mark.parametrize("splits", [1, 2, 128])
def test_rising_logits_raise_the_maximum(heads, splits):
    q, K = _inputs(heads, 2, 7, True)
    ids = torch.arange(1024).reshape(1, 1, -1).repeat(2, 1, 1).int()
    ids[1] = ids[1].flip(-1)
    _check(q, K, ids, *_decode(q, K, ids, splits))


@pytest.mark.parametrize("k_t,splits,growing", [(33, 1, False), (500, 0, False), (1025, 0, False), (1024, 2, True)])
def test_sixteen_heads_keep_fp32_probabilities(k_t, splits, growing):
    """With 16 heads the probabilities enter the second product unrounded, so nothing but the output's own rounding
    (2^-8 |o|) and fp32 errors is left: a logit is a sum of 576 products of magnitude sum |q k| / 24, each addition off
    by 2^-24 of it in the worst case, and a weight by twice the largest logit error (its own and the normaliser's),
    plus 2^-20 for the exponentials and the 32-bit sums."""
    q, K = _inputs(16, 2, 40 + k_t, growing)
    g = torch.Generator().manual_seed(k_t)
    ids = torch.stack([torch.randperm(T, generator=g)[:k_t].sort().values for _ in range(2)]).reshape(2, 1, k_t).int()
    out, _ = _decode(q, K, ids, splits)
    for s in range(2):
        k = K[s, 0][ids[s, 0].long()].double()
        w = torch.softmax((q[s].double() @ k.T) / 24.0, -1)
        o, mag = w @ k[:, :512], w @ k[:, :512].abs()
        size = ((q[s].double().abs() @ k.abs().T) / 24.0).amax(-1, keepdim=True)
        tol = 2.0 ** -8 * o.abs() + (2 * 576 * 2.0 ** -24 * size + 2.0 ** -20) * mag
        err = (out[s].double() - o).abs()
        assert bool((err <= tol).all()), (s, float((err / tol).max()))
        if not growing:  # and nearly every value is the bf16 number nearest to the result
            assert float((out[s] != o.to(torch.bfloat16)).double().mean()) < 0.01


@pytest.mark.parametrize("heads", [16, 32])
@pytest.mark.parametrize("k_t,splits", [(40, 1), (500, 0), (1024, 2)])
def test_nan_query_head_attends_nothing(heads, k_t, splits):
    """A head whose every logit is NaN has a zero output and lse = -inf; the other heads are not touched."""
    q, K = _inputs(heads, 2, 3 + k_t, False)
    ids = torch.arange(k_t).reshape(1, 1, -1).repeat(2, 1, 1).int()
    out, lse = _decode(q, K, ids, splits)
    bad = q.clone()
    bad[:, 3, 100] = math.nan
    o2, l2 = _decode(bad, K, ids, splits)
    assert bool((o2[:, 3] == 0).all()) and bool((l2[:, 3] == -math.inf).all())
    rest = [h for h in range(heads) if h != 3]
    assert torch.equal(o2[:, rest], out[:, rest]) and torch.equal(l2[:, rest], lse[:, rest])


@pytest.mark.parametrize("k_t,splits", [(40, 1), (500, 0), (1024, 2)])
def test_nan_row_leaves_its_split_out_with_sixteen_heads(k_t, splits):
    q, K = _inputs(16, 2, 5 + k_t, False)
    ids = torch.arange(k_t).reshape(1, 1, -1).repeat(2, 1, 1).int()
    K[0, 0, 7, 11] = math.nan
    out, lse = _decode(q, K, ids, splits)
    assert bool(torch.isfinite(out).all()) and not bool(torch.isnan(lse).any())


@pytest.mark.parametrize("heads", [16, 32])
@pytest.mark.parametrize("splits", [0, 3, 40])
def test_block_lists_and_the_block_pool(heads, splits):
    """The same tokens as a list of blocks and as ids over a pool of resident blocks: the bits of the ids on the direct
    layout.  Empty list entries, a ragged last block, blocks in any pool order."""
    q, K = _inputs(heads, 2, 60 + splits, False)
    k_b, m, n_slots = 9, T // 64, 30
    lens = torch.tensor([T - 21, T - 64], dtype=torch.int32)
    g = torch.Generator().manual_seed(4)
    bids = torch.full((2, 1, k_b), -1, dtype=torch.int32)
    ids = torch.full((2, 1, k_b * 64), -1, dtype=torch.int32)
    for s in range(2):
        last = (int(lens[s]) - 1) // 64
        pick = torch.cat([torch.randperm(last, generator=g)[:k_b - 2 - s], torch.tensor([last])]).sort().values
        bids[s, 0, :len(pick)] = pick.int()
        tok = (pick[:, None] * 64 + torch.arange(64)).flatten().int()
        ids[s, 0, :len(tok)] = torch.where(tok < lens[s], tok, torch.tensor(-1, dtype=torch.int32))
    layout = tls.make_layout(2, heads, 1, 576, 512, T, index_channels=64, dtype=torch.bfloat16, mla_shared_kv=True)

    def run(kv, bids_in, ids_in, k_b, k_t, mode):
        ws = tls.alloc_workspace(layout, k_b, k_t)
        out = torch.empty((2, heads, 512), dtype=torch.bfloat16, device="cuda")
        lse = torch.empty((2, heads), dtype=torch.float32, device="cuda")
        tls.tls_sparse_decode(layout, q.cuda(), kv, lens.cuda(), None, None, None, None, None, k_b, k_t, bids_in, ids_in,
                              out, lse, None, None, ws, attn_splits=splits, mode=mode)
        assert tls.tls_check_device_error(ws) == 0
        return out.cpu(), lse.cpu()

    dense = tls.KV(K.cuda(), None)
    ref = run(dense, None, ids.cuda(), 1, k_b * 64, tls.MODE_TWO_LEVEL)
    _check(q, K, ids, *ref)
    slot_map = torch.full((2, 1, m), -1, dtype=torch.int32)
    pool = torch.zeros((2, 1, n_slots, 64, 576), dtype=torch.bfloat16)
    for s in range(2):
        where = torch.randperm(n_slots, generator=g)
        for i, blk in enumerate(bids[s, 0][bids[s, 0] >= 0].tolist()):
            slot_map[s, 0, blk] = where[i]
            rows = K[s, 0, blk * 64:(blk + 1) * 64]
            pool[s, 0, where[i], :len(rows)] = rows
    for got in (run(dense, bids.cuda(), None, k_b, 1, tls.MODE_BLOCK_SPARSE),
                run(tls.KV(pool.cuda(), None, slot_map.cuda(), n_slots), None, ids.cuda(), 1, k_b * 64,
                    tls.MODE_TWO_LEVEL),
                run(tls.KV(pool.cuda(), None, slot_map.cuda(), n_slots), bids.cuda(), None, k_b, 1,
                    tls.MODE_BLOCK_SPARSE)):
        assert torch.equal(got[0].view(torch.int16), ref[0].view(torch.int16))
        assert torch.equal(got[1].view(torch.int32), ref[1].view(torch.int32))
