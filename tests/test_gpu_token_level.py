"""Token-level selection over a whole context (MODE_TOKEN_SPARSE) on each of
its kernels: the matrix-core kernels for bf16 with 1 to 8 heads (one or more
32-channel groups) and with 16 or 32 heads, the vector kernel for fp32 and the
other index widths; lengths around the kernels' chunks (1024, 4096 tokens) and
the selection's tiles (16384), budgets from one token to more than the context,
all scores equal (ties to the lowest positions), with more equal keys than the
candidate list holds.

The reference is alpha in float64 from the index rows.  An fp32 alpha is off
by under 2e-6 of its value here (logits below 32 in base 2, each rounded at
2^-24 of that), so the selected set has to hold every token whose alpha is
above the K_t-th by more than 1e-5 of it, and none below it by more."""
import math

import pytest
import torch

import paper_2604_07815_amd as tls

pytestmark = pytest.mark.gpu

CASES = [
    # (G, d_qk, d_c, dtype, mla)
    (1, 64, 32, torch.bfloat16, False), (2, 128, 64, torch.bfloat16, False), (4, 128, 32, torch.bfloat16, False),
    (8, 128, 32, torch.bfloat16, False), (8, 128, 96, torch.bfloat16, False), (4, 128, 32, torch.float32, False),
    (16, 576, 64, torch.bfloat16, True), (32, 576, 128, torch.bfloat16, True), (32, 576, 64, torch.bfloat16, True),
    (16, 576, 128, torch.bfloat16, True), (32, 576, 32, torch.bfloat16, True),
]


def _setup(G, d, d_c, dtype, mla, lens, seed, zero_q=False):
    g = torch.Generator(device="cuda").manual_seed(seed)
    b, hkv, T = len(lens), 1 if mla else 2, max(lens)
    dv = 512 if mla else d
    q = torch.randn((b, G * hkv, d), generator=g, device="cuda") / (24.0 if mla else 1.0)
    q = (q * 0 if zero_q else q).to(dtype)
    K = torch.randn((b, hkv, T, d), generator=g, device="cuda").to(dtype)
    V = None if mla else torch.randn((b, hkv, T, dv), generator=g, device="cuda").to(dtype)
    n = torch.tensor(lens, dtype=torch.int32, device="cuda")
    gc = torch.Generator().manual_seed(seed)
    ch = torch.stack([torch.randperm(d, generator=gc)[:d_c].sort().values for _ in range(hkv)]).int().cuda()
    layout = tls.make_layout(b, G * hkv, hkv, d, dv, T, index_channels=d_c, dtype=dtype, mla_shared_kv=mla)
    codes = torch.zeros((b, hkv, T, d_c // 2), dtype=torch.uint8, device="cuda")
    qp = torch.zeros((b, hkv, T, d_c // 32, 2), dtype=torch.float32, device="cuda")
    tls.tls_build_token_index(layout, K, n, ch, 0, T, codes, qp)
    return layout, q, K, V, n, ch, codes, qp


def _alpha(q, codes, qp, ch, n, s, g, G):
    c = codes[s, g, :n].long()
    x = torch.stack([c & 15, c >> 4], -1).reshape(n, -1, 32).double()
    x = (x * qp[s, g, :n, :, :1].double() + qp[s, g, :n, :, 1:].double()).reshape(n, -1)
    qq = q[s, g * G:(g + 1) * G].double()[:, ch[g].long()]
    return torch.softmax(qq @ x.T / math.sqrt(q.shape[-1]), -1).mean(0)


def _select(layout, q, K, V, n, ch, codes, qp, k_t, noalloc=False):
    b, hkv = K.shape[:2]
    out = torch.empty((b, q.shape[1], 512 if V is None else V.shape[-1]), dtype=q.dtype, device="cuda")
    tids = torch.full((b, hkv, k_t), -7, dtype=torch.int32, device="cuda")
    args = (layout, q, tls.KV(K, V), n, None, None, codes, qp, ch, 1, k_t, None, None, out, None, None, tids)
    if noalloc:
        tls.tls_sparse_decode_noalloc(*args, None, mode=tls.MODE_TOKEN_SPARSE)
    else:
        ws = tls.alloc_workspace(layout, 1, k_t)
        tls.tls_sparse_decode(*args, ws, mode=tls.MODE_TOKEN_SPARSE)
        assert tls.tls_check_device_error(ws) == 0
    torch.cuda.synchronize()
    return tids


@pytest.mark.parametrize("lens,k_t", [((1, 63, 1025), 1), ((4095, 4097, 300), 500), ((16383, 16385, 9000), 2048)])
@pytest.mark.parametrize("G,d,d_c,dtype,mla", CASES)
def test_selected_tokens(G, d, d_c, dtype, mla, lens, k_t):
    check_selected_tokens(G, d, d_c, dtype, mla, lens, k_t)


# the selection keeps the candidate masks of 262144 tokens at a time
def test_selected_tokens_of_long_contexts():
    check_selected_tokens(*CASES[2], (262143, 262145, 300000), 2048)


def check_selected_tokens(G, d, d_c, dtype, mla, lens, k_t):
    a = _setup(G, d, d_c, dtype, mla, lens, 11 * G + d_c)
    layout, q, K, V, n, ch, codes, qp = a
    tids = _select(*a, k_t).cpu()
    for s, ln in enumerate(lens):
        for g in range(K.shape[1]):
            ids = tids[s, g]
            kk = min(k_t, ln)
            assert bool((ids[kk:] == -1).all())
            ids = ids[:kk].long()
            assert bool((ids[1:] > ids[:-1]).all()) and int(ids[0]) >= 0 and int(ids[-1]) < ln
            alpha = _alpha(q, codes, qp, ch, ln, s, g, G).cpu()
            kth = alpha.sort(descending=True).values[kk - 1]
            chosen = torch.zeros(ln, dtype=torch.bool)
            chosen[ids] = True
            assert bool(chosen[alpha > kth * (1 + 1e-5)].all()), (s, g)
            assert not bool(chosen[alpha < kth * (1 - 1e-5)].any()), (s, g)


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("G,d,d_c,dtype,mla", [CASES[2], CASES[5], CASES[7]])
def test_equal_scores_take_the_lowest_positions(G, d, d_c, dtype, mla, noalloc):
    lens = (20000, 700, 5000)  # 20000 equal keys: more than the candidate list holds
    a = _setup(G, d, d_c, dtype, mla, lens, 5, zero_q=True)
    tids = _select(*a, 600, noalloc=noalloc).cpu()
    assert bool((tids == torch.arange(600, dtype=torch.int32)).all())


@pytest.mark.parametrize("G,d,d_c,dtype,mla", [CASES[0], CASES[2], CASES[4], CASES[5], CASES[7]])
def test_equal_scores_of_large_logits(G, d, d_c, dtype, mla):
    """Equal rows and queries of 1e5 to 1e9: the rounding of a logit is then up to several octaves of its exponential,
    so every key may lie above the bound that the second pass states.  Still the lowest positions, and no more."""
    lens, k_t = (2000, 1500, 5000), 500
    layout, q, K, V, n, ch, codes, qp = _setup(G, d, d_c, dtype, mla, lens, 9)
    codes[:] = codes[:, :, :1].clone()
    qp[:] = qp[:, :, :1].clone()
    for k in range(12):
        big = (q.float() * (1e5 * 2.37 ** k * (24 if mla else 1))).to(dtype)
        tids = _select(layout, big, K, V, n, ch, codes, qp, k_t).cpu()
        assert bool((tids == torch.arange(k_t, dtype=torch.int32)).all()), k


SELECT = [
    # (G, d_qk, d_c, dtype): the two-level token stage where the fused kernel does not apply
    (8, 128, 32, torch.bfloat16), (8, 64, 64, torch.bfloat16), (8, 128, 128, torch.bfloat16),
    (4, 128, 64, torch.bfloat16), (2, 128, 128, torch.bfloat16), (3, 128, 64, torch.bfloat16),
    (6, 64, 32, torch.bfloat16), (4, 128, 96, torch.bfloat16), (1, 64, 32, torch.float32), (2, 64, 64, torch.float32),
    (4, 128, 32, torch.float32), (8, 320, 256, torch.float32), (5, 128, 32, torch.float32),
]


@pytest.mark.parametrize("k_b,k_t", [(1, 3), (5, 130), (9, 1000)])
@pytest.mark.parametrize("G,d,d_c,dtype", SELECT)
def test_tokens_of_given_blocks(G, d, d_c, dtype, k_b, k_t):
    """Ragged last blocks, empty list entries, candidate counts that do not fill a work-group."""
    a = _setup(G, d, d_c, dtype, False, (700, 1337, 64), 3 * G + d_c)
    check_tokens_of_given_blocks(a, (700, 1337, 64), G, k_b, k_t, tls.alloc_workspace(a[0], k_b, k_t))


# more than 1024 candidates: several work-groups hand their keys to the last one (4 and 8 heads), or two launches; and
# one work-group of 1024 for 16 and 32 heads.  Calls of all sizes on one workspace, whose arrival counts are what the
# call before left; the last work-group is not full for 17 (1088 slots), 33 and 100.
@pytest.mark.parametrize("G,d,d_c,dtype,mla", [(4, 128, 64, torch.bfloat16, False), (4, 128, 32, torch.float32, False),
                                               (8, 128, 64, torch.bfloat16, False), (8, 64, 32, torch.bfloat16, False),
                                               (8, 128, 96, torch.float32, False), (3, 128, 64, torch.bfloat16, False),
                                               (16, 576, 64, torch.bfloat16, True), (32, 576, 128, torch.bfloat16, True)])
def test_many_candidates_on_one_workspace(G, d, d_c, dtype, mla):
    lens = (7000, 1337, 12345)
    a = _setup(G, d, d_c, dtype, mla, lens, 5 * G + d_c)
    ws = tls.alloc_workspace(a[0], 190, 2048)
    for k_b, k_t in ((100, 2048), (17, 1000), (33, 500), (16, 700), (190, 1500), (17, 1), (100, 64)):
        check_tokens_of_given_blocks(a, lens, G, k_b, k_t, ws)


def check_tokens_of_given_blocks(a, lens, G, k_b, k_t, ws):
    layout, q, K, V, n, ch, codes, qp = a
    b, hkv, _, d = K.shape
    g = torch.Generator().manual_seed(k_b)
    bids = torch.full((b, hkv, k_b), -1, dtype=torch.int32)
    for s, ln in enumerate(lens):
        m = -(-ln // 64)
        for u in range(hkv):
            pick = torch.randperm(m, generator=g)[:max(1, min(k_b - 1, m))].sort().values.int()
            pick[-1] = m - 1  # the ragged block
            bids[s, u, :len(pick)] = pick
    tids = torch.full((b, hkv, k_t), -7, dtype=torch.int32, device="cuda")
    sc = torch.empty((b, hkv, k_t), dtype=torch.float32, device="cuda")
    tls.tls_select_tokens(layout, q, codes, qp, ch, bids.cuda(), k_b, n, k_t, tids, sc, ws)
    assert tls.tls_check_device_error(ws) == 0
    tids, sc = tids.cpu(), sc.cpu()
    for s, ln in enumerate(lens):
        for u in range(hkv):
            cand = torch.cat([torch.arange(64) + 64 * int(i) for i in bids[s, u] if i >= 0])
            cand = cand[cand < ln]
            c = codes[s, u, :ln].cpu().long()
            x = torch.stack([c & 15, c >> 4], -1).reshape(ln, -1, 32).double()
            x = (x * qp[s, u, :ln, :, :1].cpu().double() + qp[s, u, :ln, :, 1:].cpu().double()).reshape(ln, -1)[cand]
            qq = q[s, u * G:(u + 1) * G].cpu().double()[:, ch[u].cpu().long()]
            alpha = torch.zeros(ln, dtype=torch.float64)
            alpha[cand] = torch.softmax(qq @ x.T / math.sqrt(d), -1).mean(0)
            kk = min(k_t, len(cand))
            ids = tids[s, u, :kk].long()
            assert bool((tids[s, u, kk:] == -1).all()) and bool((ids[1:] > ids[:-1]).all())
            kth = alpha[cand].sort(descending=True).values[kk - 1]
            chosen = torch.zeros(ln, dtype=torch.bool)
            chosen[ids] = True
            assert bool(chosen[alpha > kth * (1 + 1e-5)].all()) and not bool(chosen[alpha < kth * (1 - 1e-5)].any())
            assert torch.allclose(sc[s, u, :kk].double(), alpha[ids], rtol=1e-5, atol=0)


@pytest.mark.parametrize("G,d_qk,d_c,mla", [(1, 64, 64, False), (2, 128, 64, False), (4, 128, 64, False), (8, 128, 32, False),
                                            (8, 128, 128, False), (8, 128, 96, False), (16, 576, 64, True),
                                            (32, 576, 128, True)])
def test_codes_enter_the_products_exactly(G, d_qk, d_c, mla):
    """Channels of code 0 add nothing to a logit, however large the query is there: half of each group has queries of
    2^16 and codes 0, the rest queries of 1 and all codes, with min = 0 and scale = 1.  Then a logit is off by the
    additions of its d_c products only, 2^-24 sum |q c| each, and alpha by twice that and the exponentials (2^-20)."""
    lens = (4096, 700)
    layout, q, K, V, n, ch, codes, qp = _setup(G, d_qk, d_c, torch.bfloat16, mla, lens, 17 * G + d_c)
    hkv = K.shape[1]
    g = torch.Generator(device="cuda").manual_seed(G)
    c = torch.randint(0, 16, (*codes.shape[:3], d_c), generator=g, device="cuda", dtype=torch.uint8)
    big = (torch.arange(d_c, device="cuda") // 3) % 2 == 0
    c[..., big] = 0
    codes.copy_(c[..., 0::2] | (c[..., 1::2] << 4))
    qp[..., 0], qp[..., 1] = 1.0, 0.0
    q = torch.randn(q.shape, generator=g, device="cuda") * 0.2
    for u in range(hkv):
        q[:, u * G:(u + 1) * G, ch[u][big].long()] *= 2.0 ** 16
    q = q.to(torch.bfloat16)
    k_b = 11 if not mla else 64
    tids = torch.empty((2, hkv, k_b * 64), dtype=torch.int32, device="cuda")
    sc = torch.empty((2, hkv, k_b * 64), dtype=torch.float32, device="cuda")
    if not mla:  # the two-level scores
        bids = torch.arange(k_b, dtype=torch.int32, device="cuda").reshape(1, 1, -1).repeat(2, hkv, 1)
        ws = tls.alloc_workspace(layout, k_b, k_b * 64)
        # (64-token blocks past a length are empty entries)
        bids[1, :, 11:] = -1
        tls.tls_select_tokens(layout, q, codes, qp, ch, bids.contiguous(), k_b, n, k_b * 64, tids, sc, ws)
        assert tls.tls_check_device_error(ws) == 0
    top = _select(layout, q, K, V, n, ch, codes, qp, 100)  # the token-level operator
    for s, ln in enumerate(lens):
        for u in range(hkv):
            x = c[s, u, :ln].double()
            qq = q[s, u * G:(u + 1) * G].double()[:, ch[u].long()]
            tol = 2 * d_c * 2.0 ** -24 * float((qq.abs() @ x.T).max()) / math.sqrt(d_qk) + 2.0 ** -20
            assert tol < 2e-3
            if not mla:
                m = min(ln, k_b * 64)
                want = torch.softmax(qq @ x[:m].T / math.sqrt(d_qk), -1).mean(0)
                assert torch.equal(tids[s, u, :m], torch.arange(m, dtype=torch.int32, device="cuda"))
                assert torch.allclose(sc[s, u, :m].double(), want, rtol=tol, atol=0)
            want = torch.softmax(qq @ x.T / math.sqrt(d_qk), -1).mean(0)
            kth = want.sort(descending=True).values[99]
            chosen = torch.zeros(ln, dtype=torch.bool, device="cuda")
            chosen[top[s, u].long()] = True
            assert bool(chosen[want > kth * (1 + 2 * tol)].all()) and not bool(chosen[want < kth * (1 - 2 * tol)].any())


@pytest.mark.parametrize("G,d_qk,d_c", [(1, 320, 160), (2, 320, 256), (4, 128, 96), (8, 128, 96), (8, 128, 64)])
def test_a_large_minimum_stays_out_of_the_products(G, d_qk, d_c):
    """bf16 queries that sum to 0 over each group and rows with minima of 2^13 and scales of 2^-6: the minima cancel
    exactly where the sum of the queries is formed first, while min + scale * code is rounded at 2^-11.  A logit is then
    off by a rounding per group, 2^-24 of at most 2^6, and alpha by twice that and the exponentials."""
    lens = (1300, 700)
    layout, q, K, V, n, ch, codes, qp = _setup(G, d_qk, d_c, torch.bfloat16, False, lens, 13 * G + d_c)
    g = torch.Generator(device="cuda").manual_seed(G)
    codes.copy_(torch.randint(0, 256, codes.shape, generator=g, device="cuda", dtype=torch.uint8))
    qp[..., 0] = 2.0 ** -6 * (1 + torch.rand(qp.shape[:-1], generator=g, device="cuda"))
    qp[..., 1] = 2.0 ** 13 * (1 + torch.rand(qp.shape[:-1], generator=g, device="cuda"))
    half = torch.randint(1, 9, (2, 2 * G, d_c // 2), generator=g, device="cuda") * 0.25  # sums of these are exact
    pairs = torch.stack([half, -half], -1).reshape(2, 2 * G, d_c)
    for u in range(2):
        q[:, u * G:(u + 1) * G, ch[u].long()] = pairs[:, u * G:(u + 1) * G].to(torch.bfloat16)
    k_b = 21
    bids = torch.arange(k_b, dtype=torch.int32, device="cuda").reshape(1, 1, -1).repeat(2, 2, 1)
    bids[1, :, 11:] = -1
    tids = torch.empty((2, 2, k_b * 64), dtype=torch.int32, device="cuda")
    sc = torch.empty((2, 2, k_b * 64), dtype=torch.float32, device="cuda")
    ws = tls.alloc_workspace(layout, k_b, k_b * 64)
    tls.tls_select_tokens(layout, q, codes, qp, ch, bids.contiguous(), k_b, n, k_b * 64, tids, sc, ws)
    assert tls.tls_check_device_error(ws) == 0
    for s, ln in enumerate(lens):
        for u in range(2):
            assert torch.equal(tids[s, u, :ln], torch.arange(ln, dtype=torch.int32, device="cuda"))
            alpha = _alpha(q, codes, qp, ch, ln, s, u, G)
            assert torch.allclose(sc[s, u, :ln].double(), alpha, rtol=1e-5, atol=0)


@pytest.mark.parametrize("heads,h_kv,k_b,two", [(32, 1, 128, True), (32, 1, 16, False), (64, 8, 128, False)])
def test_stage_events_around_the_normalisation(heads, h_kv, k_b, two):
    """The normalisation has an interval of its own where it is a launch of its own (32 heads with more than 1024
    candidates: 50 MB of logits, at least 6 us at 8 TB/s, beside the few us between two events), else an empty one, as
    the ones before a given token list."""
    mla = h_kv == 1
    b, T, k_t = (48, 8192, 500) if mla else (2, 8192, 500)
    d, dv = (576, 512) if mla else (128, 128)
    g = torch.Generator(device="cuda").manual_seed(3)
    q = torch.randn((b, heads, d), generator=g, device="cuda").to(torch.bfloat16)
    K = torch.randn((b, h_kv, T, d), generator=g, device="cuda", dtype=torch.bfloat16)
    V = None if mla else torch.randn((b, h_kv, T, dv), generator=g, device="cuda", dtype=torch.bfloat16)
    n = torch.full((b,), T, dtype=torch.int32, device="cuda")
    ch = torch.arange(64, dtype=torch.int32, device="cuda").repeat(h_kv, 1).contiguous()
    layout = tls.make_layout(b, heads, h_kv, d, dv, T, index_channels=64, dtype=torch.bfloat16, mla_shared_kv=mla)
    kmax, kmin = (torch.empty((b, h_kv, T // 64, d), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    codes = torch.empty((b, h_kv, T, 32), dtype=torch.uint8, device="cuda")
    qp = torch.empty((b, h_kv, T, 2, 2), dtype=torch.float32, device="cuda")
    tls.tls_build_block_index(layout, K, n, 0, T, kmax, kmin)
    tls.tls_build_token_index(layout, K, n, ch, 0, T, codes, qp)
    out = torch.empty((b, heads, dv), dtype=torch.bfloat16, device="cuda")
    tids = torch.empty((b, h_kv, k_t), dtype=torch.int32, device="cuda")
    ws = tls.alloc_workspace(layout, k_b, k_t)
    events = [torch.cuda.Event(enable_timing=True) for _ in range(tls.NUM_STAGE_EVENTS)]
    for e in events:
        e.record()
    handles = [e.cuda_event for e in events]

    def interval(first, given):
        got = []
        for _ in range(15):
            idx = (None,) * 5 if given else (kmax, kmin, codes, qp, ch)
            tls.tls_sparse_decode(layout, q, tls.KV(K, V), n, *idx, k_b, k_t, None, tids if given else None, out, None,
                                  None, None if given else tids, ws, stage_events=handles)
            torch.cuda.synchronize()
            got.append(events[first].elapsed_time(events[first + 1]) * 1e3)
        return sorted(got)[7]

    normalisation = interval(3, False)
    empty = interval(3, True)
    assert (normalisation > empty + 5) is two, (normalisation, empty)
