"""Sparse decode of a few instances more than a multiple of the CUs, which go partly whole and partly in splits, at the edges of that rule,
against the oracle: the last whole instance and the first split one, empty and short lists on both sides, contexts that end inside a block (NaN
rows behind), paged caches, and the no-allocation call, whose results are the same bytes.  Tolerance: as for the streaming form, 2e-5 of the largest value."""
import math

import numpy as np
import pytest
import torch

from noalloc_size import fits
from oracle import attnpred_oracle as orc
from workloads import n_weight_floats, to_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,g,d,b,k,t,paged", [
    (257, 4, 128, 16, 64, 1100, False),    # one instance in as many splits as its tokens allow
    (320, 8, 128, 16, 65, 1100, True),     # most beyond 256, and one more
    (321, 8, 128, 16, 65, 1100, False),
    (300, 2, 128, 64, 17, 1090, False),    # blocks that do not go evenly into the splits
    (259, 8, 128, 16, 320, 5300, False),   # longest whole list, and a block more
    (259, 8, 128, 16, 321, 5300, False),
    (513, 1, 128, 8, 131, 1100, True),
    (576, 4, 64, 32, 64, 2100, False),     # d = 64: 2048 tokens at least; two more workgroups a CU, then one
    (577, 4, 64, 32, 64, 2100, True),
    (640, 2, 64, 16, 130, 2100, False),    # most beyond 512, and one more
    (641, 2, 64, 16, 130, 2100, False),
    (896, 4, 128, 16, 63, 1100, False),    # lists too short by a block, and long enough
    (896, 4, 128, 16, 64, 1100, False),
])
def test_whole_and_split_lists(n, g, d, b, k, t, paged):
    import paper_2502_04077_amd as ap
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(n * 7 + k)
    nb = -(-t // b)
    cap = nb + 3
    ctx = ap.Context(n_inst=n, g=g, head_dim=d, block=b, hist_len=8, t_cap=cap * b, k_blocks=k, n_sink=0, n_local=0, c1=4, c2=4,
                     kv_dtype="bf16")
    gen = torch.Generator(device=dev)
    gen.manual_seed(n + k)
    K = torch.randn((n, cap * b, d), generator=gen, device=dev).to(torch.bfloat16)
    V = torch.randn((n, cap * b, d), generator=gen, device=dev).to(torch.bfloat16)
    q = (3 * torch.randn((n, g, d), generator=gen, device=dev)).to(torch.bfloat16)
    K[:, t:], V[:, t:] = float("nan"), float("nan")
    first = n // 256 * 256                                 # the first instance behind the whole ones
    look = sorted({0, 1, 255, 256, first - 2, first - 1, first, min(first + 1, n - 1), (first + n) // 2, n - 2, n - 1})
    cnt = np.where(rng.random(n) < 0.5, k, rng.integers(0, k + 1, n)).astype(np.int32)
    cnt[first - 2], cnt[n - 2], cnt[first - 1], cnt[n - 1] = 0, 1, k, k
    idx = np.zeros((n, k), dtype=np.int32)
    for i in range(n):
        pick = np.sort(rng.choice(nb, size=cnt[i], replace=False))
        if cnt[i] and i % 2 == 0:
            pick[-1] = nb - 1                              # the block the context ends in
        idx[i, :cnt[i]] = pick
    Ka, Va = K, V
    if paged:
        table = torch.from_numpy(rng.permutation(n * cap).astype(np.int32)).to(dev).view(n, cap)
        Ka, Va = torch.empty((n * cap, b, d), dtype=K.dtype, device=dev), torch.empty((n * cap, b, d), dtype=K.dtype, device=dev)
        Ka[table.view(-1).long()] = K.view(-1, b, d)
        Va[table.view(-1).long()] = V.view(-1, b, d)
        ctx.set_block_table(table, n * cap)
    lists = torch.from_numpy(idx).to(dev), torch.from_numpy(cnt).to(dev)
    ws = torch.full((ctx.workspace_bytes() + 4096,), 255, dtype=torch.uint8, device=dev)
    results = []
    for _ in range(2):
        out = torch.full((n, g, d), 7.0, device=dev)
        row = torch.full((n, cap), 7.0, device=dev)
        ctx.sparse_decode(q, Ka, Va, t, *lists, out, row, ws)
        results.append((out, row))
    assert all(torch.equal(x, y) for x, y in zip(*results))
    assert bool((ws[ctx.workspace_bytes():] == 255).all())
    o, r = out.cpu().double().numpy(), row.cpu().double().numpy()
    assert np.isfinite(o).all() and np.isfinite(r).all()
    for i in look:
        if cnt[i] == 0:
            assert not o[i].any() and not r[i].any()
            continue
        ref, A = orc.sparse_attention(to_f64(q[i]), to_f64(K[i]), to_f64(V[i]), idx[i, :cnt[i]], b, t)
        ref_row = np.zeros(cap)
        ref_row[:nb] = orc.pooled_row(A, b)
        assert np.abs(o[i] - ref).max() <= 2e-5 * np.abs(ref).max(), i
        assert np.abs(r[i] - ref_row).max() <= 2e-5 * ref_row.max(), i
    out, row = torch.full_like(out, 7.0), torch.full_like(row, 7.0)
    if not fits(n, g, d, b, k):                            # (partials beyond the static scratch)
        with pytest.raises(ap.ApError) as refused:
            ctx.sparse_decode_noalloc(q, Ka, Va, t, *lists, out, row)
        assert refused.value.code == ap.AP_ERR_RANGE
        return
    ctx.sparse_decode_noalloc(q, Ka, Va, t, *lists, out, row)
    assert torch.equal(out, results[0][0]) and torch.equal(row, results[0][1])


FORMS = [(300, 4, 128, 16, 64, 120), (576, 8, 64, 16, 128, 200), (264, 8, 128, 32, 64, 70)]       # 44, 64 and 8 instances beyond, in 8, 8 and 16 splits


def written(ws):
    """32-bit words of a workspace of 0x5a bytes that were written."""
    return int((ws[:ws.numel() // 4 * 4].view(torch.int32) != 0x5A5A5A5A).sum())


def check(i, blocks, q, K, V, b, t, out, row):
    tok = (blocks[:, None] * b + np.arange(b)).ravel()
    tok = torch.from_numpy(tok[tok < t]).to(q.device)
    p = torch.softmax(q[i].double() @ K[i, tok].double().T.contiguous() / math.sqrt(q.shape[-1]), dim=1)
    ref = p @ V[i, tok].double()
    ref_row = torch.zeros(row.shape[1], dtype=torch.float64, device=q.device)
    ref_row.scatter_reduce_(0, tok // b, p.amax(dim=0), "amax")
    assert (out[i].double() - ref).abs().max() <= 2e-5 * ref.abs().max(), i
    assert (row[i].double() - ref_row).abs().max() <= 2e-5 * ref_row.max(), i


@pytest.mark.parametrize("d,cap,paged,mixed", [(128, 127, False, False), (128, 129, False, False), (128, 258, False, False),
                                                (64, 254, False, False), (64, 258, False, False), (64, 516, False, True), (128, 254, False, True),
                                                (128, 126, False, True), (128, 128, False, True), (128, 130, False, True), (64, 255, False, True), (128, 129, True, True)])
def test_instances_near_512_kb_apart(d, cap, paged, mixed):
    """Lists are split alike where contiguous instances lie 508 or 516 KB apart, or 1032 with d = 128; everywhere else those beyond 512 only."""
    import paper_2502_04077_amd as ap
    dev = torch.device("cuda:0")
    n, g, b, k = 544, 4, 16, 8192 // d
    t = cap * b - 3
    ctx = ap.Context(n_inst=n, g=g, head_dim=d, block=b, hist_len=8, t_cap=cap * b, k_blocks=k, n_sink=0, n_local=0, c1=4, c2=4, kv_dtype="bf16")
    gen = torch.Generator(device=dev)
    gen.manual_seed(cap + d)
    K, V = (torch.randn((n, cap * b, d), generator=gen, device=dev).to(torch.bfloat16) for _ in range(2))
    q = (2 * torch.randn((n, g, d), generator=gen, device=dev)).to(torch.bfloat16)
    if paged:
        table = torch.arange(n * cap, dtype=torch.int32, device=dev).view(n, cap)       # (the caller's: it has to live as long as the calls)
        ctx.set_block_table(table, n * cap)
    idx = torch.rand((n, cap), generator=gen, device=dev).argsort(dim=1)[:, :k].sort(dim=1).values.to(torch.int32).contiguous()
    cnt = torch.full((n,), k, dtype=torch.int32, device=dev)
    out, row = torch.full((n, g, d), 7.0, device=dev), torch.full((n, cap), 7.0, device=dev)
    ws = torch.full((ctx.workspace_bytes(),), 0x5A, dtype=torch.uint8, device=dev)
    ctx.sparse_decode(q, K, V, t, idx, cnt, out, row, ws)
    assert (written(ws) < 2 * n * g * d) == mixed          # (partials of two splits or more of everybody; of 32 instances in 8 or 16)
    for i in (0, 255, 511, 512, n - 1):
        check(i, idx[i].cpu().numpy(), q, K, V, b, t, out, row)


@pytest.mark.parametrize("n,g,d,b,k,nb", FORMS)
def test_entries_twice_and_out_of_order(n, g, d, b, k, nb):
    """Entries outside the context, repeated and in any order, in whole lists and in split ones, whose rows are written by different code.  Against float64."""
    import paper_2502_04077_amd as ap
    dev = torch.device("cuda:0")
    t, first = nb * b - 5, n // 256 * 256
    ctx = ap.Context(n_inst=n, g=g, head_dim=d, block=b, hist_len=8, t_cap=(nb + 3) * b, k_blocks=k, n_sink=0, n_local=0, c1=4, c2=4, kv_dtype="bf16")
    gen = torch.Generator(device=dev)
    gen.manual_seed(n)
    K, V = (torch.randn((n, (nb + 3) * b, d), generator=gen, device=dev).to(torch.bfloat16) for _ in range(2))
    q = (3 * torch.randn((n, g, d), generator=gen, device=dev)).to(torch.bfloat16)
    rng = np.random.default_rng(n)
    idx = rng.integers(-2, nb + 2, (n, k)).astype(np.int32)
    cnt = np.where(np.arange(n) % 4 == 1, 5, k).astype(np.int32)
    out, row = torch.full((n, g, d), 7.0, device=dev), torch.full((n, nb + 3), 7.0, device=dev)
    ws = torch.full((ctx.workspace_bytes(),), 0x5A, dtype=torch.uint8, device=dev)
    ctx.sparse_decode(q, K, V, t, torch.from_numpy(idx).to(dev), torch.from_numpy(cnt).to(dev), out, row, ws)
    beyond, splits = n - first, min(512 // (n - first), k * b // 128, 64)
    splits = -(-k // -(-k // splits))
    assert written(ws) == beyond * splits * g * (d + 2) + int(cnt[first:].sum()) * g           # (only those beyond leave partials: the mixed form)
    for i in (0, 1, 2, 255, first - 2, first - 1, first, first + 1, first + 2, n - 2, n - 1):
        check(i, np.clip(idx[i, :cnt[i]], 0, nb - 1), q, K, V, b, t, out, row)


@pytest.mark.parametrize("n,g,d,b,k,nb", FORMS)
def test_fused_step_and_replay(n, g, d, b, k, nb):
    """A whole step whose decode has this form, behind the selection's launch, and the same from a captured graph, byte for byte on every replay."""
    import paper_2502_04077_amd as ap
    dev = torch.device("cuda:0")
    t, first, hist = nb * b - 5, n // 256 * 256, 8
    ctx = ap.Context(n_inst=n, g=g, head_dim=d, block=b, hist_len=hist, t_cap=nb * b, k_blocks=k, n_sink=1, n_local=2, c1=8, c2=8, kv_dtype="bf16")
    ctx.set_weights((0.2 * np.random.default_rng(n).standard_normal(n_weight_floats(8, 8))).astype(np.float32))
    gen = torch.Generator(device=dev)
    gen.manual_seed(n)
    K, V = (torch.randn((n, nb * b, d), generator=gen, device=dev).to(torch.bfloat16) for _ in range(2))
    q = (3 * torch.randn((n, g, d), generator=gen, device=dev)).to(torch.bfloat16)
    ring = torch.rand((n, hist + 1, nb), generator=gen, device=dev)
    ring0 = ring.clone()
    pred, pstate = (torch.zeros((n, nb), device=dev) for _ in range(2))
    out, idx, cnt = torch.zeros((n, g, d), device=dev), torch.zeros((n, k), dtype=torch.int32, device=dev), torch.zeros((n,), dtype=torch.int32, device=dev)
    ws = torch.empty((ctx.workspace_bytes(),), dtype=torch.uint8, device=dev)

    def step():
        ctx.step(ring, 40, q, K, V, t, out, idx, cnt, pred, pstate, ap.AP_PRED_REBASE, ws)

    def start_over(value):
        for x in (out, pred, pstate):
            x.fill_(value)
        for x in (idx, cnt):
            x.fill_(-1)
        ring.copy_(ring0)
        ws.fill_(0x5A)

    start_over(7.0)
    step()
    beyond, splits = n - first, min(512 // (n - first), k * b // 128, 64)
    splits = -(-k // -(-k // splits))
    assert written(ws) == beyond * (splits * g * (d + 2) + g * k)
    idx2, cnt2, row = torch.zeros_like(idx), torch.zeros_like(cnt), ring[:, 40 % (hist + 1)]
    ctx.select_topk(pred, nb, idx2, cnt2, ws)
    assert torch.equal(idx, idx2) and torch.equal(cnt, cnt2)
    for i in (0, 1, 255, first - 1, first, first + 1, n - 1):
        check(i, idx[i].cpu().numpy(), q, K, V, b, t, out, row)
    want = [x.clone() for x in (out, idx, cnt, pred, pstate, ring)]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    start_over(8.0)
    with torch.cuda.graph(graph):
        step()
    for replay in range(3):
        start_over(9.0 + replay)
        torch.cuda.synchronize()
        graph.replay()
        assert all(torch.equal(x, y) for x, y in zip((out, idx, cnt, pred, pstate, ring), want)), replay
        step()                                             # (a step of the program's own in between)
        torch.cuda.synchronize()
