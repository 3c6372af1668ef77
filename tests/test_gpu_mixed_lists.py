"""Sparse decode of a few instances more than a multiple of the CUs, which go partly whole and partly in splits, at the edges of that rule,
against the oracle: the last whole instance and the first split one, empty and short lists on both sides, contexts that end inside a block (NaN
rows behind), paged caches, and the no-allocation call, whose results are the same bytes.  Tolerance: as for the streaming form, 2e-5 of the largest value."""
import numpy as np
import pytest
import torch

from oracle import attnpred_oracle as orc
from workloads import to_f64

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
    try:
        ctx.sparse_decode_noalloc(q, Ka, Va, t, *lists, out.fill_(7.0), row.fill_(7.0))
    except ap.binding.ApError:
        return                                             # (partials beyond the static scratch: refused)
    assert torch.equal(out, results[0][0]) and torch.equal(row, results[0][1])
