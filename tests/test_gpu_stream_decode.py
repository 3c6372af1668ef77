"""The streaming form of sparse decode (bf16 lists of fewer than 1024 instances, split or whole, and g = 8), at the sizes
where it can go wrong, against the oracle: lists that end half way into a 16-token pass, one token, empty lists, contexts
that end inside a block (with NaN rows behind), blocks of 8 to 64, paged caches.  Tolerance: fp32 sums of at most 2048
bf16 products and exponentials good to 2 ulp, 2^-24 sqrt(2048) x a few: 2e-5 of the largest value."""
import numpy as np
import pytest
import torch

from oracle import attnpred_oracle as orc
from workloads import to_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,g,d,b,k,t,paged", [
    (1, 4, 128, 8, 33, 700, False),        # odd list of 8-token blocks, split
    (3, 1, 64, 8, 17, 301, True),
    (5, 2, 128, 16, 64, 1600, False),      # two passes a wave
    (2, 8, 64, 64, 9, 1025, False),        # one token in the last block of 64
    (256, 4, 128, 16, 8, 333, False),      # one workgroup per instance and CU
    (300, 2, 64, 32, 5, 257, True),
    (260, 8, 128, 8, 41, 999, False),
    (300, 1, 128, 16, 24, 401, False),
    (520, 8, 128, 16, 20, 777, True),
    (1030, 8, 64, 16, 7, 500, False),      # whole lists, g = 8
    (2, 4, 128, 16, 600, 16001, False),    # a long list in many short splits
    (128, 4, 128, 16, 600, 16001, False),  # ... and in two of 4800 tokens, several sets of sums a wave
    (280, 2, 64, 32, 60, 2500, True),      # a second workgroup for some CUs unless the lists are split
    (40, 4, 128, 16, 2, 40, False),        # fewer tokens than a workgroup has lanes
])
def test_stream_decode_vs_oracle(n, g, d, b, k, t, paged):
    import paper_2502_04077_amd as ap
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(n * 7 + k)
    nb = -(-t // b)
    cap = nb + 3
    k = min(k, cap)
    ctx = ap.Context(n_inst=n, g=g, head_dim=d, block=b, hist_len=8, t_cap=cap * b, k_blocks=k, n_sink=0, n_local=0, c1=4, c2=4,
                     kv_dtype="bf16")
    gen = torch.Generator(device=dev)
    gen.manual_seed(n + k)
    K = torch.randn((n, cap * b, d), generator=gen, device=dev).to(torch.bfloat16)
    V = torch.randn((n, cap * b, d), generator=gen, device=dev).to(torch.bfloat16)
    q = (3 * torch.randn((n, g, d), generator=gen, device=dev)).to(torch.bfloat16)
    K[:, t:], V[:, t:] = float("nan"), float("nan")
    cnt = np.minimum(np.where(np.arange(n) % 3 == 0, k, rng.integers(0, k + 1, n)), nb).astype(np.int32)
    idx = np.zeros((n, k), dtype=np.int32)
    for i in range(n):
        pick = np.sort(rng.choice(nb, size=cnt[i], replace=False))
        if cnt[i] and i % 2 == 0:
            pick[-1] = nb - 1                              # the block the context ends in
        idx[i, :cnt[i]] = pick
    out = torch.full((n, g, d), 7.0, device=dev)
    row = torch.full((n, cap), 7.0, device=dev)
    ws = torch.full((max(16, ctx.workspace_bytes()),), 255, dtype=torch.uint8, device=dev)
    Ka, Va = K, V
    if paged:
        table = torch.from_numpy(rng.permutation(n * cap).astype(np.int32)).to(dev).view(n, cap)
        Ka, Va = torch.empty((n * cap, b, d), dtype=K.dtype, device=dev), torch.empty((n * cap, b, d), dtype=K.dtype, device=dev)
        Ka[table.view(-1).long()] = K.view(-1, b, d)
        Va[table.view(-1).long()] = V.view(-1, b, d)
        ctx.set_block_table(table, n * cap)
    ctx.sparse_decode(q, Ka, Va, t, torch.from_numpy(idx).to(dev), torch.from_numpy(cnt).to(dev), out, row, ws)
    o, r = out.cpu().double().numpy(), row.cpu().double().numpy()
    assert np.isfinite(o).all() and np.isfinite(r).all()
    for i in sorted({0, 1, 2, n // 2, n - 2, n - 1} & set(range(n))):
        if cnt[i] == 0:
            assert not o[i].any() and not r[i].any()
            continue
        ref, A = orc.sparse_attention(to_f64(q[i]), to_f64(K[i]), to_f64(V[i]), idx[i, :cnt[i]], b, t)
        ref_row = np.zeros(cap)
        ref_row[:nb] = orc.pooled_row(A, b)
        assert np.abs(o[i] - ref).max() <= 2e-5 * np.abs(ref).max(), i
        assert np.abs(r[i] - ref_row).max() <= 2e-5 * ref_row.max(), i


@pytest.mark.parametrize("n,g,d,k", [(128, 4, 128, 5000), (256, 2, 64, 5000)])
def test_long_lists_of_small_blocks(n, g, d, k):
    """Lists of so many blocks that their entries exceed a workgroup's LDS at the usual number of splits take more.  The
    blocks share 64 physical ones through the table.  Tolerance: 40000 terms, 2^-24 sqrt(40000) x a few."""
    import paper_2502_04077_amd as ap
    dev = torch.device("cuda:0")
    b, phys = 8, 64
    ctx = ap.Context(n_inst=n, g=g, head_dim=d, block=b, hist_len=8, t_cap=k * b, k_blocks=k, n_sink=0, n_local=0, c1=4, c2=4,
                     kv_dtype="bf16")
    gen = torch.Generator(device=dev)
    gen.manual_seed(k)
    K = torch.randn((phys, b, d), generator=gen, device=dev).to(torch.bfloat16)
    V = torch.randn((phys, b, d), generator=gen, device=dev).to(torch.bfloat16)
    q = (3 * torch.randn((n, g, d), generator=gen, device=dev)).to(torch.bfloat16)
    table = torch.randint(0, phys, (n, k), generator=gen, device=dev, dtype=torch.int32)
    ctx.set_block_table(table, phys)
    idx = torch.arange(k, dtype=torch.int32, device=dev).repeat(n, 1).contiguous()
    cnt = torch.full((n,), k, dtype=torch.int32, device=dev)
    out, row = torch.empty((n, g, d), device=dev), torch.empty((n, k), device=dev)
    ws = torch.full((max(16, ctx.workspace_bytes()),), 255, dtype=torch.uint8, device=dev)
    ctx.sparse_decode(q, K, V, k * b - 3, idx, cnt, out, row, ws)
    for i in (0, n // 2, n - 1):
        Kd, Vd = (to_f64(x[table[i].long()].reshape(k * b, d)) for x in (K, V))
        ref, A = orc.sparse_attention(to_f64(q[i]), Kd, Vd, np.arange(k), b, k * b - 3)
        ref_row = orc.pooled_row(A, b)
        assert np.abs(out[i].cpu().double().numpy() - ref).max() <= 6e-5 * np.abs(ref).max(), i
        assert np.abs(row[i].cpu().double().numpy() - ref_row).max() <= 6e-5 * ref_row.max(), i
