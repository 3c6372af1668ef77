"""Dense calibration where its units and passes end: contexts a token short of or beyond a pass, a unit of 256, 512 or 1024
tokens, blocks longer than a pass, more units than the chip holds workgroups, paged caches, against float64.
Tolerance: fp32 logits of bf16 products (2^-24 sqrt(128) x a few relative to the logit, which is below 16 here) and fp32 sums
of up to 40000 exponentials: 2e-5 of the row's largest value."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,g,d,b,cap,lengths", [
    (8, 4, 128, 16, 131072, (1, 255, 256, 257, 8192, 32769, 131072)),      # units of 256 tokens, then 512, then 1024
    (1, 8, 64, 8, 65536, (65536, 4096, 65535)), (300, 2, 64, 32, 8192, (700, 8192, 2048)), (2, 1, 128, 64, 300000, (299999, 20000)),
])
def test_lengths_in_one_cache(n, g, d, b, cap, lengths):
    """The unit goes by the length of the call, not by the room there is: one context and workspace through several lengths, the
    last one first again.  Against float64, tolerance as below (a third more for 300000 terms)."""
    import paper_2502_04077_amd as ap
    dev = torch.device("cuda:0")
    cap = -(-cap // b) * b
    ctx = ap.Context(n_inst=n, g=g, head_dim=d, block=b, hist_len=8, t_cap=cap, k_blocks=1, n_sink=0, n_local=0, c1=4, c2=4,
                     kv_dtype="bf16")
    gen = torch.Generator(device=dev)
    gen.manual_seed(cap)
    K = torch.empty((n, cap, d), dtype=torch.bfloat16, device=dev).normal_(generator=gen)
    q = (2 * torch.randn((n, g, d), generator=gen, device=dev)).to(torch.bfloat16)
    size = max(16, ctx.workspace_bytes())
    ws = torch.full((size + 4096,), 255, dtype=torch.uint8, device=dev)
    for t in lengths + lengths[:1]:
        row = torch.full((n, cap // b), 7.0, device=dev)
        ctx.calibrate(q, K, t, row, ws)
        for i in sorted({0, n // 2, n - 1}):
            p = torch.softmax(q[i].double() @ K[i, :t].double().T.contiguous() / math.sqrt(d), dim=1)
            ref = torch.zeros((g, cap), dtype=torch.float64, device=dev)
            ref[:, :t] = p
            ref = ref.view(g, cap // b, b).amax(dim=(0, 2))
            assert (row[i].double() - ref).abs().max() <= 2.7e-5 * ref.max(), (t, i)
    assert (ws[size:] == 255).all()                       # nothing is written beyond the workspace


@pytest.mark.parametrize("n,g,d,b,t,paged", [
    (1, 4, 128, 16, 1, False), (1, 4, 128, 8, 15, False), (2, 1, 64, 8, 257, True), (3, 8, 128, 32, 255, False),
    (2, 2, 64, 64, 1025, True), (1, 4, 128, 16, 4097, False), (33, 4, 128, 16, 32001, False), (70, 2, 128, 8, 16385, True),
    (2000, 4, 64, 16, 1030, False), (1600, 1, 128, 64, 2049, True), (5, 8, 64, 16, 40000, False),
])
def test_calibrate_vs_float64(n, g, d, b, t, paged):
    import paper_2502_04077_amd as ap
    dev = torch.device("cuda:0")
    nb = -(-t // b)
    cap = nb + 2
    ctx = ap.Context(n_inst=n, g=g, head_dim=d, block=b, hist_len=8, t_cap=cap * b, k_blocks=1, n_sink=0, n_local=0, c1=4, c2=4,
                     kv_dtype="bf16")
    gen = torch.Generator(device=dev)
    gen.manual_seed(n + t)
    K = torch.randn((n, cap * b, d), generator=gen, device=dev).to(torch.bfloat16)
    q = (2 * torch.randn((n, g, d), generator=gen, device=dev)).to(torch.bfloat16)
    K[:, t:] = float("nan")
    Ka = K
    if paged:
        table = torch.randperm(n * cap, generator=gen, device=dev, dtype=torch.int32).view(n, cap)
        Ka = torch.empty((n * cap, b, d), dtype=K.dtype, device=dev)
        Ka[table.view(-1).long()] = K.view(-1, b, d)
        ctx.set_block_table(table, n * cap)
    ws = torch.full((max(16, ctx.workspace_bytes()),), 255, dtype=torch.uint8, device=dev)
    for again in range(2):
        row = torch.full((n, cap), 7.0, device=dev)
        ctx.calibrate(q, Ka, t, row, ws)
        for i in sorted({0, 1, n // 2, n - 1} & set(range(n))):
            p = torch.softmax(q[i].double() @ K[i, :t].double().T.contiguous() / math.sqrt(d), dim=1)
            ref = torch.zeros((g, cap * b), dtype=torch.float64, device=dev)
            ref[:, :t] = p
            ref = ref.view(g, cap, b).amax(dim=(0, 2))
            assert (row[i].double() - ref).abs().max() <= 2e-5 * ref.max(), (i, again)


@pytest.mark.parametrize("n,g,d,b,lengths", [
    (1, 4, 64, 16, (2051, 255, 257, 1)), (3, 8, 128, 8, (5003, 513)),      # units of 256 tokens, one a workgroup
    (700, 2, 64, 32, (1100, 2000)), (200, 4, 128, 16, (2000, 2700, 1000)),            # of 512 and 1024; d = 128: 512, 1024 and 256
    (2100, 1, 64, 16, (1025, 300, 2000)), (1100, 2, 128, 64, (1900,)),     # more units than the chip can hold workgroups (2048)
])
def test_fp32_units(n, g, d, b, lengths):
    """fp32 caches: units of 256, 512 or 1024 tokens, as the length of the call goes, one a workgroup."""
    import paper_2502_04077_amd as ap
    dev = torch.device("cuda:0")
    cap = -(-max(lengths) // b) * b + b
    ctx = ap.Context(n_inst=n, g=g, head_dim=d, block=b, hist_len=8, t_cap=cap, k_blocks=1, n_sink=0, n_local=0, c1=4, c2=4, kv_dtype="f32")
    gen = torch.Generator(device=dev)
    gen.manual_seed(cap)
    K = torch.randn((n, cap, d), generator=gen, device=dev)
    q = 2 * torch.randn((n, g, d), generator=gen, device=dev)
    size = max(16, ctx.workspace_bytes())
    ws = torch.full((size + 4096,), 255, dtype=torch.uint8, device=dev)
    for t in lengths + lengths[:1]:
        row = torch.full((n, cap // b), 7.0, device=dev)
        ctx.calibrate(q, K, t, row, ws)
        for i in sorted({0, n // 2, n - 1}):
            p = torch.softmax(q[i].double() @ K[i, :t].double().T.contiguous() / math.sqrt(d), dim=1)
            ref = torch.zeros((g, cap), dtype=torch.float64, device=dev)
            ref[:, :t] = p
            ref = ref.view(g, cap // b, b).amax(dim=(0, 2))
            assert (row[i].double() - ref).abs().max() <= 2e-5 * ref.max(), (t, i)
    assert (ws[size:] == 255).all()


@pytest.mark.parametrize("n,g,d,b,t", [
    (5, 4, 128, 16, 20000), (17, 2, 64, 8, 257), (16, 1, 128, 64, 256), (9, 8, 128, 32, 4099), (70, 4, 128, 16, 17000),
])
def test_several_units_a_workgroup(n, g, d, b, t):
    """K in pinned host memory: 16 workgroups go through several units each (25, two or three, one, ten, 75 of 1024 tokens), the largest logits in one
    half of LDS or the other in turn.  Byte for byte what a workgroup per unit makes of the same K in device memory."""
    import paper_2502_04077_amd as ap
    dev = torch.device("cuda:0")
    cap = -(-t // b) * b + b
    ctx = ap.Context(n_inst=n, g=g, head_dim=d, block=b, hist_len=8, t_cap=cap, k_blocks=1, n_sink=0, n_local=0, c1=4, c2=4, kv_dtype="bf16")
    gen = torch.Generator(device=dev)
    gen.manual_seed(t)
    K = torch.randn((n, cap, d), generator=gen, device=dev).to(torch.bfloat16)
    q = (2 * torch.randn((n, g, d), generator=gen, device=dev)).to(torch.bfloat16)
    K_host = torch.empty(K.shape, dtype=K.dtype, pin_memory=True)
    K_host.copy_(K)
    ws = torch.full((max(16, ctx.workspace_bytes()),), 255, dtype=torch.uint8, device=dev)
    rows = []
    for k in (K_host, K):
        rows.append(torch.full((n, cap // b), 7.0, device=dev))
        ctx.calibrate(q, k, t, rows[-1], ws)
    assert torch.equal(rows[0], rows[1])
    p = torch.softmax(q[0].double() @ K[0, :t].double().T.contiguous() / math.sqrt(d), dim=1)
    ref = torch.zeros((g, cap), dtype=torch.float64, device=dev)
    ref[:, :t] = p
    ref = ref.view(g, cap // b, b).amax(dim=(0, 2))
    assert (rows[0][0].double() - ref).abs().max() <= 2e-5 * ref.max()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_more_units_than_a_launch_has_threads_for(dtype):
    """65535 instances of 257 units, more than 2^32 / 256 in all, over one short paged pool: workgroups take several units each (bf16), or the launch has a
    second dimension (fp32).  Against softmax in 64 bits, 2e-5 of the largest value as for the units above."""
    import paper_2502_04077_amd as ap
    dev = torch.device("cuda:0")
    n, d, b, n_phys = 65535, 64, 64, 40
    t = 256 * 1024 + 70
    nb = -(-t // b)
    assert n * -(-t // 1024) * 256 >= 1 << 32
    ctx = ap.Context(n_inst=n, g=1, head_dim=d, block=b, hist_len=8, t_cap=nb * b, k_blocks=1, n_sink=0, n_local=0, c1=4, c2=4, kv_dtype=dtype)
    gen = torch.Generator(device=dev)
    gen.manual_seed(3)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    pool = torch.randn((n_phys, b, d), generator=gen, device=dev).to(dt)
    q = (2 * torch.randn((n, 1, d), generator=gen, device=dev)).to(dt)
    places = torch.randint(0, n_phys, (2, nb), generator=gen, device=dev, dtype=torch.int32)
    table = places[torch.arange(n, device=dev) % 2].contiguous()
    ctx.set_block_table(table, n_phys)
    row = torch.full((n, nb), 7.0, device=dev)
    ws = torch.empty((ctx.workspace_bytes(),), dtype=torch.uint8, device=dev)
    ctx.calibrate(q, pool, t, row, ws)
    assert float(row.max()) <= 1.0 and float(row.min()) >= 0.0
    for i in (0, 1, 32639, 32640, 32641, 32767, 65280, n - 2, n - 1):
        logits = (pool.double().view(-1, d) @ q[i, 0].double() / math.sqrt(d)).view(n_phys, b)[places[i % 2].long()].view(-1)[:t]
        p = torch.zeros(nb * b, dtype=torch.float64, device=dev)
        p[:t] = torch.softmax(logits, dim=0)
        ref = p.view(nb, b).amax(dim=1)
        assert (row[i].double() - ref).abs().max() <= 2e-5 * ref.max(), i
