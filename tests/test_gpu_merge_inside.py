"""A fused step of few instances - the selection made by every split for itself, the splits merged by the last workgroup to finish -
against the selection's own launch and the decode without a workspace, whose splits are always merged by a launch of their own: the same bytes, call
after call with new queries, whichever workgroup happens to be the last."""
import numpy as np
import pytest
import torch

from noalloc_size import fits
from workloads import n_weight_floats

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,g,d,block,k,nb,dtype,hist", [
    (1, 4, 64, 16, 16, 130, "f32", 16),       # fp32 form
    (3, 8, 128, 16, 130, 300, "f32", 16),
    (2, 1, 128, 8, 1024, 1100, "f32", 8),     # more splits than a wave has lanes
    (8, 4, 128, 16, 64, 130, "f32", 8), (8, 4, 128, 16, 68, 130, "f32", 8),           # most splits merged inside, and one more
    (8, 8, 128, 16, 48, 130, "f32", 8), (8, 8, 128, 16, 52, 130, "f32", 8),           # most sums, and more
    (32, 2, 64, 16, 64, 90, "f32", 8), (33, 2, 64, 16, 64, 90, "f32", 8),             # most workgroups, and more
    (4, 8, 128, 16, 96, 200, "bf16", 8), (4, 4, 128, 16, 128, 200, "bf16", 8),
    (8, 4, 128, 16, 64, 2050, "bf16", 64), (1, 1, 128, 16, 300, 700, "bf16", 16), (128, 2, 64, 16, 64, 500, "bf16", 16),
    (5, 8, 128, 32, 64, 131, "bf16", 16), (1, 4, 128, 64, 256, 300, "bf16", 16), (2, 8, 64, 8, 4096, 4099, "bf16", 8),
    (4, 4, 128, 8, 64, 2307, "bf16", 8), (4, 4, 128, 8, 64, 2308, "bf16", 8),         # most candidates the decode selects from, and one more
    (4, 4, 64, 8, 64, 2307, "f32", 8), (4, 4, 64, 8, 64, 2308, "f32", 8),
    (7, 1, 64, 16, 121, 3841, "bf16", 8), (7, 2, 128, 16, 128, 3841, "bf16", 8), (7, 4, 128, 16, 128, 3841, "bf16", 8),   # 15 and 16 splits behind a selection's launch
    (3, 2, 128, 16, 99, 400, "bf16", 8), (3, 2, 128, 16, 100, 400, "bf16", 8),        # most free places of a selection inside, and one more
    (3, 2, 128, 16, 131, 400, "bf16", 8), (3, 2, 128, 16, 132, 400, "bf16", 8),
    (256, 4, 128, 16, 64, 700, "bf16", 8), (500, 8, 64, 16, 64, 90, "bf16", 8), (513, 8, 64, 16, 16, 90, "bf16", 8),   # whole lists, and a workgroup too many
    (300, 4, 128, 16, 64, 200, "bf16", 16), (3, 4, 128, 16, 64, 40, "bf16", 16),      # (the last: lists shorter than the budget)
])
def test_same_bytes(n, g, d, block, k, nb, dtype, hist):
    import paper_2502_04077_amd as ap
    assert fits(n, g, d, block, k)
    dev = torch.device("cuda:0")
    cap = nb + 5
    ctx = ap.Context(n_inst=n, g=g, head_dim=d, block=block, hist_len=hist, t_cap=cap * block, k_blocks=k, n_sink=1, n_local=2, c1=4, c2=4,
                     kv_dtype=dtype)
    rng = np.random.default_rng([n, k, nb])
    blob = (0.2 * rng.standard_normal(n_weight_floats(4, 4))).astype(np.float32)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device=dev)
    gen.manual_seed(n * 1000 + k)
    K, V = (torch.randn((n, cap * block, d), generator=gen, device=dev).to(dt) for _ in range(2))
    ring = torch.rand((n, hist + 1, cap), generator=gen, device=dev)
    pred, pstate, row = (torch.zeros((n, cap), device=dev) for _ in range(3))
    out, out2 = (torch.zeros((n, g, d), device=dev) for _ in range(2))
    idx, idx2 = (torch.full((n, k), -7, dtype=torch.int32, device=dev) for _ in range(2))
    cnt, cnt2 = (torch.zeros((n,), dtype=torch.int32, device=dev) for _ in range(2))
    ws = torch.zeros((ctx.workspace_bytes(),), dtype=torch.uint8, device=dev)
    t, pushed = nb * block - 3, 4 * hist
    for i in range(12):
        q = torch.randn((n, g, d), generator=gen, device=dev).to(dt)
        ws.random_(0, 256, generator=gen)                # whatever an earlier call left there
        ring[:, pushed % (hist + 1)] = 9.0
        out.fill_(7.0)
        ctx.set_weights(blob * (i != 5))                 # (all weights zero: scores that are all the same)
        ctx.step(ring, pushed, q, K, V, t, out, idx, cnt, pred, pstate, ap.AP_PRED_REBASE, ws)
        ctx.select_topk(pred, nb, idx2, cnt2, ws)
        assert torch.equal(idx, idx2) and torch.equal(cnt, cnt2), i
        ctx.sparse_decode_noalloc(q, K, V, t, idx, cnt, out2, row)
        assert torch.equal(out, out2), i
        assert torch.equal(ring[:, pushed % (hist + 1)], row), i
        pushed += 1


@pytest.mark.parametrize("c1,c2,fp32", [(4, 4, False), (8, 8, False), (16, 32, False), (8, 8, True), (16, 32, True)])
@pytest.mark.parametrize("hist", [16, 4])                # (below 6 every call evaluates the full tile)
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_every_predictor_clears_the_counters(c1, c2, fp32, hist, dtype):
    """The counters of the merge lie in the workspace, and whichever predictor runs sets them to zero: all of its forms over a
    workspace of garbage - re-base with and without a state of the caller's, advance, hold, a tile that grows - with selections made and reused."""
    import paper_2502_04077_amd as ap
    dev = torch.device("cuda:0")
    n, g, d, block, k, nb = 5, 4, 128, 16, 64, 300
    cap = nb + 4
    ctx = ap.Context(n_inst=n, g=g, head_dim=d, block=block, hist_len=hist, t_cap=cap * block, k_blocks=k, n_sink=1, n_local=2, c1=c1, c2=c2,
                     kv_dtype=dtype, flags=ap.AP_FLAG_PREDICTOR_FP32 if fp32 else 0)
    rng = np.random.default_rng(c1 + hist)
    ctx.set_weights((0.2 * rng.standard_normal(n_weight_floats(c1, c2))).astype(np.float32))
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device=dev)
    gen.manual_seed(c1 * 100 + hist)
    K, V = (torch.randn((n, cap * block, d), generator=gen, device=dev).to(dt) for _ in range(2))
    ring = torch.rand((n, hist + 1, cap), generator=gen, device=dev) * 0.01
    pred, pstate, row = (torch.zeros((n, cap), device=dev) for _ in range(3))
    out, out2 = (torch.zeros((n, g, d), device=dev) for _ in range(2))
    idx, idx2 = (torch.full((n, k), -7, dtype=torch.int32, device=dev) for _ in range(2))
    cnt, cnt2 = (torch.zeros((n,), dtype=torch.int32, device=dev) for _ in range(2))
    ws = torch.zeros((ctx.workspace_bytes(),), dtype=torch.uint8, device=dev)
    pushed, end = 4 * hist, nb * block
    reuse = ap.AP_STEP_REUSE_SELECTION
    for i, (mode, t, state) in enumerate([
            (ap.AP_PRED_REBASE, end - 3, pstate), (ap.AP_PRED_ADVANCE, end - 2, pstate), (ap.AP_PRED_HOLD, end - 2, pstate), (ap.AP_PRED_ADVANCE, end, pstate),
            (ap.AP_PRED_ADVANCE, end + 1, pstate), (ap.AP_PRED_ADVANCE | reuse, end + 2, pstate), (ap.AP_PRED_HOLD | reuse, end + 2, pstate),
            (ap.AP_PRED_SKIP | reuse, end + 3, pstate), (ap.AP_PRED_REBASE, end + 4, None), (ap.AP_PRED_REBASE, end + 5, pstate)]):
        q = torch.randn((n, g, d), generator=gen, device=dev).to(dt)
        ws.random_(0, 256, generator=gen)
        ring[:, pushed % (hist + 1)] = 9.0
        out.fill_(7.0)
        ctx.step(ring, pushed, q, K, V, t, out, idx, cnt, pred, state, mode, ws)
        if not mode & reuse:
            ctx.select_topk(pred, -(-t // block), idx2, cnt2, ws)
            assert torch.equal(idx, idx2) and torch.equal(cnt, cnt2), i
        ctx.sparse_decode_noalloc(q, K, V, t, idx, cnt, out2, row)
        assert torch.equal(out, out2), i
        assert torch.equal(ring[:, pushed % (hist + 1)], row), i
        pushed += 1


FILL = 0x5A


def lone_words(ws):
    """64-bit words of a workspace that was all FILL which were written while the 15 behind them were not, as those are that workgroups count in:
    where they lie and what they hold."""
    words = ws[:ws.numel() // 8 * 8].view(torch.int64)
    blank = words == int.from_bytes(bytes([FILL]) * 8, "little")
    alone = ~blank[:-15]
    for i in range(1, 16):
        alone &= blank[i:blank.numel() - 15 + i]
    at = alone.nonzero().view(-1)
    return at, words[at]


@pytest.mark.parametrize("c1,c2", [(4, 4), (8, 8), (16, 32)])
@pytest.mark.parametrize("n,g,d,block,k,nb,dtype", [(8, 4, 128, 16, 64, 2000, "bf16"), (3, 4, 64, 16, 64, 300, "f32"), (128, 2, 64, 16, 64, 500, "bf16"), (1, 8, 128, 32, 48, 200, "bf16"),
                                                       (128, 4, 128, 16, 16, 90, "f32")])
def test_fused_step_only_adds(n, g, d, block, k, nb, dtype, c1, c2):
    """The decode behind a predictor, with the selection in the same launch or one from a step before, finds the counters at zero and adds to them, no more: they are
    left at the number of splits.  (Asking for each word and setting it back cost a step of 17 us 0.07, one of 14.6 us without a selection 0.5.)"""
    import paper_2502_04077_amd as ap
    dev = torch.device("cuda:0")
    ctx = ap.Context(n_inst=n, g=g, head_dim=d, block=block, hist_len=16, t_cap=nb * block, k_blocks=k, n_sink=1, n_local=2, c1=c1, c2=c2, kv_dtype=dtype)
    ctx.set_weights((0.2 * np.random.default_rng(k).standard_normal(n_weight_floats(c1, c2))).astype(np.float32))
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    K, V = (torch.randn((n, nb * block, d), device=dev).to(dt) for _ in range(2))
    q = torch.randn((n, g, d), device=dev).to(dt)
    ring = torch.rand((n, 17, nb), device=dev)
    pred, pstate = (torch.zeros((n, nb), device=dev) for _ in range(2))
    out, idx, cnt = torch.zeros((n, g, d), device=dev), torch.zeros((n, k), dtype=torch.int32, device=dev), torch.zeros((n,), dtype=torch.int32, device=dev)
    ws = torch.empty((ctx.workspace_bytes(),), dtype=torch.uint8, device=dev)
    for i, mode in enumerate((ap.AP_PRED_REBASE, ap.AP_PRED_ADVANCE, ap.AP_PRED_ADVANCE | ap.AP_STEP_REUSE_SELECTION, ap.AP_PRED_ADVANCE)):
        ws.fill_(FILL)
        ctx.step(ring, 40 + i, q, K, V, nb * block, out, idx, cnt, pred, pstate, mode, ws)
        at, held = lone_words(ws)
        at, held = at[(held > 1) & (held <= 16)], held[(held > 1) & (held <= 16)]        # (other words alone: the ends of the partials, floats)
        assert at.numel() == n and bool((held == held[0]).all()), (i, held.tolist())
        assert bool((at.diff() == 16).all()), i


@pytest.mark.parametrize("n,g,d,block,k,dtype,inside", [
    (16, 4, 128, 16, 192, "bf16", True), (16, 4, 128, 16, 208, "bf16", False),       # 16 splits of many sums: short lists, and longer ones
    (17, 4, 128, 16, 256, "bf16", True), (16, 2, 128, 16, 256, "bf16", True),         # 15 splits; 16 of few sums
    (32, 8, 64, 16, 128, "bf16", False), (33, 8, 64, 16, 128, "bf16", True), (20, 8, 128, 16, 128, "bf16", True),
    (52, 4, 128, 16, 256, "bf16", True), (52, 4, 128, 16, 272, "bf16", False),        # more than a workgroup a CU, nine splits of many sums: 4096 tokens, and more
    (100, 1, 128, 16, 800, "bf16", True), (100, 1, 128, 16, 805, "bf16", False),      # the same, five splits: 2560 tokens each, and more
    (28, 4, 128, 16, 256, "bf16", True), (28, 4, 128, 16, 257, "bf16", False),        # up to a workgroup a CU, many sums: nine splits, 4096 tokens and more;
    (24, 4, 128, 16, 448, "bf16", True), (24, 4, 128, 16, 449, "bf16", False),        # ten, 7168;
    (17, 4, 128, 16, 1408, "bf16", True), (17, 4, 128, 16, 1409, "bf16", False),      # fifteen, 22528;
    (28, 2, 128, 16, 1024, "bf16", True),             # few sums
    (8, 8, 64, 16, 64, "f32", False), (8, 8, 64, 16, 60, "f32", True), (8, 4, 64, 16, 64, "f32", True), (64, 4, 128, 16, 16, "f32", True),
    (65, 4, 128, 16, 16, "f32", False), (128, 4, 64, 16, 16, "f32", True), (129, 4, 64, 16, 16, "f32", False),
])
def test_single_call_forms(n, g, d, block, k, dtype, inside):
    """Which single calls merge inside the decode, and that the others leave the counters alone."""
    import paper_2502_04077_amd as ap
    dev = torch.device("cuda:0")
    ctx = ap.Context(n_inst=n, g=g, head_dim=d, block=block, hist_len=8, t_cap=k * block, k_blocks=k, n_sink=0, n_local=0, c1=4, c2=4, kv_dtype=dtype)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    K, V = (torch.randn((n, k * block, d), device=dev).to(dt) for _ in range(2))
    q = torch.randn((n, g, d), device=dev).to(dt)
    idx, cnt = torch.arange(k, dtype=torch.int32, device=dev).repeat(n, 1), torch.full((n,), k, dtype=torch.int32, device=dev)
    got, ref = ([torch.zeros((n, g, d), device=dev), torch.zeros((n, k), device=dev)] for _ in range(2))
    ws = torch.full((ctx.workspace_bytes(),), FILL, dtype=torch.uint8, device=dev)
    ctx.sparse_decode(q, K, V, k * block - 3, idx, cnt, *got, ws)
    at, held = lone_words(ws)
    assert int((held == 0).sum()) == (n if inside else 0)
    ctx.sparse_decode_noalloc(q, K, V, k * block - 3, idx, cnt, *ref)
    assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])


def test_offload_step_clears_the_counters():
    """The same where the launch of the appended row does it: offload steps over a workspace of garbage against the single calls, their decode without a
    workspace."""
    from paper_2502_04077_amd.offload import OffloadRun
    from test_gpu_parity import small
    from workloads import kv_cache, predictor_weights, queries
    dev = torch.device("cuda:0")
    w = small("offload", layers=2, batch=1, kv_heads=3, g=4, head_dim=128, t0=1010, budget_tokens=512, hist_len=16, steps=12, calib_every=5)
    K, V = kv_cache(w, dev)
    hosts = []
    for x in (K, V):
        hosts.append(torch.empty(x.shape, dtype=x.dtype, pin_memory=True))
        hosts[-1].copy_(x)
    runs = [OffloadRun(w, *hosts, dev, rebase_every=4, single_calls=single) for single in (False, True)]
    for L in runs[1].layers:
        L.ctx.sparse_decode = lambda *args, ctx=L.ctx: ctx.sparse_decode_noalloc(*args[:-1])
    for run in runs:
        run.set_weights(predictor_weights(w))
        for j in range(w.hist_len):
            run.warmup_calibrate(queries(w, j - w.hist_len, dev), w.t0 - w.hist_len + 1 + j)
        run.start(w.t_at(0))
    for s in range(w.steps):
        t, q = w.t_at(s), queries(w, s, dev)
        for run in runs:
            for L in run.layers:
                L.ws.random_(0, 256)
                L.out.fill_(7.0)
            run.step(q, K[:, t - 1, :].contiguous(), V[:, t - 1, :].contiguous(), t, calibrate=w.is_calibration_step(s))
        assert torch.equal(runs[0].out(), runs[1].out()), s
        assert torch.equal(runs[0].logical_history(), runs[1].logical_history()), s
        for a, b in zip(runs[0].staged_selection(), runs[1].staged_selection()):
            assert torch.equal(a, b), s
    for run in runs:
        run.finish()


@pytest.mark.parametrize("n,g,d,block,k,nb,dtype", [
    (8, 4, 128, 16, 64, 300, "bf16"), (1, 8, 64, 8, 240, 400, "bf16"), (50, 8, 64, 16, 128, 130, "bf16"), (3, 4, 64, 16, 64, 90, "f32"),
    (16, 2, 64, 16, 40, 90, "f32"), (64, 4, 128, 16, 16, 90, "f32"),
    (16, 2, 128, 16, 256, 257, "bf16"), (256, 1, 64, 16, 128, 129, "bf16"),           # most splits; most workgroups, and the last counter
])
def test_single_calls_count_in_any_workspace(n, g, d, block, k, nb, dtype):
    """Single calls merge inside too, counting in words of the workspace that may hold anything - garbage, zeros, all ones, what the call before left -
    and from a captured graph, whose launches count under the same number every time.  Against the call without counters, whose
    merge is a launch of its own: the same bytes."""
    import paper_2502_04077_amd as ap
    dev = torch.device("cuda:0")
    ctx = ap.Context(n_inst=n, g=g, head_dim=d, block=block, hist_len=8, t_cap=nb * block, k_blocks=k, n_sink=0, n_local=0, c1=4, c2=4, kv_dtype=dtype)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device=dev)
    gen.manual_seed(n + k)
    K, V = (torch.randn((n, nb * block, d), generator=gen, device=dev).to(dt) for _ in range(2))
    q = torch.randn((n, g, d), generator=gen, device=dev).to(dt)
    ref = torch.zeros((n, g, d), device=dev), torch.zeros((n, nb), device=dev)
    got = torch.zeros((n, g, d), device=dev), torch.zeros((n, nb), device=dev)
    size = ctx.workspace_bytes()
    ws = torch.full((size + 4096,), 255, dtype=torch.uint8, device=dev)
    idx = torch.zeros((n, k), dtype=torch.int32, device=dev)
    cnt = torch.full((n,), k, dtype=torch.int32, device=dev)

    def lists(i):
        order = torch.rand((n, nb), generator=gen, device=dev).argsort(dim=1)[:, :k]
        idx.copy_(order.sort(dim=1).values)
        cnt.copy_(torch.tensor([k, 1, k // 2, 0][i % 4]).expand(n))

    def fill(i):
        for x in got:
            x.fill_(7.0)
        if i % 4 == 1:
            ws[:size].random_(0, 256, generator=gen)
        elif i % 4 == 2:
            ws[:size].zero_()
        elif i % 4 == 3:
            ws[:size].fill_(255)

    def check(what):
        ctx.sparse_decode_noalloc(q, K, V, nb * block - 3, idx, cnt, *ref)
        assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1]), what

    lists(0)
    ws[:size].fill_(FILL)
    ctx.sparse_decode(q, K, V, nb * block - 3, idx, cnt, *got, ws)
    assert int((lone_words(ws[:size])[1] == 0).sum()) == n                           # (they are merged inside)
    for i in range(9):
        lists(i)
        fill(i)
        ctx.sparse_decode(q, K, V, nb * block - 3, idx, cnt, *got, ws)
        check(i)
    lists(0)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ctx.sparse_decode(q, K, V, nb * block - 3, idx, cnt, *got, ws)
    for i in range(5):
        lists(i)
        fill(i)
        if i == 2:
            ctx.sparse_decode(q, K, V, nb * block - 3, idx, cnt, *got, ws)      # (a launch of the program's own in between)
        graph.replay()
        check(("replay", i))
        torch.cuda.synchronize()
    assert (ws[size:] == 255).all()
