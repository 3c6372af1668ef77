"""Predictor on histories that are zero almost everywhere (what sparse steps push): the kernels leave out what is
zero, so values are planted where leaving out can go wrong - ends of the tile, ends of passes, of 32- and 64-column
words, next to and two columns from each other - and every column is checked against a float64 evaluation."""
import numpy as np
import pytest
import torch

from workloads import n_weight_floats

pytestmark = pytest.mark.gpu


def _reference(hist, blob, c1, c2):
    """(score relative to the all-zero history's, bound on an f16-operand evaluation's error), [n][nb], float64.
    The error: x, w1, y1, b1 and w2 each carry a relative rounding of at most 2^-11 and the ReLUs are 1-Lipschitz, so it
    is below 5 * 2^-11 times the same sums over absolute values, b1 counting wherever a value (or the tile's end) is
    within reach; fp32 sums and f16 subnormals stay below the 1e-7 added by the caller."""
    n, H, nb = hist.shape
    b = torch.from_numpy(blob.astype(np.float64))
    o = np.cumsum([0, 9 * c1, c1, 9 * c1 * c2, c2, c2, 1])
    w1, b1, w2, b2, w3 = (b[o[i]:o[i + 1]] for i in range(5))
    w1, w2 = w1.view(c1, 1, 3, 3), w2.view(c2, c1, 3, 3)
    conv = torch.nn.functional.conv2d

    def net(x):
        y = torch.relu(conv(x[:, None], w1, b1, padding=1))
        return (torch.relu(conv(y, w2, b2, padding=1)).sum(dim=2) / H * w3.view(1, -1, 1)).sum(dim=1)

    p0 = net(torch.zeros((1, H, 9), dtype=torch.float64))[0, 4]
    x = hist.double()
    near = torch.nn.functional.max_pool2d((x != 0).double()[:, None], 3, 1, 1)
    near[:, :, :, 0] = near[:, :, :, -1] = 1.0
    reach = conv(x.abs()[:, None], w1.abs(), padding=1) + b1.abs().view(1, -1, 1, 1) * near
    size = (conv(reach, w2.abs(), padding=1).sum(dim=2) / H * w3.abs().view(1, -1, 1)).sum(dim=1)
    return net(x) - p0, 5 * 2.0 ** -11 * size


def _sparse_row(rng, n, nb, marks):
    """One row per instance: one to three values at marked columns, most of them different for every instance."""
    row = np.zeros((n, nb), dtype=np.float32)
    for i in range(n):
        for j in range(1 + i % 3):
            row[i, marks[(i * 7 + j * (1 + i % 5)) % len(marks)]] = rng.uniform(1e-5, 0.6)
        if i % 11 == 0:
            row[i] = rng.uniform(0, 1e-2, nb)             # and now and then a dense one
    return row


def _passes(n, nb):
    """(columns of a pass, of an instance's last one) as the 8/8 step predictor cuts nb columns of n instances."""
    best = None
    for p in range(-(-nb // 376), -(-nb // 112) + 1):
        cols = -(-nb // p)
        cost = -(-n * -(-nb // cols) // 1024) * (cols + 100)
        if best is None or cost < best[0]:
            best = (cost, cols)
    used = -(-nb // best[1])
    cols = -(-nb // used)
    return cols, nb - (used - 1) * cols


def _passes16(n, nb):
    """The same for the 16/32 step predictor, and the passes of a workgroup."""
    best = None
    for p in range(-(-nb // 252), -(-nb // 62) + 1):
        cols = -(-nb // p)
        cost = -(-n * -(-nb // cols) // 512) * (cols + 100)
        if best is None or cost < best[0]:
            best = (cost, cols)
    used = -(-nb // best[1])
    if -(-n * used // 512) >= 8:                          # many passes a workgroup: the longest ones, and a rest
        used, cols = -(-nb // 252), 252
    else:
        cols = -(-nb // used)
    return cols, nb - (used - 1) * cols, -(-n * used // min(512, n * used))


def _sample(n, c1):
    """Instances that are compared: for 16/32 channels, whose float64 evaluation takes long, 130 of them, the first and the last among them."""
    return list(range(n)) if c1 == 8 or n <= 130 else sorted(set(np.linspace(0, n - 1, 130).astype(int).tolist()))


@pytest.mark.parametrize("c1,c2", [(8, 8), (16, 32)])
@pytest.mark.parametrize("n,nb,H,cols,last", [
    (1040, 752, 8, 251, 250),      # more passes than the chip holds workgroups
    (1040, 377, 6, 189, 188),      # a column more than the longest pass
    (512, 752, 6, 376, 376),       # two of the longest passes per instance, all workgroups at once
    (1100, 376, 6, 188, 188), (1024, 376, 6, 376, 376),
    (128, 2735, 6, 342, 341),      # passes that end in the last of the staged pieces of 64 columns
    (9, 1130, 64, 103, 100),       # few instances: many short passes
    (1, 12433, 6, 112, 1),         # the last pass is one column: the one before reaches beyond the tile
    (2, 12434, 6, 112, 2), (1, 12435, 6, 112, 3), (1, 12436, 6, 112, 4),
    (5, 5, 6, 5, 5), (5, 1, 7, 1, 1), (3, 30, 9, 30, 30), (3, 31, 9, 31, 31), (3, 33, 9, 33, 33), (3, 64, 9, 64, 64),
])
def test_sparse_history_every_column(n, nb, H, cols, last, c1, c2):
    import paper_2502_04077_amd as ap
    assert _passes(n, nb) == (cols, last)
    dev = torch.device("cuda:0")
    check = _sample(n, c1)
    b = 8
    ctx = ap.Context(n_inst=n, g=1, head_dim=64, block=b, hist_len=H, t_cap=(nb + 3) * b, k_blocks=2, n_sink=1, n_local=1,
                     c1=c1, c2=c2, kv_dtype="bf16")
    R, cap = ctx.hist_slots(), ctx.nb_cap()
    rng = np.random.default_rng(nb * 100 + H)
    blob = (rng.standard_normal(n_weight_floats(c1, c2)) * 0.2).astype(np.float32)
    ctx.set_weights(blob)
    ends = [0, 1, 2, 3, nb - 4, nb - 3, nb - 2, nb - 1]
    inner = [x for m in (28, 30, 32, 60, 62, 64, 112, 124, 128, 188, 251, 313, 342, 376, 384) for x in range(m - 5, m + 5)]
    marks = sorted({x for x in ends + inner + list(range(0, nb, 37)) if 0 <= x < nb})
    hist = torch.zeros((n, R, cap), device=dev)
    row, pred, pstate = (torch.zeros((n, cap), device=dev) for _ in range(3))
    ws = torch.zeros((max(16, ctx.workspace_bytes()),), dtype=torch.uint8, device=dev)
    window = np.zeros((n, H, nb), dtype=np.float32)
    n_pushed = 0
    for step in range(H + 9):                             # the planted rows reach every place of the window and leave it
        r = _sparse_row(rng, n, nb, marks) if step % 4 == 0 or step < 3 else np.zeros((n, nb), dtype=np.float32)
        row[:, :nb] = torch.from_numpy(r)
        ctx.update_history(hist, n_pushed, row)
        n_pushed += 1
        window = np.concatenate([window[:, 1:], r[:, None]], axis=1)
        modes = [ap.AP_PRED_ADVANCE] if step > 0 else [ap.AP_PRED_REBASE]
        if step in (1, H // 2, H + 8):
            modes.append(ap.AP_PRED_REBASE)
        ref, bound = _reference(torch.from_numpy(window[check]), blob, c1, c2)
        for mode in modes:
            ctx.predict_incremental(hist, n_pushed, nb, nb, mode, pstate, pred, ws)
            got = pred[check, :nb].cpu().double()
            off = (got - ref).abs() - bound * (2 if mode == ap.AP_PRED_ADVANCE else 1) - 1e-7
            assert off.max() <= 0, f"step {step} mode {mode}: {(off > 0).sum()} columns, worst {off.max():.3g} at {np.unravel_index(int(off.argmax()), off.shape)}"


@pytest.mark.parametrize("n,nb,last", [(6, 12433, 1), (8, 12881, 1), (2, 12434, 2), (1, 12435, 3), (1, 12436, 4), (3, 500, 100)])
def test_tile_end_beside_a_short_last_pass(n, nb, last):
    """Large values in the last five columns of the tile and nowhere else: what lies beyond the tile counts as zero, also for
    a pass that ends a column or two before the tile does.  (A column beyond the tile read as a copy of the last one moves
    scores by up to some 0.01; the bound there is a few 0.001.)"""
    import paper_2502_04077_amd as ap
    assert _passes(n, nb)[1] == last
    dev = torch.device("cuda:0")
    c, b, H = 8, 8, 6
    ctx = ap.Context(n_inst=n, g=1, head_dim=64, block=b, hist_len=H, t_cap=(nb + 3) * b, k_blocks=2, n_sink=1, n_local=1,
                     c1=c, c2=c, kv_dtype="bf16")
    rng = np.random.default_rng(nb)
    blob = (rng.standard_normal(n_weight_floats(c, c)) * 0.2).astype(np.float32)
    ctx.set_weights(blob)
    hist = torch.zeros((n, H + 1, ctx.nb_cap()), device=dev)
    hist[:, :, nb - 5:nb] = torch.from_numpy(rng.uniform(0.5, 1.0, (n, H + 1, 5)).astype(np.float32)).to(dev)
    hist[:, :, nb:] = 7.0                                 # (capacity beyond the context: not read)
    pred, pstate = (torch.zeros((n, ctx.nb_cap()), device=dev) for _ in range(2))
    ws = torch.zeros((max(16, ctx.workspace_bytes()),), dtype=torch.uint8, device=dev)
    window = hist[:, :H, :nb].cpu()                       # (2 H + 1 pushes: rows H + 1 .. 2 H are in slots 0 .. H - 1)
    ref, bound = _reference(window, blob, c, c)
    ctx.predict_incremental(hist, 2 * H + 1, nb, nb, ap.AP_PRED_REBASE, pstate, pred, ws)
    off = (pred[:, :nb].cpu().double() - ref).abs() - bound - 1e-7
    assert off.max() <= 0, f"{(off > 0).sum()} columns, worst {off.max():.3g} at {np.unravel_index(int(off.argmax()), off.shape)}"
    assert bound.max() < 0.1


@pytest.mark.parametrize("n,nb,H,c1,c2,plan", [(*c, 8, 8, None) for c in (
    (1024, 376, 6), (128, 2735, 6), (1040, 377, 7), (6, 12433, 6), (3, 31, 9), (2, 33, 6), (1, 1, 6), (9, 500, 64))] + [
    # 16/32 channels: (columns of a pass, of the last one, passes of a workgroup); a chunk of a list yields 126 outputs
    (512, 126, 6, 16, 32, (126, 126, 1)), (512, 127, 7, 16, 32, (127, 127, 1)), (512, 252, 6, 16, 32, (252, 252, 1)), (700, 505, 6, 16, 32, (169, 167, 5)),
    (3, 1251, 9, 16, 32, (60, 51, 1)), (2, 5, 6, 16, 32, (5, 5, 1)),
    # ... many passes a workgroup: the longest ones, and a rest of any length
    (3600, 252, 6, 16, 32, (252, 252, 8)), (2100, 253, 6, 16, 32, (252, 1, 9)), (2048, 254, 7, 16, 32, (252, 2, 8)), (3600, 128, 6, 16, 32, (252, 128, 8)),
    (2100, 505, 6, 16, 32, (252, 1, 13)), (2050, 379, 64, 16, 32, (252, 127, 9)),
])
def test_dense_history_every_column(n, nb, H, c1, c2, plan):
    """Passes in which every column has a value look nothing up: all of them, all but one column in one half, all but a run in
    both, changing as the rows move on; every column against float64."""
    import paper_2502_04077_amd as ap
    assert plan is None or _passes16(n, nb) == plan
    check = _sample(n, c1)
    dev = torch.device("cuda:0")
    b = 8
    ctx = ap.Context(n_inst=n, g=1, head_dim=64, block=b, hist_len=H, t_cap=(nb + 3) * b, k_blocks=2, n_sink=1, n_local=1,
                     c1=c1, c2=c2, kv_dtype="bf16")
    rng = np.random.default_rng(nb + H)
    blob = (rng.standard_normal(n_weight_floats(c1, c2)) * 0.2).astype(np.float32)
    ctx.set_weights(blob)
    R, cap = ctx.hist_slots(), ctx.nb_cap()
    hist = torch.zeros((n, R, cap), device=dev)
    hist[:, :, :nb] = torch.from_numpy(rng.uniform(1e-3, 0.5, (n, R, nb)).astype(np.float32)).to(dev)
    n_pushed = 3 * R
    hist[0, [(n_pushed + i) % R for i in range(5)], nb // 2] = 0.0          # the top half's rows, or most of them
    hist[n - 1, :, nb // 3:nb // 3 + 40] = 0.0
    if c1 == 16 and n > 100:                              # (lists that are neither empty nor every column, most of them longer than a chunk)
        for i in check[1:-1:3]:
            hist[i, :, (7 * i) % nb:(7 * i) % nb + 6 + i % 50] = 0.0
    row, pred, pstate = (torch.zeros((n, cap), device=dev) for _ in range(3))
    ws = torch.zeros((max(16, ctx.workspace_bytes()),), dtype=torch.uint8, device=dev)
    for step in range(4):
        if step:
            row[:, :nb] = torch.from_numpy(rng.uniform(1e-3, 0.5, (n, nb)).astype(np.float32))
            ctx.update_history(hist, n_pushed, row)
            n_pushed += 1
        mode = ap.AP_PRED_ADVANCE if step else ap.AP_PRED_REBASE
        ctx.predict_incremental(hist, n_pushed, nb, nb, mode, pstate, pred, ws)
        window = hist[check][:, [(n_pushed - H + r) % R for r in range(H)], :nb].cpu()
        ref, bound = _reference(window, blob, c1, c2)
        off = (pred[check, :nb].cpu().double() - ref).abs() - bound * (2 if step else 1) - 1e-7
        assert off.max() <= 0, f"step {step}: {(off > 0).sum()} columns, worst {off.max():.3g} at {np.unravel_index(int(off.argmax()), off.shape)}"
