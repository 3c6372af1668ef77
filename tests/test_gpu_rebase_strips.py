"""The full tile (8/8 channels): strips of rows, segments of the time axis, tiles and items of columns, dense
strips and listed columns, each at its edges, every column against float64 - and one more row pushed on the state it leaves."""
import numpy as np
import pytest
import torch

from test_gpu_sparse_rows import _reference
from workloads import n_weight_floats

pytestmark = pytest.mark.gpu


def _rows(mode, rng, n, H, nb):
    x = np.zeros((n, H, nb), np.float32)
    if mode == "dense":
        x = rng.uniform(1e-6, 0.3, (n, H, nb)).astype(np.float32)
    elif mode == "run":                                  # what a decode run leaves: a slowly changing selection, now and then a dense row
        liked = rng.random((n, nb)) < 0.06
        for r in range(H):
            liked ^= rng.random((n, nb)) < 0.004
            row = rng.uniform(1e-5, 0.2, (n, nb))
            x[:, r] = row if r % 31 == 17 else row * liked
    elif mode == "single":                               # one value per instance, wherever it may be; first and last rows and columns first
        rows = [0, 1, 2, 3, H - 1, H - 2, H - 3, H - 4] + list(range(H))
        for i in range(n):
            r = rows[i % len(rows)]
            c = [0, nb - 1, 1, nb - 2, i % nb, (29 * i) % nb, nb // 2][i % 7] % nb
            x[i, r, c] = 0.37
    elif mode == "half":                                 # strips that matter in about half of the columns
        x = rng.uniform(1e-6, 0.3, (n, H, nb)).astype(np.float32) * (np.arange(nb) < nb // 2 + rng.integers(-3, 4, (n, H, 1)))
    return x.astype(np.float32)


@pytest.mark.parametrize("n,nb,H", [
    (3, 1, 6), (3, 2, 7), (4, 55, 64), (4, 57, 64), (2, 113, 8), (40, 300, 64), (30, 241, 65), (1100, 241, 6), (1030, 480, 9),
    (300, 450, 64), (5, 200, 66), (5, 130, 67), (3, 260, 96), (2, 90, 256), (2, 61, 255), (520, 240, 33),
])
@pytest.mark.parametrize("mode", ["zero", "dense", "run", "single", "half"])
def test_full_tile(n, nb, H, mode):
    import paper_2502_04077_amd as ap
    dev = torch.device("cuda:0")
    b, c1, c2 = 8, 8, 8
    ctx = ap.Context(n_inst=n, g=1, head_dim=64, block=b, hist_len=H, t_cap=(nb + 3) * b, k_blocks=2, n_sink=1, n_local=1,
                     c1=c1, c2=c2, kv_dtype="bf16")
    R, cap = ctx.hist_slots(), ctx.nb_cap()
    rng = np.random.default_rng([n, nb, H])
    blob = (rng.standard_normal(n_weight_floats(c1, c2)) * 0.2).astype(np.float32)
    ctx.set_weights(blob)
    x = _rows(mode, rng, n, H + 1, nb)                   # the window, and one row more
    n_pushed = 3 * H + 5 + int(rng.integers(R))
    ring = np.full((n, R, cap), 77.0, np.float32)        # (the slot of the next row and what lies beyond the context are not looked at)
    for r in range(H):
        ring[:, (n_pushed - H + r) % R, :nb] = x[:, r]
    hist = torch.from_numpy(ring).to(dev)
    pred, pstate, row = (torch.zeros((n, cap), device=dev) for _ in range(3))
    ws = torch.zeros((max(16, ctx.workspace_bytes()),), dtype=torch.uint8, device=dev)
    check = sorted({0, 1, n // 2, n - 1} & set(range(n))) if mode != "single" else list(range(min(n, 60)))

    def off(window, slack=0.0):
        ref, bound = _reference(torch.from_numpy(window[check]), blob, c1, c2)
        return ((pred[check, :nb].cpu().double() - ref).abs() - bound - slack - 1e-7).max()

    ctx.predict_incremental(hist, n_pushed, nb, nb, ap.AP_PRED_REBASE, pstate, pred, ws)
    assert off(x[:, :H]) <= 0
    row[:, :nb] = torch.from_numpy(x[:, H])
    ctx.update_history(hist, n_pushed, row)
    ctx.predict_incremental(hist, n_pushed + 1, nb, nb, ap.AP_PRED_ADVANCE, pstate, pred, ws)
    # The state carries the first window's errors, and the row that leaves it is evaluated again, by the other kernel, with errors of
    # its own: a value that left may leave as much as twice the first window's bound.
    assert off(x[:, 1:], 2 * _reference(torch.from_numpy(x[check, :H]), blob, c1, c2)[1]) <= 0
    ctx.predict(hist, n_pushed + 1, nb, pred, ws)        # without a state of the caller's
    assert off(x[:, 1:]) <= 0


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), 1e4])
def test_what_is_not_finite_stays_where_it_is(bad):
    """A value that is not finite (or leaves f16's range: 2^12 x) reaches the columns within two of it and no others."""
    import paper_2502_04077_amd as ap
    dev = torch.device("cuda:0")
    n, nb, H, b, c1, c2 = 3, 300, 64, 8, 8, 8
    ctx = ap.Context(n_inst=n, g=1, head_dim=64, block=b, hist_len=H, t_cap=nb * b, k_blocks=2, n_sink=1, n_local=1, c1=c1, c2=c2, kv_dtype="bf16")
    rng = np.random.default_rng(5)
    ctx.set_weights((rng.standard_normal(n_weight_floats(c1, c2)) * 0.2).astype(np.float32))
    x = _rows("dense", rng, n, H + 1, nb)
    hist = torch.from_numpy(x).to(dev)                   # (H rows pushed after H + 1 others fill the ring in order)
    pred, pstate, ref = (torch.zeros((n, nb), device=dev) for _ in range(3))
    ws = torch.zeros((max(16, ctx.workspace_bytes()),), dtype=torch.uint8, device=dev)
    ctx.predict_incremental(hist, H, nb, nb, ap.AP_PRED_REBASE, pstate, ref, ws)
    for i, col in enumerate((0, 29, 173)):
        hist[i, 30 + i, col] = bad
    ctx.predict_incremental(hist, H, nb, nb, ap.AP_PRED_REBASE, pstate, pred, ws)
    for i, col in enumerate((0, 29, 173)):
        far = (torch.arange(nb, device=dev) - col).abs() > 2
        assert torch.equal(pred[i][far], ref[i][far]), i
