"""What a re-base sums, and in which order, is part of its result (8/8 channels): a score moved in its last digits decides blocks whose
scores all but coincide the other way, and with them the selection, the pooled row and the output of a step."""
import os

import numpy as np
import pytest
import torch

from test_gpu_rebase_strips import _rows
from workloads import n_weight_floats

pytestmark = pytest.mark.gpu
GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "rebase_bits.npz")


def _rebased(x, H, blob, spare):
    """Rows x [n][H][nb] re-based in a ring that wraps, the spare slot holding `spare`: (state, pred) [n][nb]."""
    import paper_2502_04077_amd as ap
    dev = torch.device("cuda:0")
    n, nb, b = x.shape[0], x.shape[2], 8
    ctx = ap.Context(n_inst=n, g=1, head_dim=64, block=b, hist_len=H, t_cap=(nb + 3) * b, k_blocks=2, n_sink=1, n_local=1, c1=8, c2=8,
                     kv_dtype="bf16")
    ctx.set_weights(blob)
    R, cap = ctx.hist_slots(), ctx.nb_cap()
    n_pushed = 3 * H + 5 + nb % R
    ring = np.full((n, R, cap), spare, np.float32)
    for r in range(H):
        ring[:, (n_pushed - H + r) % R, :nb] = x[:, r]
    hist = torch.from_numpy(ring).to(dev)
    pred, pstate = (torch.zeros((n, cap), device=dev) for _ in range(2))
    ws = torch.zeros((max(16, ctx.workspace_bytes()),), dtype=torch.uint8, device=dev)
    ctx.predict_incremental(hist, n_pushed, nb, nb, ap.AP_PRED_REBASE, pstate, pred, ws)
    return pstate[:, :nb].cpu().numpy(), pred[:, :nb].cpu().numpy()


def _golden_case(n, nb, H, mode):
    rng = np.random.default_rng([n, nb, H])
    blob = (rng.standard_normal(n_weight_floats(8, 8)) * 0.2).astype(np.float32)
    return _rows(mode, rng, n, H, nb), blob


GOLDEN_CASES = [(4, 57, 64, "run"), (2, 113, 8, "dense"), (3, 67, 67, "run"), (2, 61, 96, "half"), (2, 55, 255, "run"), (3, 2, 7, "dense"),
                (2, 250, 64, "single"), (2, 300, 64, "run")]


@pytest.mark.parametrize("n,nb,H,mode", GOLDEN_CASES)
def test_bits_stay(n, nb, H, mode):
    """State and scores, bit for bit, as tests/golden/rebase_bits.npz has them from a kernel that evaluates every strip of every column."""
    x, blob = _golden_case(n, nb, H, mode)
    state, pred = _rebased(x, H, blob, 0.25)
    with np.load(GOLDEN) as want:
        key = f"{n}_{nb}_{H}_{mode}"
        assert np.array_equal(state.view(np.int32), want[key + "_state"].view(np.int32))
        assert np.array_equal(pred.view(np.int32), want[key + "_pred"].view(np.int32))


@pytest.mark.parametrize("n,nb,H,at", [(40, 700, 64, (50, 411)), (40, 700, 64, (236, 500)), (20, 260, 96, (20, 200)), (30, 2050, 33, (7, 1900))])
def test_equal_windows_have_equal_states(n, nb, H, at):
    """Two columns whose surroundings are the same have the same state and score, whatever else their tiles hold: the one beside
    columns that are all zero, the other beside dense ones, rows that are dense in one tile and not in the other."""
    rng = np.random.default_rng([nb, H, at[0]])
    blob = (rng.standard_normal(n_weight_floats(8, 8)) * 0.2).astype(np.float32)
    x = _rows("run", rng, n, H, nb)
    x[: n // 2, :, nb // 3:] *= rng.random((n // 2, 1, nb - nb // 3)) < 0.05     # sparse to the right, dense rows only on the left
    x[n // 2:, :, nb // 2:] = rng.uniform(1e-6, 0.3, (n - n // 2, H, nb - nb // 2))
    window = _rows("run", rng, n, H, 9) + (rng.random((n, H, 9)) < 0.3) * rng.uniform(1e-6, 0.3, (n, H, 9))
    for c in at:
        x[:, :, c - 4:c + 5] = window
    state, pred = _rebased(x.astype(np.float32), H, blob, 0.0)
    for c in range(-2, 3):                               # (columns within two of the window's middle see nothing beyond it)
        assert np.array_equal(state[:, at[0] + c].view(np.int32), state[:, at[1] + c].view(np.int32))
        assert np.array_equal(pred[:, at[0] + c].view(np.int32), pred[:, at[1] + c].view(np.int32))


@pytest.mark.parametrize("spare", [float("nan"), float("inf"), 1e4])
def test_the_row_that_left_is_not_looked_at(spare):
    rng = np.random.default_rng(3)
    blob = (rng.standard_normal(n_weight_floats(8, 8)) * 0.2).astype(np.float32)
    for H, nb in ((6, 30), (64, 400)):
        x = _rows("run", rng, 3, H, nb)
        want, got = _rebased(x, H, blob, 0.0), _rebased(x, H, blob, spare)
        assert all(np.array_equal(w.view(np.int32), g.view(np.int32)) for w, g in zip(want, got))
