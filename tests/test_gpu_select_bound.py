"""The selection that ranks the few keys above a lower bound, where it can go wrong: each workgroup size and number of keys
per thread at its edges, 1, 64, 65, 96, 97, 128 and 129 free places (128 groups, 256 groups, radix select), and scores that put the
largest keys into few groups, let too many keys reach the bound, or leave fewer groups with a key than there are places."""
import numpy as np
import pytest
import torch

import oracle.attnpred_oracle as orc

pytestmark = pytest.mark.gpu


def _scores(mode, n_inst, nb, k, rng):
    p = rng.standard_normal((n_inst, nb)).astype(np.float32)
    if mode == "few_groups":                     # the largest keys 512 blocks apart: with them in one group, thousands reach the bound
        p[:, 3::512] += 100.0
    elif mode == "runs":                         # runs of large keys, equal ones among them
        p = np.repeat(rng.integers(0, 5 * k, size=(n_inst, -(-nb // 7))), 7, axis=1)[:, :nb].astype(np.float32)
    elif mode == "zeros":                        # hardly any score but zero, of either sign
        p = np.where(rng.random((n_inst, nb)) < 0.5 * k / nb, p, np.where(rng.random((n_inst, nb)) < 0.5, 0.0, -0.0)).astype(np.float32)
    elif mode == "close":                        # scores that differ in their last digits
        p = (1.0 + 2.0 ** -22 * rng.integers(0, 64, size=(n_inst, nb))).astype(np.float32)
    elif mode == "equal":                        # nothing but one score; the places go to the first blocks
        p[:] = 0.25
    elif mode == "few_values":                   # far more blocks on the last wanted score than there are places
        p = rng.integers(0, 8, size=(n_inst, nb)).astype(np.float32)
    elif mode == "ties_below":                   # fewer distinct large scores than places, the rest a tie
        p = np.zeros((n_inst, nb), np.float32)
        p[:, 1::max(1, nb // max(1, k // 2))] = rng.standard_normal((n_inst, nb))[:, 1::max(1, nb // max(1, k // 2))]
    elif mode == "extreme":
        p[:, ::5] = np.inf
        p[:, 1::5] = -np.inf
        p[:, 2::5] = -np.finfo(np.float32).max
    return p


@pytest.mark.parametrize("n_inst,nb,k,n_sink,n_local", [
    (3, 131, 16, 1, 2), (2, 130, 128, 0, 0), (3, 1024 + 6, 68, 2, 4), (3, 1024 + 7, 69, 1, 4), (2, 2048 + 8, 64, 4, 4),
    (2, 3072 + 4, 132, 4, 0), (2, 3072 + 5, 132, 3, 0), (1, 4096, 129, 0, 0), (2, 4097, 5, 2, 2), (1, 8194, 128, 4, 4),
    (1, 16384 + 8, 128, 4, 4), (1, 16384 + 9, 128, 4, 4), (520, 4096, 72, 4, 4), (520, 4200, 72, 4, 4), (1030, 2304, 65, 0, 1),
    (1030, 2313, 64, 4, 4), (600, 2300, 200, 1, 1), (600, 2500, 200, 0, 1),          # (the last two: 9 and 10 keys a thread, radix select alone)
    (3, 300, 98, 1, 1), (3, 300, 99, 1, 1), (3, 1126, 126, 1, 1), (3, 1027, 126, 1, 1), (520, 3074, 126, 1, 1), (520, 3075, 126, 1, 1),
])
@pytest.mark.parametrize("mode", ["normal", "few_groups", "runs", "zeros", "close", "equal", "few_values", "ties_below", "extreme"])
def test_bit_exact(n_inst, nb, k, n_sink, n_local, mode):
    import paper_2502_04077_amd as ap
    dev = torch.device("cuda:0")
    nb_cap = nb + 3
    ctx = ap.Context(n_inst=n_inst, g=1, head_dim=64, block=8, hist_len=4, t_cap=nb_cap * 8, k_blocks=k, n_sink=n_sink,
                     n_local=n_local, c1=4, c2=4, kv_dtype="f32")
    p = np.full((n_inst, nb_cap), 1e30, np.float32)                     # (what lies beyond the context is larger and not looked at)
    p[:, :nb] = _scores(mode, n_inst, nb, k, np.random.default_rng([nb, k, n_inst]))
    idx = torch.full((n_inst, k), -7, dtype=torch.int32, device=dev)
    cnt = torch.zeros((n_inst,), dtype=torch.int32, device=dev)
    ws = torch.zeros((max(16, ctx.workspace_bytes()),), dtype=torch.uint8, device=dev)
    ctx.select_topk(torch.from_numpy(p).to(dev), nb, idx, cnt, ws)
    idx, cnt = idx.cpu().numpy(), cnt.cpu().numpy()
    assert (cnt == k).all()
    for i in sorted({0, 1, n_inst // 2, n_inst - 1} & set(range(n_inst))):
        assert idx[i].tolist() == orc.select_blocks(p[i].astype(np.float64), nb, k, n_sink, n_local).tolist(), i


@pytest.mark.parametrize("bits", [0xffffffff, 0x7fffffff, 0xffc00000])
def test_scores_that_are_not_numbers(bits):
    """Whichever blocks are chosen: k different ones, inside the context, ascending, the forced ones among them."""
    import paper_2502_04077_amd as ap
    dev = torch.device("cuda:0")
    n_inst, nb, k = 2, 700, 72
    ctx = ap.Context(n_inst=n_inst, g=1, head_dim=64, block=8, hist_len=4, t_cap=nb * 8, k_blocks=k, n_sink=4, n_local=4, c1=4, c2=4, kv_dtype="f32")
    p = np.full((n_inst, nb), bits, np.uint32).view(np.float32).copy()
    p[1, 100:140] = 1.0
    idx = torch.full((n_inst, k), -7, dtype=torch.int32, device=dev)
    cnt = torch.zeros((n_inst,), dtype=torch.int32, device=dev)
    ws = torch.zeros((max(16, ctx.workspace_bytes()),), dtype=torch.uint8, device=dev)
    ctx.select_topk(torch.from_numpy(p).to(dev), nb, idx, cnt, ws)
    idx = idx.cpu().numpy()
    assert (cnt.cpu().numpy() == k).all() and (np.diff(idx, axis=1) > 0).all() and (idx >= 0).all() and (idx < nb).all()
    assert idx[:, :4].tolist() == [[0, 1, 2, 3]] * 2 and idx[:, -4:].tolist() == [[nb - 4, nb - 3, nb - 2, nb - 1]] * 2
