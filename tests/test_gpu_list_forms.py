"""Lists as the header allows them - entries outside the context, which are clamped into it and may then come twice - give the
same attention and the same pooled row whether a list is cut into splits or streamed whole: a column holds the largest probability
of its block, wherever in the list the block stands.  Against float64; tolerance as in test_gpu_stream_decode.py."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,g,d,b,k,nb", [
    (8, 4, 128, 16, 40, 90),        # split
    (300, 4, 128, 16, 40, 90),      # whole lists, one workgroup per instance
    (400, 2, 64, 8, 33, 70),
    (1030, 8, 64, 16, 12, 40),      # whole lists, g = 8
])
def test_clamped_entries(n, g, d, b, k, nb):
    import paper_2502_04077_amd as ap
    dev = torch.device("cuda:0")
    t = nb * b - 5
    ctx = ap.Context(n_inst=n, g=g, head_dim=d, block=b, hist_len=8, t_cap=(nb + 3) * b, k_blocks=k, n_sink=0, n_local=0, c1=4, c2=4,
                     kv_dtype="bf16")
    gen = torch.Generator(device=dev)
    gen.manual_seed(n)
    K, V = (torch.randn((n, (nb + 3) * b, d), generator=gen, device=dev).to(torch.bfloat16) for _ in range(2))
    q = (3 * torch.randn((n, g, d), generator=gen, device=dev)).to(torch.bfloat16)
    rng = np.random.default_rng(n)
    idx = np.sort(rng.choice(nb, size=(n, k), replace=True), axis=1).astype(np.int32)
    idx[:, :3] = [-7, -2, -1]
    idx[:, -2:] = [nb, 1 << 30]
    idx = np.sort(idx, axis=1)
    cnt = np.where(np.arange(n) % 4 == 1, 5, k).astype(np.int32)
    out, row = torch.full((n, g, d), 7.0, device=dev), torch.full((n, nb + 3), 7.0, device=dev)
    ws = torch.full((max(16, ctx.workspace_bytes()),), 255, dtype=torch.uint8, device=dev)
    ctx.sparse_decode(q, K, V, t, torch.from_numpy(idx).to(dev), torch.from_numpy(cnt).to(dev), out, row, ws)
    for i in (0, 1, 2, n // 2, n - 1):
        blocks = np.clip(idx[i, :cnt[i]], 0, nb - 1)
        tok = (blocks[:, None] * b + np.arange(b)).ravel()
        tok = torch.from_numpy(tok[tok < t]).to(dev)
        p = torch.softmax(q[i].double() @ K[i, tok].double().T.contiguous() / math.sqrt(d), dim=1)
        ref = p @ V[i, tok].double()
        ref_row = torch.zeros(nb + 3, dtype=torch.float64, device=dev)
        ref_row.scatter_reduce_(0, tok // b, p.amax(dim=0), "amax")
        assert (out[i].double() - ref).abs().max() <= 2e-5 * ref.abs().max(), i
        assert (row[i].double() - ref_row).abs().max() <= 2e-5 * ref_row.max(), i
