"""How exact the streaming forms are (sparse decode of lists that are split or streamed whole, bf16 calibration), against
float64: long lists, whose error is that of the additions in a row, and logits that rise, fall or jump from pass to pass, where
the running sums change the maximum they refer to."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


def _context(n, g, d, b, k, cap):
    import paper_2502_04077_amd as ap
    return ap.Context(n_inst=n, g=g, head_dim=d, block=b, hist_len=8, t_cap=cap * b, k_blocks=k, n_sink=0, n_local=0, c1=4, c2=4,
                      kv_dtype="bf16")


def _run(ctx, q, K, V, t, idx):
    dev, n, cap = q.device, q.shape[0], ctx.nb_cap()
    out, row, dense = (torch.full(s, 7.0, device=dev) for s in ((n,) + q.shape[1:], (n, cap), (n, cap)))
    ws = torch.full((max(16, ctx.workspace_bytes()),), 255, dtype=torch.uint8, device=dev)
    cnt = torch.full((n,), idx.shape[1], dtype=torch.int32, device=dev)
    ctx.sparse_decode(q, K, V, t, idx, cnt, out, row, ws)
    ctx.calibrate(q, K, t, dense, ws)
    return out.double(), row.double(), dense.double()


def _exact(q, K, V, t, idx, b, cap):
    """(output, pooled row, dense pooled row) of one instance."""
    d, g = q.shape[-1], q.shape[0]
    logit = q.double() @ K[:t].double().T.contiguous() / math.sqrt(d)
    tok = (idx.long()[:, None] * b + torch.arange(b, device=q.device)).view(-1)
    tok = tok[tok < t]

    def pooled(p, at):
        full = torch.zeros((g, cap * b), dtype=torch.float64, device=q.device)
        full[:, at] = p
        return full.view(g, cap, b).amax(dim=(0, 2))

    p = torch.softmax(logit[:, tok], 1)
    return p @ V[tok].double(), pooled(p, tok), pooled(torch.softmax(logit, 1), torch.arange(t, device=q.device))


@pytest.mark.parametrize("n,g,d,b,k,t", [(300, 2, 128, 16, 250, 4000), (128, 4, 128, 16, 2050, 32790), (512, 4, 64, 16, 64, 4000)])
def test_error_of_long_lists(n, g, d, b, k, t):
    """2-norm of the error over all checked values.  A rounding is 2.6e-8 of the value in the mean square; a chain of 32
    additions (16 at d = 64) and as many sets of it as a wave has make at most 1.8e-7 of a sum of terms of either sign, the
    exponents (up to 8 in units of log2) and the fp32 logits 1e-7 each: 2.3e-7 together, and a third of it to spare.  One chain
    over the whole list gives 3.4e-7 to 4.6e-7."""
    dev = torch.device("cuda:0")
    nb = -(-t // b)
    cap = nb + 3
    gen = torch.Generator(device=dev)
    gen.manual_seed(n)
    K, V = (torch.empty((n, cap * b, d), dtype=torch.bfloat16, device=dev).normal_(generator=gen) for _ in range(2))
    q = torch.randn((n, g, d), generator=gen, device=dev).to(torch.bfloat16)
    k = min(k, nb)
    idx = torch.rand((n, nb), generator=gen, device=dev).topk(k, dim=1).indices.sort(dim=1).values.to(torch.int32).contiguous()
    out, row, dense = _run(_context(n, g, d, b, k, cap), q, K, V, t, idx)
    err, ref = torch.zeros(3, dtype=torch.float64), torch.zeros(3, dtype=torch.float64)
    for i in range(0, n, n // 24):
        for j, (got, want) in enumerate(zip((out[i], row[i], dense[i]), _exact(q[i], K[i], V[i], t, idx[i], b, cap))):
            err[j] += ((got - want) ** 2).sum().item()
            ref[j] += (want ** 2).sum().item()
    assert ((err / ref).sqrt() <= 3.0e-7).all(), (err / ref).sqrt()


@pytest.mark.parametrize("n,g,d,b,t", [(1, 4, 128, 16, 3000), (300, 2, 128, 8, 1500), (260, 8, 64, 32, 2000), (40, 1, 64, 16, 5000)])
@pytest.mark.parametrize("shape", ["rise 10.9", "rise 11.1", "rise 3", "fall 11.1", "last", "first", "jump"])
def test_moving_maximum(shape, n, g, d, b, t):
    """Logits set token by token (one dim of q and K is not zero, so that they are exact), in units of log2: rising or falling by a
    little less or more than the 11 at which a wave rescales its sums, per 64 tokens - a pass of every wave -, one large logit at
    either end, or one far above the rest in the middle.  Exact logits leave the rounding of exponents below 16 and of sums: 1e-6."""
    dev = torch.device("cuda:0")
    nb = -(-t // b)
    cap = nb + 2
    gen = torch.Generator(device=dev)
    gen.manual_seed(t)
    at = torch.arange(t, device=dev)
    level = torch.rand((n, t), generator=gen, device=dev)
    kind, _, step = shape.partition(" ")
    if kind in ("rise", "fall"):
        steps = (at // 64).float() * float(step)
        level += steps if kind == "rise" else steps.flip(0)
    else:
        level[:, {"last": t - 1, "first": 0, "jump": t // 2 + 5}[kind]] += 40.0
    K = torch.full((n, cap * b, d), float("nan"), dtype=torch.bfloat16, device=dev)
    K[:, :t] = 0.0
    K[:, :t, 5] = (level * math.sqrt(d) / (8.0 * math.log2(math.e))).to(torch.bfloat16)
    V = torch.randn((n, cap * b, d), generator=gen, device=dev).to(torch.bfloat16)
    q = torch.zeros((n, g, d), dtype=torch.bfloat16, device=dev)
    q[:, :, 5] = 8.0
    q[:, g - 1, 5] = 4.0 if g > 1 else 8.0
    idx = torch.arange(nb, dtype=torch.int32, device=dev).repeat(n, 1).contiguous()
    got = _run(_context(n, g, d, b, nb, cap), q, K, V, t, idx)
    for i in sorted({0, n // 2, n - 1}):
        for g_i, want in zip((x[i] for x in got), _exact(q[i], K[i], V[i], t, idx[i], b, cap)):
            assert (g_i - want).abs().max() <= 1e-6 * want.abs().max(), (i, (g_i - want).abs().max(), want.abs().max())
