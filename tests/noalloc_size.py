"""What the call without a workspace needs of its 4 MiB of static scratch: the split partials of a context."""


def scratch_bytes(n, g, d, block, k):
    groups = -(-k * block // 16)                           # of 16 tokens, at least one for each of a workgroup's four waves
    want = min(-(-1024 // n), max(1, groups // 4))
    want = max(1, min(max(want, -(-g * k * block * 4 // 32768)), k))
    n_split = -(-k // -(-k // want))
    if n_split == 1:
        return 0
    return 4 * sum(-(-floats // 4) * 4 for floats in (n * n_split * g * 2, n * n_split * g * d, n * g * k))


def fits(n, g, d, block, k):
    return scratch_bytes(n, g, d, block, k) <= 4 << 20
