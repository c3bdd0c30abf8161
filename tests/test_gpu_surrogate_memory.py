"""Device memory of a surrogate context: what grows with max_batch is the activations, the FP32
pre-activations and outputs, and for nets trained layer by layer two buffers of output gradients."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def pad(n):
    return (n + 63) // 64 * 64


@pytest.mark.parametrize("kw, K, rows", [(dict(din=153, width=256, depth=4, dout=6), 5, 65536), (dict(din=20, width=64, depth=7, dout=3), 2, 1 << 20),
                                         (dict(din=70, width=100, depth=0, dout=70), 3, 1 << 20), (dict(din=100, width=300, depth=2, dout=6), 2, 65536)])
def test_bytes_per_row(kw, K, rows):
    import torch
    from paper_1902_09171_amd import rsur
    dp = [pad(kw["din"])] + [pad(kw["width"])] * kw["depth"] + [pad(kw["dout"])]
    row = 2 * dp[0] + K * (2 * sum(dp[1:-1]) + 4 * sum(dp[1:])) + K * 4 / 32       # and the partial losses
    if max(dp) > 256:
        row += K * 2 * 2 * max(dp)
    rsur.Surrogate(ensemble=1, max_batch=64, **kw).close()        # the library loaded
    torch.cuda.synchronize()
    used = []
    for n in (64, rows):
        free = torch.cuda.mem_get_info()[0]
        net = rsur.Surrogate(ensemble=K, max_batch=n, **kw)
        used.append(free - torch.cuda.mem_get_info()[0])
        net.close()
    split = 4 * 8 * K * sum(a * b + b for a, b in zip(dp, dp[1:]))       # the partial sums of up to 8 ranges
    print(f"{kw}: {used[1] - used[0]} bytes more for {rows} rows, expected {row * (rows - 64):.0f} and up to {split}", flush=True)
    assert used[1] - used[0] <= row * rows + split + 2 * (1 << 21) * (4 * len(dp) + 8)   # allocations in pages of 2 MiB
