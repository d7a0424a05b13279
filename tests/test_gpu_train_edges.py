"""The training kernels at the edges of their blocks (needs an MI355X): 16 rows per block forward
and backward, 128 rows per chunk of the weight gradients.

Every row of a batch is independent, and a gradient is the sum of its rows' gradients, so a
batch is compared with the same rows alone and in other company: outputs bit for bit, gradients
as a sum of two parts.  FP32 sums of n terms in another order differ by at most n 2^-24 of the
sum of their magnitudes; the bfloat16 inputs of the products are the same bits in both."""
import numpy as np
import pytest

from helpers import say

pytestmark = pytest.mark.gpu


def _run(x, dy, wb, params, norm):
    import torch
    import paper_2211_16933_amd as elb
    n = x.shape[0]
    y = torch.full((n, 16), np.nan, dtype=torch.float32, device="cuda:0")
    grad = torch.full_like(params, np.nan)
    # the workspace may hold anything (here NaNs in every format)
    ws = torch.full((elb.mlp_workspace_bytes(n),), 0xff, dtype=torch.uint8, device="cuda:0")
    elb.mlp_forward(params, wb, norm, x, None, n, y, ws)
    elb.mlp_backward(wb, dy, n, grad, ws)
    torch.cuda.synchronize()
    return y.cpu().numpy(), grad.cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("batch", [1, 15, 16, 17, 112, 127, 128, 129, 145, 2049])
def test_batches_at_block_edges(batch):
    import torch
    import paper_2211_16933_amd as elb
    from paper_2211_16933_amd import learned
    say(f"case training kernels batch={batch}")
    rng = np.random.default_rng(batch)
    extra = 37
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a.astype(np.float32))).to("cuda:0")  # noqa: E731
    x, dy = dev(rng.normal(size=(batch + extra, 12))), dev(rng.normal(size=(batch + extra, 16)))
    params = dev(learned.init_params(12, batch))
    norm = dev(learned.make_norm(np.zeros(12), np.ones(12), np.zeros(12), np.ones(12), -np.ones(12), np.ones(12)))
    wb = torch.empty(params.numel(), dtype=torch.int16, device="cuda:0")
    elb.mlp_round(params, wb)
    y, g = _run(x[:batch].contiguous(), dy[:batch].contiguous(), wb, params, norm)
    y2, g2 = _run(x[batch:].contiguous(), dy[batch:].contiguous(), wb, params, norm)
    ya, ga = _run(x, dy, wb, params, norm)
    assert np.array_equal(y, ya[:batch]) and np.array_equal(y2, ya[batch:])
    assert np.all(np.isfinite(g))
    # magnitudes of the summed terms: rows of order-one signals, so about (n rows) times a few
    n = batch + extra
    assert np.max(np.abs(g + g2 - ga)) <= n * 2.0 ** -24 * n * 4.0
