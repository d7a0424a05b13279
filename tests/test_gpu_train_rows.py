"""The training kernels' rows (needs an MI355X): every row of a batch is in its outputs and gradients,
at batches where a block of the forward takes 1, 2, 4 and 8 tiles of 16 rows, with remainders.

A batch is compared with its two parts run alone.  The rows of the second part, the batch's last
ones, carry an output gradient 1000 times the others', so that one missing row stands far above
the rounding of the sums: FP32 sums of 128-row chunks, added in order, are off by at most
(128 + chunks) 2^-24 of the sum of the terms' magnitudes, which is formed in FP64 on the CPU."""
import numpy as np
import pytest

from helpers import say

pytestmark = pytest.mark.gpu

def _magnitudes(params, x, dy):
    """Per weight and bias, sum over the rows of |dz| |a| and |dz| (FP64, without roundings)."""
    from paper_2211_16933_amd import learned
    p = learned.unpack_params(params, 16)
    weights, biases = p[0::2], p[1::2]
    a, acts, zs = x, [], []
    for w, b in zip(weights, biases):
        acts.append(np.abs(a))
        zs.append(a @ w.T + b)
        a = zs[-1] / (1.0 + np.exp(-zs[-1]))
    g, out = dy, [None] * 8
    for i in (3, 2, 1, 0):
        out[2 * i], out[2 * i + 1] = np.abs(g).T @ acts[i], np.abs(g).sum(0)
        if i:
            s = 1.0 / (1.0 + np.exp(-zs[i - 1]))
            g = (g @ weights[i]) * (s * (1.0 + zs[i - 1] * (1.0 - s)))
    return learned.pack_params(out).astype(np.float64)


@pytest.mark.parametrize("batch,tail", [(1, 1), (16, 1), (129, 1), (2049, 16), (32800, 17), (65537, 1), (131072 + 130, 2)])
def test_every_row_counts(batch, tail):
    import torch
    import paper_2211_16933_amd as elb
    from paper_2211_16933_amd import learned
    say(f"case rows batch={batch} tail={tail}")
    rng = np.random.default_rng(batch)
    n = batch + tail
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")  # noqa: E731
    hx, hdy = rng.normal(size=(n, 12)).astype(np.float32), rng.normal(size=(n, 16)).astype(np.float32)
    hdy[batch:] *= 1e3
    x, dy, hp = dev(hx), dev(hdy), learned.init_params(16, batch)
    params = dev(hp)
    norm = dev(learned.make_norm(np.zeros(12), np.ones(12), np.zeros(16), np.ones(16), -np.ones(12), np.ones(12)))
    wb = torch.empty(params.numel(), dtype=torch.int16, device="cuda:0")
    elb.mlp_round(params, wb)

    def run(lo, hi, index=None):
        m = hi - lo
        y = torch.full((m, 16), np.nan, dtype=torch.float32, device="cuda:0")
        g = torch.full_like(params, np.nan)
        # the workspace may hold anything (here NaNs in every format)
        ws = torch.full((elb.mlp_workspace_bytes(m),), 0xff, dtype=torch.uint8, device="cuda:0")
        elb.mlp_forward(params, wb, norm, x if index is not None else x[lo:hi].contiguous(), index, m, y, ws)
        elb.mlp_backward(wb, dy[lo:hi].contiguous(), m, g, ws)
        torch.cuda.synchronize()
        return y.cpu().numpy(), g.cpu().numpy().astype(np.float64)

    ya, ga = run(0, n)
    y1, g1 = run(0, batch)
    y2, g2 = run(batch, n)
    assert np.array_equal(ya, np.concatenate([y1, y2])) and np.all(np.isfinite(ga))
    perm = rng.permutation(n).astype(np.int32)
    yp, _ = run(0, n, dev(perm))
    assert np.array_equal(yp, ya[perm])
    # bf16 operands are off by 2^-9 each, their products' magnitudes by a few per cent at most
    mag = 1.1 * _magnitudes(hp, hx.astype(np.float64), hdy.astype(np.float64)) + 1e-30
    tol = 2.0 * (128 + n / 128 + 2) * 2.0 ** -24 * mag
    assert np.all(np.abs(g1 + g2 - ga) <= tol)
    # and the last rows alone stand above it
    used = mag > 1e-6
    assert np.median(np.abs(g2[used]) / tol[used]) > 10.0
