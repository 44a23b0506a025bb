"""Layer-by-layer network path on narrow layers with many rows (H = 16: workgroup tiles of 64 x 16
and output blocks of 64 rows; H = 32: tiles of 32 x 32) and on batches of many chunks of the weight
gradients: at most 256 rows each up to 16384 rows, longer ones of up to 64 beyond, the last one
short.  Outputs have the bits of a batch that takes the small tiles; outputs and gradients agree
with the f64 oracle with bfloat16 rounding at the same points (gradients from an output gradient
that is zero outside a subset of rows)."""
import numpy as np
import pytest

import oracle
from oracle import mlp as OM

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return float(np.max(np.abs(a - b)) / max(np.max(np.abs(b)), 1e-30))


# 16461 rows: 61 chunks of 272, the last one of 141 rows and its last block of 13
@pytest.mark.parametrize("dims,N,chunk", [((3, 16, 2), 16461, 272), ((40, 16, 16), 20031, 320), ((64, 32, 5), 17001, 272),
                                          ((4, 64, 3), 5120, 256), ((9, 48, 4), 16384, 256)])
def test_many_rows_match_oracle(dims, N, chunk):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_21784_amd import mlp
    oracle.lib()
    d_in, H, d_out = dims
    net = mlp.MLP(*dims, max_batch=N, seed=1)
    rng = np.random.default_rng(2)
    p = net.get_params()
    for o in (d_in * H, d_in * H + H + H * H):
        p[o:o + H] = rng.normal(0, 0.1, H)
    net.set_params(p)
    p = p.astype(np.float64)
    x = rng.normal(0, 1, (N, d_in)).astype(np.float32)
    xd = torch.from_numpy(x).cuda()
    small = torch.cat([net.forward(xd[i:i + 1000].contiguous()) for i in range(0, N, 1000)])
    yd = net.forward(xd)
    assert torch.equal(yd, small)
    edges = [0, chunk - 1, chunk, 2 * chunk - 1, 2 * chunk, (N - 1) // chunk * chunk, N - 1]
    rows = np.unique(np.concatenate([edges, rng.integers(0, N, 30)]))
    xs = x[rows].astype(np.float64)
    # fp32 sums in another order flip some bfloat16 roundings; the outputs move by well under 2e-3
    # of their scale, the gradients by under 5e-3 of a block's
    assert _rel(yd.cpu().numpy()[rows], OM.forward(p, dims, xs, round_bf16=True)) < 2e-3
    dy = np.zeros((N, d_out), np.float32)
    dy[rows] = rng.normal(0, 1, (len(rows), d_out))
    g = net.backward(xd, torch.from_numpy(dy).cuda()).cpu().numpy().astype(np.float64)
    go = OM.backward(p, dims, xs, dy[rows].astype(np.float64), round_bf16=True)
    for name, a, b in zip(["W1", "b1", "W2", "b2", "W3", "b3"], OM.split(g, dims), OM.split(go, dims)):
        assert _rel(a, b) < 5e-3, (name, _rel(a, b))
