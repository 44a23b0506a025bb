"""Layer-by-layer network path (forward, backward, loss gradient) at the edges of its workgroup
tiles, reduction blocks and batch chunks, against the f64 oracle with bfloat16 rounding at the same
points.  Rows are independent in the forward pass, so the oracle runs a subset of them; gradients
are checked with an output gradient that is zero outside a subset, whose rows alone contribute."""
import ctypes as C

import numpy as np
import pytest

import oracle
from oracle import mlp as OM

pytestmark = pytest.mark.gpu


def _mlp():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_21784_amd import mlp
    oracle.lib()
    return mlp


def _rel(a, b):
    return float(np.max(np.abs(a - b)) / max(np.max(np.abs(b)), 1e-30))


# 128 x 64, 64 x 64 and 32 x 32 workgroup tiles; widths that end inside a tile and inside a block of
# 64 of the reduction (16, 48, 528, 784); one chunk, several in one workgroup (H >= 720) or in
# workgroups of their own, the last one short (208 and 200 rows of 600; 1 of 257).
SHAPES = [((64, 1024, 16), 2050), ((4, 1024, 3), 1000), ((33, 48, 16), 70), ((64, 16, 1), 17),
          ((10, 528, 9), 300), ((5, 784, 7), 600), ((17, 272, 2), 257)]


@pytest.mark.parametrize("dims,N", SHAPES)
def test_tiles_match_oracle(dims, N):
    import torch
    M = _mlp()
    net = M.MLP(*dims, max_batch=N + 3, seed=1)
    rng = np.random.default_rng(2)
    d_in, H, d_out = dims
    p = net.get_params()
    o = d_in * H
    p[o:o + H] = rng.normal(0, 0.1, H)
    p[o + H + H * H:o + 2 * H + H * H] = rng.normal(0, 0.1, H)
    net.set_params(p)
    p = p.astype(np.float64)
    x = rng.normal(0, 1, (N, d_in)).astype(np.float32)
    rows = np.unique(np.concatenate([[0, N - 1], rng.integers(0, N, 30)]))
    xd = torch.from_numpy(x).cuda()
    y = net.forward(xd).cpu().numpy()
    xs = x[rows].astype(np.float64)
    # fp32 sums in another order flip some bfloat16 roundings; the outputs move by well under 2e-3
    # of their scale, the gradients by under 5e-3 of a block's
    assert _rel(y[rows], OM.forward(p, dims, xs, round_bf16=True)) < 2e-3
    dy = np.zeros((N, d_out), np.float32)
    dy[rows] = rng.normal(0, 1, (len(rows), d_out))
    g = net.backward(xd, torch.from_numpy(dy).cuda()).cpu().numpy().astype(np.float64)
    go = OM.backward(p, dims, xs, dy[rows].astype(np.float64), round_bf16=True)
    for name, a, b in zip(["W1", "b1", "W2", "b2", "W3", "b3"], OM.split(g, dims), OM.split(go, dims)):
        assert _rel(a, b) < 5e-3, (name, _rel(a, b))


@pytest.mark.parametrize("dims,N", [((4, 64, 3), 130), ((9, 1024, 5), 300)])
def test_unaligned_buffers_give_the_same_bits(dims, N):
    """Buffers at odd multiples of their element size: same outputs and gradients."""
    import torch
    M = _mlp()
    from paper_2606_21784_amd import _lib
    net = M.MLP(*dims, max_batch=N, seed=3)
    rng = np.random.default_rng(4)
    x = torch.from_numpy(rng.normal(0, 1, (N, dims[0])).astype(np.float32)).cuda()
    dy = torch.from_numpy(rng.normal(0, 1, (N, dims[2])).astype(np.float32)).cuda()
    y = net.forward(x)
    g = net.backward(x, dy).clone()
    shift = lambda t: torch.cat([t.reshape(-1)[:1], t.reshape(-1)])[1:]
    par, wts, xs, ds = shift(net.params), shift(net.weights), shift(x), shift(dy)
    ws = torch.empty(net.ws.numel() + 4, dtype=torch.uint8, device="cuda")[4:]
    ys, gs = torch.empty(y.numel() + 1, device="cuda")[1:], torch.empty(g.numel() + 1, device="cuda")[1:]
    s = _lib.Mlp(*dims, 0, par.data_ptr(), wts.data_ptr())
    L = _lib.lib()
    assert L.cae_mlp_forward(C.byref(s), xs.data_ptr(), ys.data_ptr(), N, ws.data_ptr(), net.stream) == 0
    assert L.cae_mlp_backward(C.byref(s), xs.data_ptr(), ds.data_ptr(), gs.data_ptr(), N, ws.data_ptr(), net.stream) == 0
    torch.cuda.synchronize()
    assert torch.equal(ys.reshape(y.shape), y) and torch.equal(gs, g)
    m = shift(torch.zeros_like(net.m)), shift(torch.zeros_like(net.v))
    assert L.cae_mlp_adam(C.byref(s), gs.data_ptr(), m[0].data_ptr(), m[1].data_ptr(), 1, 1e-3, 0.9, 0.999, 1e-8,
                          net.stream) == 0
    net.adam(1e-3)
    torch.cuda.synchronize()
    assert torch.equal(par, net.params) and torch.equal(wts, net.weights) and torch.equal(m[1], net.v)


@pytest.mark.parametrize("n", [1, 2048, 2049, 70000])
@pytest.mark.parametrize("delta", [None, 0.1])
def test_loss_gradient_in_place_and_split(n, delta):
    """One workgroup, or the gradient in workgroups of its own; dy may be y itself."""
    import torch
    M = _mlp()
    net = M.MLP(4, 16, 3, max_batch=16, seed=0)
    rng = np.random.default_rng(5)
    y = torch.from_numpy(rng.normal(0, 1, n).astype(np.float32)).cuda()
    t = torch.from_numpy(rng.normal(0, 1, n).astype(np.float32)).cuda()
    r = (y.double() - t.double()).cpu().numpy()
    if delta is None:
        loss, dy = np.mean(r * r), 2 * r / n
    else:
        loss = np.mean(np.where(np.abs(r) <= delta, 0.5 * r * r, delta * (np.abs(r) - 0.5 * delta)))
        dy = np.clip(r, -delta, delta) / n
    out = net.loss_grad(y, t, huber_delta=delta)
    l0 = net.loss.clone()
    same = net.loss_grad(y, t, dy=y, huber_delta=delta)
    assert torch.equal(out, same) and torch.equal(l0, net.loss)
    # r rounds once in fp32 (2^-24 of the larger operand), so dy is off by a few 1e-7 of its scale
    assert np.max(np.abs(out.cpu().numpy() - dy)) < 1e-6 * np.max(np.abs(dy))
    assert abs(float(l0.item()) - loss) < 1e-5 * loss


# two and four groups of rows to a workgroup, one or several blocks of 16 rows to a wave, a
# workgroup with several tiles and a short last one, inputs past 32 columns
@pytest.mark.parametrize("dims,N", [((9, 112, 5), 20000), ((2, 64, 2), 40001), ((64, 16, 16), 5),
                                    ((40, 304, 3), 9000), ((64, 256, 1), 8209)])
def test_predict_tiles_equal_forward(dims, N):
    import torch
    M = _mlp()
    net = M.MLP(*dims, max_batch=8192, seed=6)
    x = torch.from_numpy(np.random.default_rng(7).normal(0, 1, (N, dims[0])).astype(np.float32)).cuda()
    yf = torch.cat([net.forward(x[i:i + 8192].contiguous()) for i in range(0, N, 8192)])
    assert torch.equal(net.predict(x), yf)
