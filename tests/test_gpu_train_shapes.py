"""The fused training step at every hidden width it takes (each has its own code) and at both sides
of the sizes where its loads and sums divide: inputs and outputs of 1, 4, 5, 8, 9 and the largest,
batches of one row, around one 16-row workgroup, one 32-row step, one pass of the parameter
kernel's four waves (1024) and 64 loss partials.  Gradients and loss against the oracle's
back-propagation, the updated parameters against its Adam on the GPU's gradient."""
import numpy as np
import pytest

from oracle import mlp as OM

pytestmark = pytest.mark.gpu

CASES = [((1, 32, 1), 1, None), ((4, 64, 4), 16, 0.05), ((5, 96, 5), 17, None), ((8, 128, 8), 31, 0.05),
         ((9, 160, 9), 33, None), ((17, 192, 12), 1023, 0.05), ((32, 224, 16), 1025, None), ((4, 256, 3), 96, 0.05),
         ((25, 256, 16), 1056, 0.7)]


@pytest.mark.parametrize("indexed", [False, True])
@pytest.mark.parametrize("dims,N,delta", CASES)
def test_step(dims, N, delta, indexed):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_21784_amd import mlp as M
    net = M.MLP(*dims, max_batch=N, seed=3)
    rng = np.random.default_rng(4)
    p0 = net.get_params().astype(np.float64)
    p0 += rng.normal(0, 0.05, p0.size)  # nonzero biases
    net.set_params(p0)
    p0 = net.get_params().astype(np.float64)
    X = rng.normal(0, 1, (N + 9, dims[0])).astype(np.float32)
    T = rng.normal(0, 0.3, (N + 9, dims[2])).astype(np.float32)
    idx = rng.permutation(N + 9)[:N].astype(np.int32) if indexed else np.arange(N, dtype=np.int32)
    loss = net.train_step_fused(torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda(), 1e-3,
                                idx=torch.from_numpy(idx).cuda() if indexed else None, n=N, huber_delta=delta,
                                grads=True)
    xb, tb = X[idx].astype(np.float64), T[idx].astype(np.float64)
    d = OM.forward(p0, dims, xb, round_bf16=True) - tb
    if delta is None:
        dy, ref = 2 * d / d.size, (d * d).mean()
    else:
        small = np.abs(d) <= delta
        dy, ref = np.clip(d, -delta, delta) / d.size, np.where(small, d * d / 2, delta * (np.abs(d) - delta / 2)).mean()
    g = net.grads.cpu().numpy().astype(np.float64)
    go = OM.backward(p0, dims, xb, dy, round_bf16=True)
    # bfloat16 roundings of sums that differ in the last fp32 bits flip now and then: one flip is
    # 2^-8 of one of the products that make up a gradient, in norm well below 1 %
    for name, u, w in zip(["W1", "b1", "W2", "b2", "W3", "b3"], OM.split(g, dims), OM.split(go, dims)):
        assert np.linalg.norm(u - w) <= 1e-2 * np.linalg.norm(w), name
    assert abs(float(loss.item()) - ref) <= 4e-3 * ref
    z = np.zeros(p0.size)
    p1, m1, _ = OM.adam(p0, g, z, z, 1, 1e-3)
    np.testing.assert_allclose(net.get_params(), p1, rtol=1e-5, atol=1e-6)
    np.testing.assert_allclose(net.m.cpu().numpy(), m1, rtol=1e-5, atol=1e-9)
    W = (net.weights.cpu().numpy().view(np.uint16).astype(np.uint32) << 16).view(np.float32)
    W1, _, W2, _, W3, _ = OM.split(net.get_params(), dims)
    want = np.concatenate([W1.ravel(), W2.ravel(), W3.ravel(), W2.T.ravel()])
    np.testing.assert_array_equal(W[:want.size], OM.bf16(want).astype(np.float32))
