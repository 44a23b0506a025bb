"""cae_mlp_predict where some waves have no tile of columns, or one instead of two, and where a
narrow layer's spare waves take rows: same bits as the layer-by-layer forward pass."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# one tile of columns on 4, 2 and 1 waves (H = 16: 64, 128 and 256 rows to a tile); two on 4 and 2,
# with one and two blocks of rows to a wave; three and five tiles on 4 and 8 waves; 17 .. 31 tiles
# on 16 waves with one, two or four blocks; up to four and up to eight input values per thread;
# inputs of one and of two steps; short last tiles
@pytest.mark.parametrize("dims,N", [((4, 16, 3), 7), ((4, 16, 3), 16385), ((15, 16, 16), 32769), ((16, 16, 2), 70001),
                                    ((17, 16, 1), 70001), ((40, 16, 16), 70001), ((64, 16, 5), 16400), ((9, 32, 2), 17001),
                                    ((2, 32, 16), 40001), ((64, 32, 1), 17001), ((64, 48, 1), 16999), ((40, 48, 7), 300),
                                    ((5, 80, 4), 8200), ((33, 208, 3), 4100), ((4, 272, 3), 1), ((40, 272, 3), 4100),
                                    ((64, 288, 16), 8201), ((4, 400, 3), 8201), ((48, 448, 2), 8200), ((33, 464, 16), 4500),
                                    ((4, 496, 3), 8201)])
def test_predict_equals_forward(dims, N):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_21784_amd import mlp
    d_in, H, d_out = dims
    net = mlp.MLP(*dims, max_batch=8192, seed=d_in + H)
    rng = np.random.default_rng(N)
    p = net.get_params()
    for o in (d_in * H, d_in * H + H + H * H):
        p[o:o + H] = rng.normal(0, 0.1, H)
    net.set_params(p)
    x = torch.from_numpy(rng.normal(0, 1, (N, d_in)).astype(np.float32)).cuda()
    yf = torch.cat([net.forward(x[i:i + 8192].contiguous()) for i in range(0, N, 8192)])
    guard = torch.full((N * d_out + 64,), 7.0, device="cuda")
    net.predict(x, guard[:N * d_out].view(N, d_out))
    assert torch.equal(guard[:N * d_out].view(N, d_out), yf)
    assert bool((guard[N * d_out:] == 7.0).all())
