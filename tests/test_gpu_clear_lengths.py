"""cae_clear where books of 33 to 64 ticks take pairs of ticks per lane by their length (L mod 4, and
250 MB of books for odd lengths), and where the longest books on rows of lanes go one to a wave
(350 MB), against the oracle."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,size", [(34, 100000), (50, 100000), (62, 100000), (33, 250000000), (45, 250000000),
                                    (49, 250000000), (63, 250000000), (64, 250000000), (120, 350000000),
                                    (124, 350000000), (128, 350000000)])
@pytest.mark.parametrize("past", [0, 1])
def test_clear_lengths(L, size, past):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_21784_amd import engine as E
    n = size // (8 * L) + past
    g = torch.Generator(device="cuda")
    g.manual_seed(L + past)
    books = torch.randint(0, 50, (n, 2, L), generator=g, device="cuda", dtype=torch.int32)
    edge = torch.randint(0, L + 1, (n, 1), generator=g, device="cuda")
    tick = torch.arange(L, device="cuda")[None, :]
    thin = torch.arange(n, device="cuda")[:, None] % 3 != 0  # most books: bids low, asks high, a few crossing
    books[:, 0] *= ~(thin & (tick > edge + 2))
    books[:, 1] *= ~(thin & (tick < edge - 2))
    rows = np.unique(np.concatenate([np.arange(40), np.arange(n - 40, n), np.random.default_rng(L).integers(0, n, 4000)]))
    rp, rv, rres = O.clear_batch(books[rows].cpu().numpy().view(np.uint32))
    guard = torch.cat([books.reshape(-1), torch.full((16,), 7, dtype=torch.int32, device="cuda")])
    p, v = E.clear_books(guard[:books.numel()], L, n)
    assert np.array_equal(p[rows].cpu().numpy().view(np.uint32), rp)
    assert np.array_equal(v[rows].cpu().numpy().view(np.uint32), rv)
    out = guard[:books.numel()].view(n, 2, L)
    assert np.array_equal(out[rows].cpu().numpy().view(np.uint32), np.asarray(rres).reshape(len(rows), 2, L))
    assert bool((guard[books.numel():] == 7).all())
    # every book: what is taken from its bids is what is taken from its asks, V*
    taken = (books - out).sum(2, dtype=torch.int64)
    assert torch.equal(taken[:, 0], v.long()) and torch.equal(taken[:, 1], v.long())
