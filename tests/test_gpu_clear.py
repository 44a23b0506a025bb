"""cae_clear where its rules change: books on rows of 16 lanes (up to 128 ticks) or whole waves,
1, 2, 4 or 8 ticks per lane, one, two or four chunks of 256 ticks, lanes that hold part of their
ticks, waves with fewer books than rows; against the oracle."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [1, 3, 16, 17, 31, 32, 33, 48, 63, 64, 65, 100, 127, 128, 129, 255, 256, 257, 259, 511,
                               512, 513, 767, 769, 1021, 1024])
def test_clear_edges(L):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_21784_amd import engine as E
    rng = np.random.default_rng(L)
    for n in (1, 3, 66):
        books = np.zeros((n, 2, L), np.uint32)
        for i in range(n):
            hi = int(rng.choice([1, 2, 50, 2**31 // L]))
            books[i] = rng.integers(0, hi, (2, L))
            if i % 3 == 1:  # bids below, asks above: nothing trades; or one side empty
                c = int(rng.integers(0, L + 1))
                books[i, 0, c:] = 0
                books[i, 1, :c] = 0
        rp, rv, rres = O.clear_batch(books)
        dev = torch.from_numpy(books.reshape(-1).view(np.int32).copy()).cuda()
        guard = torch.cat([dev, torch.full((16,), 7, dtype=torch.int32, device="cuda")])
        p, v = E.clear_books(guard[:dev.numel()], L, n)
        assert np.array_equal(p.cpu().numpy().view(np.uint32), rp)
        assert np.array_equal(v.cpu().numpy().view(np.uint32), rv)
        assert np.array_equal(guard[:dev.numel()].cpu().numpy().view(np.uint32), np.asarray(rres).reshape(-1))
        assert bool((guard[dev.numel():] == 7).all())
