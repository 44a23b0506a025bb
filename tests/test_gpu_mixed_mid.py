"""The library's choice for mixtures with mid-price markets, against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _engine():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_21784_amd import engine
    oracle.lib()
    return engine


def _check(E, d, tuning, S=5):
    ens = E.Ensemble(d, 6, tuning=tuning)
    ens.step(S - 2)
    ens.step(2)
    st, bk = ens.read_state(), ens.read_books()
    rst, rbk = oracle.run(d, 6, S)
    assert np.array_equal(bk, rbk)
    for f in ("last", "prev", "steps_done", "n_trade", "sum_vol", "sum_px", "sum_spread", "n_spread", "ref2"):
        assert np.array_equal(st[f], rst[f]), f
    t = ens.tuning()
    ens.close()
    again = E.Ensemble(d, 6, tuning=t)
    assert again.tuning() == t
    again.close()
    return t


@pytest.mark.parametrize("big,small,n_big,n_small,w,overlapped", [
    ((64, 8192, 4), (64, 64, 4), 0.2, 0.2, 16, False), ((1000, 2048, 60), (64, 256, 4), 1.0, 1.0, 8, False),
    ((1000, 2048, 60), (64, 256, 4), 0.1, 0.1, 16, False), ((256, 1024, 13), (64, 64, 4), 0.2, 0.2, 16, True)])
def test_mixed_mid_price(big, small, n_big, n_small, w, overlapped):
    """n_big and n_small markets per CU."""
    import torch
    E = _engine()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    flags = E.model_flags(1, 0.05)
    d = np.concatenate([E.markets(*big, 7, M=int(n_big * cus), flags=flags), E.markets(*small, 7, M=int(n_small * cus), flags=flags)])
    t = _check(E, d, None, S=3)
    c = E.size_class(*big[:2])
    assert t["waves_per_market"][c] == w and (t["overlap"].get(c, 0) > 0) == overlapped


@pytest.mark.parametrize("n_big,n_small,w", [(0.4, 3.5, 2), (0.1, 0.5, 4)])
def test_mixed_four_rows(n_big, n_small, w):
    """Last-tick markets of four rows of agents beside large ones: two waves where a share of the
    chip's waves in proportion to cost would be less than four (2.0; 10.2 in the second ensemble)."""
    import torch
    E = _engine()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    d = np.concatenate([E.markets(64, 4096, 4, 7, M=int(n_big * cus)), E.markets(64, 256, 4, 7, n_noise=200, n_mom=30, M=int(n_small * cus))])
    t = _check(E, d, None, S=3)
    assert t["waves_per_market"][E.size_class(64, 256)] == w
