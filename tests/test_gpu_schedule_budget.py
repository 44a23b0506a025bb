"""The library's own schedule under a caller's LDS budget: what it reports is what it uses, so the
reported schedule passed back with the budget reproduces itself, and both match the oracle."""
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


def _same_as_oracle(E, d, tuning):
    out = []
    for t in (tuning, None):
        ens = E.Ensemble(d, 3, tuning=out[0] if t is None else t)
        ens.step(2)
        st, bk = ens.read_state(), ens.read_books()
        rst, rbk = oracle.run(d, 3, 2)
        assert np.array_equal(bk, rbk)
        for f in ("last", "prev", "n_trade", "sum_vol", "sum_px", "sum_spread", "n_spread"):
            assert np.array_equal(st[f], rst[f]), f
        out.append(ens.tuning())
        ens.close()
    assert out[0] == out[1]
    return out[0]


# order bins of K = 500 take 2 x 8 KB beside a book of 512 bytes; K = 4 takes 2 x 256 bytes
@pytest.mark.parametrize("Ks,budget,overlap", [((500, 500, 500), 4096, False), ((4, 500, 4), 4096, False),
                                               ((4, 4, 4), 4096, True), ((500, 4, 4), 32768, True),
                                               ((1500, 1500, 1500), 65536, False)])
def test_overlap_needs_the_budget(Ks, budget, overlap):
    E = _engine()
    d = np.concatenate([E.markets(64, 600, K, 7) for K in Ks])
    t = _same_as_oracle(E, d, {"max_lds_bytes": budget})
    assert bool(t["overlap"].get(E.size_class(64, 600), 0)) == overlap


# a wave of four packed books of 128 ticks takes 4864 bytes, of two 2432, a book by itself 1152; a
# budget that holds no wave of packed books leaves the markets unpacked
@pytest.mark.parametrize("budget,pack", [(4864, 4), (4863, 2), (2432, 2), (2431, 0), (1152, 0), (0, 4)])
def test_packing_needs_the_budget(budget, pack):
    E = _engine()
    d = np.concatenate([E.markets(128, 16, 8, 7, M=4000), E.markets(20, 30, 2, 7, M=100)])
    t = _same_as_oracle(E, d, {"max_lds_bytes": budget})
    assert set(t["pack"].values()) == ({pack} if pack else set())
