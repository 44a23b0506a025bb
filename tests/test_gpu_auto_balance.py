"""The library's own schedule where workgroups of fewer, larger shares would leave CUs uneven, where
three rows of agents run in lock step, where SplitMix64 markets are many, and where mid-price markets
hold mostly NOISE agents: the rule's choice, and books and states against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

# markets per CU, L, A, K, model ("last", "mid", "split"), NOISE share -> waves per market, overlapped
RULE = [(4.7, 64, 4096, 4, "last", 1.0, 4, True), (4.7, 64, 4096, 4, "split", 1.0, 4, False),
        (7.8, 64, 4096, 4, "last", 1.0, 2, True),  # (already even)
        (8.2, 64, 2048, 4, "last", 1.0, 4, True), (8.2, 64, 1500, 4, "split", 1.0, 2, False),
        (2.34, 64, 4096, 4, "split", 1.0, 8, False), (3.1, 64, 4096, 4, "split", 1.0, 4, False),
        (4.3, 400, 2048, 20, "last", 1.0, 4, False), (4.7, 400, 4096, 20, "last", 1.0, 4, True),
        (4.3, 1000, 2048, 60, "split", 1.0, 4, False), (4.3, 1000, 2048, 60, "mid", 1.0, 2, False),
        (6.25, 64, 512, 4, "split", 1.0, 1, False), (4.7, 64, 512, 4, "split", 1.0, 2, False),
        (0.25, 64, 192, 4, "split", 1.0, 4, False), (0.25, 400, 192, 20, "last", 1.0, 4, False),
        (0.25, 64, 8192, 4, "mid", 1.0, 16, False), (0.25, 64, 8192, 4, "mid", 0.7, 16, True)]


@pytest.mark.parametrize("per_cu,L,A,K,model,noise,w,overlapped", RULE)
def test_choice_and_results(per_cu, L, A, K, model, noise, w, overlapped):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_21784_amd import engine as E
    oracle.lib()
    M = int(per_cu * torch.cuda.get_device_properties(0).multi_processor_count)
    n = int(noise * A)
    mid = model == "mid"
    d = E.markets(L, A, K, 7, M=M, n_noise=n, n_mom=(A - n) // 2, h=2,
                  flags=E.model_flags(int(mid), 0.05 if mid else 0.0, int(model == "split")))
    ens = E.Ensemble(d, 9)
    t = ens.tuning()
    c = E.size_class(L, A)
    assert t["waves_per_market"][c] == w
    assert (t["overlap"].get(c, 0) > 0) == overlapped
    again = E.Ensemble(d, 9, tuning=t)
    assert again.tuning() == t
    again.close()
    ens.step(1)
    ens.step(2)
    st, bk = ens.read_state(), ens.read_books()
    rst, rbk = oracle.run(d, 9, 3)
    assert np.array_equal(bk, rbk)
    for f in ("last", "prev", "n_trade", "sum_vol", "sum_px", "sum_spread", "n_spread", "ref2"):
        assert np.array_equal(st[f], rst[f]), f
    ens.close()
