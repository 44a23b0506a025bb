"""Overlapped mid-price markets on both sides of the flush that places every bin in one pass
(2 (2 K + 1) + 8 <= 64, so K <= 13), in ensembles with and without SplitMix64 markets, and per-step
series on both sides of the lengths at which the waves store them (16 and 64 steps): books,
states and series against the oracle."""
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


def _check(ens, descs, seed, S):
    st, bk = ens.read_state(), ens.read_books()
    rst, rbk = oracle.run(descs, seed, S)
    assert np.array_equal(bk, rbk)
    for f in ("last", "prev", "steps_done", "n_trade", "sum_vol", "sum_px", "sum_spread", "n_spread", "ref2"):
        assert np.array_equal(st[f], rst[f]), f


def _descs(E, mix, L, A, K, M):
    kinds = {"mid": [(1, 0)], "last": [(0, 0)], "mid+last": [(1, 0), (0, 0)], "mid+split": [(1, 0), (1, 1), (0, 1)]}[mix]
    out = []
    for m in range(M):
        model, gen = kinds[m % len(kinds)]
        out.append(E.markets(L, A, K, 1 + 6 * (m % 2), n_noise=(A, A // 2, 0)[m % 3], n_mom=(0, A // 3, A - A // 9)[m % 3],
                             h=min(2 + m % 3, L - 1),
                             flags=E.model_flags(model, 0.05 if model else 0.0, gen)))
    return np.concatenate(out)


@pytest.mark.parametrize("mix", ["mid", "mid+last", "mid+split"])
@pytest.mark.parametrize("K", [1, 13, 14, 40])
@pytest.mark.parametrize("w,ov", [(2, 1), (4, 3)])
def test_overlapped(mix, K, w, ov):
    E = _engine()
    L, A = 200, 450
    d = _descs(E, mix, L, A, K, 12)
    c = E.size_class(L, A)
    ens = E.Ensemble(d, 5, tuning={"waves_per_group": 4, "waves_per_market": {c: w}, "overlap": {c: ov}})
    assert ens.tuning()["overlap"][c] == ov
    ens.step(17)
    ens.step(2)
    _check(ens, d, 5, 19)
    ens.close()


@pytest.mark.parametrize("mix", ["last", "mid", "mid+split"])
@pytest.mark.parametrize("w,ov", [(1, 0), (4, 0), (4, 2)])
@pytest.mark.parametrize("S", [1, 16, 63, 64, 65, 130])
def test_series(mix, w, ov, S):
    import torch
    E = _engine()
    L, A, M = 70, 300, 5
    d = _descs(E, mix, L, A, 6, M)
    c = E.size_class(L, A)
    tn = {"waves_per_group": 4, "waves_per_market": {c: w}}
    if ov:
        tn["overlap"] = {c: ov}
    ens = E.Ensemble(d, 8, tuning=tn)
    price = torch.full((M, S + 5), -7, dtype=torch.int32, device="cuda")
    vol = price.clone()
    ens.step_traced(2, out=(price, None), col=1)  # one series alone
    ens.step_traced(S, out=(price, vol), col=4)
    P, V = price.cpu().numpy(), vol.cpu().numpy()
    _, _, rp, rv = oracle.run(d, 8, S + 2, trace=True)
    want = np.full((2, M, S + 5), -7, np.int64)
    want[0, :, 1:3], want[0, :, 4:4 + S], want[1, :, 4:4 + S] = rp[:, :2], rp[:, 2:], rv[:, 2:]
    assert np.array_equal(P, want[0]) and np.array_equal(V, want[1])
    _check(ens, d, 8, S + 2)
    ens.close()
