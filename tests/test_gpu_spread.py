"""Ensembles of fewer work items than CUs, whose fullest items are halved: uniform and mixed ones,
in descriptor order and longest first, single-wave, lock-step, overlapped, paired and packed markets,
against the oracle."""
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


@pytest.mark.parametrize("keep", [0, 1])
@pytest.mark.parametrize("mode", ["w1", "w2", "ov2", "pairs", "pack"])
@pytest.mark.parametrize("M", [1, 3, 17, 63, 64, 65, 300, 1100])
def test_spread(M, mode, keep):
    E = _engine()
    L, A = 70, 200
    c, c2 = E.size_class(L, A), E.size_class(30, 90)
    d = np.concatenate([E.markets(L, A, 5, 7, n_noise=A - A // 3, n_mom=A // 5, M=M), E.markets(30, 90, 2, 7, M=M // 3 + 1)])
    d = d[np.random.default_rng(M).permutation(len(d))]
    t = {"waves_per_group": 8, "flags": keep, "waves_per_market": {c: 2 if mode in ("w2", "ov2") else 1, c2: 1}}
    if mode == "ov2":
        t["overlap"] = {c: 2}
    if mode == "pairs":
        t["pipelined"] = {c: 1}
    if mode == "pack":
        t["pack"] = {c: 4, c2: 4}
    _check(E, d, t)
