"""The library's own schedule (no tuning given) on both sides of the lines its rules draw: books,
states and statistics against the oracle, and the reported schedule passed back reproduces itself."""
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
    for f in ("sum_r", "sum_r2"):
        assert np.allclose(st[f], rst[f], rtol=1e-6, atol=0.0), f


# (markets, L, A, K), what the rule should pick: packed four or two to a wave, one wave, several
# waves with or without the overlapped schedule
UNIFORM = [((2048, 20, 32, 2), {"pack": 4}), ((2047, 20, 32, 2), {"w": 1}), ((4100, 128, 50, 8), {"pack": 2}),
           ((8192, 5, 128, 1), {"pack": 4}), ((5, 64, 129, 4), {"w": 2, "ov": 1}), ((5, 64, 128, 4), {"w": 1}),
           ((700, 64, 300, 4), {"w": 2, "ov": 1}), ((1024, 256, 1024, 16), {"w": 4, "ov": 4}),
           ((3, 1024, 700, 64), {"w": 4, "ov": 0}), ((3, 512, 2100, 32), {"w": 16, "ov": 1}),
           ((3, 64, 5000, 1022), {"w": 16}), ((3, 64, 5000, 1500), {"w": 16})]


@pytest.mark.parametrize("shape,want", UNIFORM)
def test_uniform_rule(shape, want):
    E = _engine()
    M, L, A, K = shape
    d = E.markets(L, A, K, 7, M=M, n_noise=A - A // 3, n_mom=A // 5, h=min(2, L - 1))
    ens = E.Ensemble(d, 9)
    t = ens.tuning()
    c = E.size_class(L, A)
    assert t["pack"].get(c, 0) == want.get("pack", 0)
    if "w" in want:
        assert t["waves_per_market"][c] == want["w"]
    if "ov" in want:
        assert t["overlap"].get(c, 0) == want["ov"]
    again = E.Ensemble(d, 9, tuning=t)
    assert again.tuning() == t
    S = 3
    for e in (ens, again):
        e.step(S - 1)
        e.step(1)
        _check(e, d, 9, S)
        e.close()


@pytest.mark.parametrize("mid", [0, 1])
@pytest.mark.parametrize("M", [8, 300])
def test_mixed_rule(M, mid):
    E = _engine()
    rng = np.random.default_rng(3)
    flags = E.model_flags(mid, 0.05 if mid else 0.0)
    d = np.concatenate([E.markets(int(L), int(A), max(1, int(L) // 16), 7, n_noise=int(A) // 2, n_mom=int(A) // 4,
                                  flags=flags if k % 2 else 0)
                        for k, (L, A) in enumerate(zip(rng.choice([64, 200, 256, 512, 1024], M),
                                                       np.rint(np.exp(rng.uniform(3, 8.5, M)))))])
    ens = E.Ensemble(d, 4)
    t = ens.tuning()
    again = E.Ensemble(d, 4, tuning=t)
    assert again.tuning() == t
    for e in (ens, again):
        e.step(4)
        _check(e, d, 4, 4)
        e.close()


def test_callers_limits_are_kept():
    """A group size below what the class needs is refused as before; above it, the library's waves
    fit the group; an LDS budget without room for the order bins turns the overlap off."""
    E = _engine()
    from paper_2606_21784_amd import _lib
    d = E.markets(64, 4096, 4, 7, M=3)
    with pytest.raises(_lib.CaeError):
        E.Ensemble(d, 1, tuning={"waves_per_group": 4})
    ens = E.Ensemble(d, 1, tuning={"waves_per_group": 8})
    assert set(ens.tuning()["waves_per_market"].values()) == {8}
    ens.step(2)
    _check(ens, d, 1, 2)
    ens.close()
    d = E.markets(64, 600, 500, 7, M=3)
    ens = E.Ensemble(d, 1, tuning={"max_lds_bytes": 4096})
    ens.step(2)
    _check(ens, d, 1, 2)
    ens.close()
