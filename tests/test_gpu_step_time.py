"""cae_last_step_ms (device clock, first workgroup's start to last one's end) against events around
the call, for launches whose items all fit at once, launches that claim items from the queue, and
the naive engine; and its error before any step."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,S,tuning", [(3, 400, None), (600, 50, {"groups_per_cu": 1, "waves_per_group": 4}),
                                        (5000, 30, {"groups_per_cu": 1, "waves_per_group": 1})])
@pytest.mark.parametrize("naive", [False, True])
def test_last_step_ms(M, S, tuning, naive):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_21784_amd import _lib, engine
    ens = engine.Ensemble(engine.markets(64, 300, 4, 10, M=M), 5, tuning=tuning)
    with pytest.raises(_lib.CaeError):
        ens.last_step_ms()
    call = ens.step_naive if naive else ens.step
    call(1)
    last = ens.last_step_ms()
    for _ in range(3):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        call(S)
        e1.record()
        torch.cuda.synchronize()
        ms, around = ens.last_step_ms(), e0.elapsed_time(e1)
        # inside the events (to their own few us), and most of what lies between them
        assert 0.0 < ms <= around + 0.01 and ms >= 0.5 * around - 0.05, (ms, around)
        assert ms != last
        last = ms
    ens.close()
