"""Pairs of 8-token windows where a wave's run is longer than the 64 items it describes
ahead, one per lane: the items past those are described one by one, with a split plan
and without one (a routing interval of more than W + 1 steps), runs that end in a
partial (open) window, in a sink window and without a partner."""
import pytest

import synthetic as syn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("splits,kf,kq,R,bits,hq,hkv,sink", [
    (1, 80, 181, 8, 2, 8, 2, 5),       # 261 live and a handful of recent windows: 66 or 67 a wave
    (1, 80, 215, 8, 42, 8, 2, 0),      # 74 or 75 a wave; the last run ends in the open window
    (1, 200, 95, 12, 2, 6, 2, 5),      # the third count of a period has no plan; GQA 3
    (2, 100, 480, 8, 4, 4, 4, 0),      # 73 a wave, eight waves
    (1, 30, 600, 12, 42, 8, 2, 20),    # 158 a wave
])
def test_runs_of_more_than_64_windows(splits, kf, kq, R, bits, hq, hkv, sink):
    from tests.gpu_harness import Lockstep
    wl = syn.get_workload("c6w8s").replace(name=f"w8long{splits}-{kf}-{kq}-{R}", bits=bits, num_q_heads=hq,
                                           num_kv_heads=hkv, retier_interval=R, sink=sink, steps=2 * R + 3,
                                           prompt_len=8 * (kf + kq + 60) + 13)
    ls = Lockstep(wl, capacity_full=kf, capacity_quant=kq, num_splits=splits)
    try:
        ls.run()
        assert ls.events >= 2 and kf + kq > 64 * 4 * splits
    finally:
        ls.close()
