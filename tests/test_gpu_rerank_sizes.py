"""Routing lockstep where the re-rank kernel changes its form: caches whose
candidates (the kept windows and the one that ages) just fill 256, 512 and 1024
threads and just exceed them."""
import pytest

import synthetic as syn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [2, 42])
@pytest.mark.parametrize("kept", [255, 256, 511, 512, 1023, 1024])
def test_rerank_at_thread_count_edges(kept, bits):
    from tests.gpu_harness import Lockstep
    wl = syn.get_workload("c6w8s").replace(prompt_len=5 + 32 + 8 * (kept + 30) + 3, bits=bits,
                                           num_q_heads=4, num_kv_heads=2)
    ls = Lockstep(wl, capacity_full=kept // 4, capacity_quant=kept - kept // 4, steps=17)
    try:
        ls.prefill()
        for _ in range(ls.steps):
            ls.step()
    finally:
        ls.close()
