"""Split merge where a thread holds more than eight split rows or statistics: just past
eight, partial blocks of eight and the largest split counts, against the oracle."""
import pytest

import synthetic as syn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,splits", [("c2s", 33), ("c2s", 65), ("c2s", 127), ("c6w8s", 128),
                                         ("c5s", 33), ("c5s", 63), ("c5s", 64)])   # 64 heads
def test_merge_of_many_splits(name, splits):
    from tests.gpu_harness import Lockstep
    ls = Lockstep(syn.get_workload(name), num_splits=splits, steps=10)
    try:
        ls.run()
    finally:
        ls.close()


@pytest.mark.parametrize("splits", [129, 256])
def test_merge_of_most_splits(splits):
    from tests.gpu_harness import Lockstep
    wl = syn.get_workload("c2s").replace(num_q_heads=8, num_kv_heads=2)
    ls = Lockstep(wl, num_splits=splits, steps=10)
    try:
        ls.run()
    finally:
        ls.close()
