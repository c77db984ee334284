"""The two forms of the migration kernel: half a part per wave for routing events of few
windows and a part per wave for larger ones, on both sides of the line between them,
with many promotions an event (slots that a quantization vacates and a promotion fills in
the same event), and the time of a small event."""
import pytest

import synthetic as syn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,bits,rope", [(32, 4, 0.0), (32, 42, 0.0), (32, 2, 5e5), (32, 4, 5e5), (64, 2, 0.0),
                                         (64, 42, 0.0), (64, 4, 5e5), (64, 2, 5e5)])
@pytest.mark.parametrize("R", [1, 16, 17])   # 6, 64 and 68 windows: 192, 2048 and 2176 workgroups
def test_both_forms_match_oracle(W, bits, rope, R):
    from tests.gpu_harness import Lockstep
    wl = syn.get_workload("c2s").replace(name=f"mig{W}-{bits}-{R}", window=W, group=W, bits=bits, num_q_heads=8,
                                         retier_interval=R, steps=6 if R == 1 else 2 * R + 1,
                                         prompt_len=W * 150 + 5)
    # the decay leaves little but the last period's attention, so tiers turn over
    ls = Lockstep(wl, capacity_full=40, capacity_quant=70, score_decay=0.01, rope_base=rope)
    try:
        ls.run()
        # more promotions an event than there are spare slots
        assert ls.promotions > 8 * ls.events, (ls.promotions, ls.events)
    finally:
        ls.close()


@pytest.mark.parametrize("rope,most", [(0.0, 0.9), (5e5, 1.2)])
def test_small_events_take_no_longer_than_the_rerank(rope, most):
    """A routing event after one decode step moves a few windows (4 here); their migrations run
    side by side and take no longer than the re-rank before them (0.81 and 1.0 of its time
    between events around the launches; 0.97 and 1.66 with a wave per part)."""
    import torch
    import paper_2608_05326_amd as qv
    from tests.gpu_harness import gpu_config, to_dev_bf16
    wl = syn.get_workload("c2s").replace(prompt_len=32 * 500 + 5, steps=60)
    c = qv.Cache(gpu_config(wl, 1, capacity_full=8, capacity_quant=150, score_decay=0.01, rope_base=rope))
    try:
        k, v = syn.prompt_kv(wl, 0, 0, 0)
        s = syn.init_scores(wl, 0, 0, 0)
        c.prefill_assign(0, to_dev_bf16(k[None]), to_dev_bf16(v[None]), torch.from_numpy(s[None].copy()).cuda())
        dec = [to_dev_bf16(x[:, None]) for x in syn.decode_inputs(wl, 0, 0, 0, wl.steps)]
        out = torch.empty((1, wl.num_q_heads, 128), device="cuda")
        c.profile_enable()
        moved, at = 0, []
        for t in range(wl.steps):
            c.decode_attend(0, *(x[t] for x in dec), out)
            st = c.retier(0, stats=True)
            moved += st["promotions"] + st["first_quantizations"]
            torch.cuda.synchronize()
            at.append([c.profile_read(i) for i in (2, 3)])
        us = [1e3 * sorted(b[i][0] - a[i][0] for a, b in zip(at[9:], at[10:]))[25] for i in (0, 1)]   # medians
        print(f"re-rank {us[0]:.2f} us, migrations {us[1]:.2f} us an event of {moved / wl.steps:.1f} moves", flush=True)
        assert us[1] <= most * us[0], us
    finally:
        c.close()
