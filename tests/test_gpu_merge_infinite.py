"""An infinite value in the recent window stays an infinity in its channel (and changes
no other) at split counts that leave the merge's last round partly empty: the recent
window lies in the last split, whose row the empty places read again.  (Not with
8-token windows: two share a matrix product there, and the other's zero
probabilities times an infinity are NaN.)"""
import numpy as np
import pytest

import synthetic as syn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,splits", [(32, 1), (32, 8), (32, 16), (32, 31), (32, 33), (64, 16)])
def test_infinite_recent_value(W, splits):
    import torch
    import paper_2608_05326_amd as qv
    from tests.gpu_harness import to_dev_bf16
    H_q, H_kv, T = 8, 2, 40 * W
    rng = np.random.default_rng(W + splits)
    bits = lambda *s: syn.f32_to_bf16_bits(0.1 * rng.standard_normal(s, dtype=np.float32))   # noqa: E731
    k, v = to_dev_bf16(bits(1, H_kv, T, 128)), to_dev_bf16(bits(1, H_kv, T, 128))
    q, kn, vn = (to_dev_bf16(bits(1, h, 128)) for h in (H_q, H_kv, H_kv))
    cfg = qv.Config(batch=1, num_q_heads=H_q, num_kv_heads=H_kv, window_tokens=W, quant_bits=4,
                    max_context=T + 64, capacity_full=8, capacity_quant=32, num_splits=splits)
    outs = []
    for bad in (None, float("inf"), float("-inf")):
        x = vn.clone()
        if bad is not None:
            x[0, 1, 5] = bad     # one channel of the second KV head's new value
        c = qv.Cache(cfg)
        try:
            c.prefill_assign(0, k, v, torch.ones(1, T // W, device="cuda"))
            out = torch.empty(1, H_q, 128, device="cuda")
            c.decode_attend(0, q, kn, x, out)
            outs.append(out.cpu())
        finally:
            c.close()
    assert torch.isfinite(outs[0]).all()
    for out, bad in zip(outs[1:], (float("inf"), float("-inf"))):
        want = outs[0].clone()
        want[0, H_q // 2:, 5] = bad
        assert torch.equal(out, want), (out - want).abs().nan_to_num(9e9).max()
