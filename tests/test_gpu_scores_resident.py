"""Initial window scores where the chunks outnumber the waves the chip holds (the
resident workgroups of k_obs_chunks, each wave several chunks): every window size,
sinks and ragged tails, rows that are not whole tiles and rows beyond one LDS stage,
against the float64 oracle."""
import numpy as np
import pytest

import synthetic as syn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,W,T,n_obs,sink,scale", [
    (8, 32, 4163, 40, 0, 2.0),      # 66 chunks x 64 (sequence, head) pairs: one or two a wave
    (8, 64, 4485, 33, 37, 2.0),     # sink inside a chunk, 66 rows
    (8, 8, 4171, 40, 100, 2.0),     # two sink chunks, 8-token windows
    (8, 32, 13001, 300, 5, 1.0),    # 600 rows (two LDS stages), 204 chunks: six or seven a wave
    (8, 32, 4200, 50, 0, 60.0),     # logits spread over hundreds of octaves
    (17, 32, 2041, 40, 0, 2.0),     # 136 pairs x 32 chunks: workgroups that cross from pair to pair
    (33, 8, 1067, 33, 3, 2.0),      # 264 pairs x 17 chunks, the last round of a pair with one
    (5, 32, 13001, 300, 5, 1.0),    # 40 pairs, two LDS stages within each part
])
def test_resident_chunk_pass_matches_oracle(B, W, T, n_obs, sink, scale):
    import torch
    import paper_2608_05326_amd as qv
    from oracle.qevict_oracle import prefill_window_scores
    from tests.gpu_harness import to_dev_bf16
    H_q, H_kv, at = 16, 8, 3 if B < 16 else B - 2
    rng = np.random.default_rng(W + T + n_obs)
    bits = lambda *s: syn.f32_to_bf16_bits(rng.standard_normal(s, dtype=np.float32))   # noqa: E731
    q1 = syn.f32_to_bf16_bits(scale * rng.standard_normal((H_q, n_obs, 128)).astype(np.float32))
    k1 = bits(H_kv, T, 128)
    q = to_dev_bf16(q1).expand(B, -1, -1, -1).contiguous()
    k = torch.randn(B, H_kv, T, 128, device="cuda").bfloat16()
    k[at] = to_dev_bf16(k1)
    cfg = qv.Config(batch=B, num_q_heads=H_q, num_kv_heads=H_kv, window_tokens=W, quant_bits=4,
                    max_context=T + 64, capacity_full=4, capacity_quant=4, sink_tokens=sink)
    cache = qv.Cache(cfg)
    try:
        got = cache.prefill_scores(q, k)
        again = cache.prefill_scores(q, k)
        assert torch.equal(got, again)
        total = got.double().sum(1).cpu().numpy()
        got = got[at].cpu().numpy().astype(np.float64)
    finally:
        cache.close()
    ref = prefill_window_scores(syn.bf16_bits_to_f32(q1).astype(np.float64),
                                syn.bf16_bits_to_f32(k1).astype(np.float64), sink, W)
    # fp32 logits of magnitude x carry an error near 2^-23 x, which the exponential
    # turns into the relative error of a mass
    x = 128 ** 0.5 * scale * 4
    tol = max(1e-5, 8 * x * 2.0 ** -23)
    err = np.abs(got - ref) / np.maximum(np.abs(ref), 1e-7 * ref.sum())
    assert err.max() <= tol, err.max()
    if sink == 0:   # all mass lies in windows
        assert np.allclose(total, n_obs, rtol=tol)


@pytest.mark.parametrize("full,over", [(16, 17), (32, 33)])
def test_one_sequence_more_than_fills_the_chip(full, over):
    """128 and 256 (sequence, KV head) pairs fill the 256 compute units evenly; one sequence
    more costs its share of the keys and a second staging (1.13 and 1.06 times the time), not
    idle units or a second wave of workgroups (1.42, 1.48)."""
    import torch
    import paper_2608_05326_amd as qv
    H_q, H_kv, T, n_obs = 32, 8, 8192, 32

    def caller(B):
        cfg = qv.Config(batch=B, num_q_heads=H_q, num_kv_heads=H_kv, window_tokens=32, quant_bits=4,
                        max_context=T + 64, capacity_full=4, capacity_quant=4)
        cache = qv.Cache(cfg)
        k = torch.randn(B, H_kv, T, 128, device="cuda").bfloat16()
        q = torch.randn(B, H_q, n_obs, 128, device="cuda").bfloat16()
        scores = torch.empty(B, T // 32, device="cuda")
        scratch = torch.empty(qv.qevict.prefill_scores_scratch_size(cfg, T, n_obs), dtype=torch.uint8, device="cuda")
        return lambda: cache.prefill_scores(q, k, scores, scratch)

    calls = caller(full), caller(over)
    us = [[], []]
    for _ in range(25):   # in turn; the first ones warm up
        for call, t in zip(calls, us):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                call()
            b.record()
            torch.cuda.synchronize()
            t.append(a.elapsed_time(b) * 100)
    one, more = (sorted(t[10:])[7] for t in us)
    print(f"{full}: {one:.1f} us, {over}: {more:.1f} us", flush=True)
    assert more <= 1.25 * one
