"""Codes, scales and promoted values of prompt windows whose values sit where the
fp32 code decision could go wrong: exact half steps, values far below the scale,
zero points near zero, constant and single-outlier groups, the ends of fp16.  And what
is no number or outside fp16: reported, or left out of its group."""
import numpy as np
import pytest

import synthetic as syn

pytestmark = pytest.mark.gpu


def edge_windows(rng, H, W, d):
    """[n, H, W, d] float32 windows of bf16 values."""
    n01 = lambda: rng.standard_normal((H, W, d))   # noqa: E731
    ws = [
        n01(),
        rng.integers(-15, 16, (H, W, d)) / 4.0,                    # every quotient on a half-step grid
        rng.integers(0, 31, (H, W, d)) / 2.0,                      # zero point 0, ties
        rng.integers(-3, 4, (H, W, d)) * 0.5 + 2.0 ** -24,         # ties missed by less than fp32 resolves
        n01() * 2.0 ** rng.integers(-30, 1, (H, W, d)),            # values far below the scale
        np.abs(n01()) * 2.0 ** rng.integers(-40, 8, (H, W, d)),    # zero points near zero
        np.abs(n01()) + 2.0 ** -20,                                # positive groups
        np.full((H, W, d), 1.7),                                   # scale 0
        np.where(rng.random((H, W, d)) < 0.05, n01() * 1000, n01() * 1e-3),
        n01() * 60000 / 5.5,                                       # ends of fp16
        n01() * 2.0 ** -24,                                        # fp16 subnormals
        n01() * 1e-12,                                             # far below fp16
        np.where(rng.random((H, W, d)) < 0.5, 0.0, n01()),
        np.where(rng.random((H, W, d)) < 0.5, -0.0, -np.abs(n01())),
    ]
    x = np.clip(np.stack(ws), -65000, 65000).astype(np.float32)
    return syn.bf16_bits_to_f32(syn.f32_to_bf16_bits(x))


@pytest.mark.parametrize("bits", [4, 2])
@pytest.mark.parametrize("W", [8, 32, 64])
def test_codes_and_promotions_on_edge_values(W, bits):
    import torch
    import paper_2608_05326_amd as qv
    from oracle.numerics import from_bf16_bits, from_fp16_bits, rne_bf16
    from oracle.qevict_oracle import dequantize_window, quantize_window
    H, d, G = 2, 128, 32 if W == 8 else W
    rng = np.random.default_rng(100 * W + bits)
    reps = 6 if W == 8 else 2
    kw = np.concatenate([edge_windows(rng, H, W, d) for _ in range(reps)])
    vw = np.concatenate([edge_windows(rng, H, W, d) for _ in range(reps)])
    n = len(kw)

    def dev(x):   # [n, H, W, d] -> [1, H, n W, d]
        b = syn.f32_to_bf16_bits(np.ascontiguousarray(x.transpose(1, 0, 2, 3)).reshape(1, H, n * W, d))
        return torch.from_numpy(b.view(np.int16)).view(torch.bfloat16).cuda()

    cfg = qv.Config(batch=1, num_q_heads=H, num_kv_heads=H, window_tokens=W, quant_bits=bits,
                    max_context=n * W + 8, capacity_full=2, capacity_quant=n)
    c = qv.Cache(cfg)
    try:
        scores = torch.arange(n, 0, -1, dtype=torch.float32, device="cuda")[None] + 1
        c.prefill_assign(0, dev(kw), dev(vw), scores)   # windows 0, 1 Full, the others Quantized
        for w in range(2):
            ex = c.export_window(0, 0, w, quant=False, full=True)
            assert np.array_equal(from_bf16_bits(ex["full_k"]), kw[w])
            assert np.array_equal(from_bf16_bits(ex["full_v"]), vw[w])
        c.quantize_window(0, 0, 0)                      # from its bf16 slot
        c.quantize_window(0, 0, 1)
        for w in range(n):
            e = quantize_window(kw[w].astype(np.float64), vw[w].astype(np.float64), bits, G)
            ex = c.export_window(0, 0, w)
            for name, kc, ks in (("codes_k", "kc", ("ks", "kz")), ("codes_v", "vc", ("vs", "vz"))):
                m = from_fp16_bits(ex["meta_" + name[-1]])
                assert np.array_equal(m[:, 0], e[ks[0]]) and np.array_equal(m[:, 1], e[ks[1]]), (name, w)
                assert np.array_equal(ex[name], e[kc].astype(np.uint8)), (name, w)
            k, v = dequantize_window(e)
            c.promote_window(0, 0, w)
            ex = c.export_window(0, 0, w, quant=False, full=True)
            assert np.array_equal(from_bf16_bits(ex["full_k"]), rne_bf16(k)), w
            assert np.array_equal(from_bf16_bits(ex["full_v"]), rne_bf16(v)), w
            c.quantize_window(0, 0, w)
    finally:
        c.close()


def _edge_cache(W, bits, k, v, n_full):
    import torch
    import paper_2608_05326_amd as qv
    H, n = k.shape[1], k.shape[2] // W
    c = qv.Cache(qv.Config(batch=1, num_q_heads=H, num_kv_heads=H, window_tokens=W, quant_bits=bits,
                           max_context=n * W + 8, capacity_full=n_full, capacity_quant=n))
    scores = torch.arange(n, 0, -1, dtype=torch.float32, device="cuda")[None] + 1
    c.prefill_assign(0, k, v, scores)   # the first n_full windows Full, the others Quantized
    return c


@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), 65536.0, -65536.0, "nan group"])
@pytest.mark.parametrize("area", ["k", "v"])
@pytest.mark.parametrize("W", [8, 32, 64])
def test_groups_outside_fp16_are_reported(W, area, bad):
    """A group with an extreme outside fp16 or without a number latches the error, when a
    prompt is quantized and when a window of the Full tier is."""
    import torch
    import paper_2608_05326_amd as qv
    H, n = 2, 4
    k, v = (torch.randn(1, H, n * W, 128, device="cuda").bfloat16() for _ in range(2))
    x, w = (k if area == "k" else v), 1
    if bad == "nan group":
        if area == "k":
            x[0, 1, w * W:(w + 1) * W, 77] = float("nan")    # a channel over the window
        else:
            x[0, 1, w * W + 5, 64:] = float("nan")           # a token's groups of half the channels
    else:
        x[0, 1, w * W + 5, 77] = bad
    for n_full in (1, 2):
        c = _edge_cache(W, 4, k, v, n_full)
        try:
            if n_full == 2:
                c.get_state(0, 0)                            # held in bf16: no error yet
            with pytest.raises(qv.QEvictError) as ei:
                c.get_state(0, 0) if n_full == 1 else c.quantize_window(0, 0, w)
            assert ei.value.status == -5 and "fp16 range" in str(ei.value), str(ei.value)
        finally:
            c.close()


@pytest.mark.parametrize("bits", [4, 2])
@pytest.mark.parametrize("W", [8, 32, 64])
def test_nan_beside_numbers_codes_to_zero(W, bits):
    """A NaN in a group of numbers leaves the group's scale, zero point and other codes as they
    are without it and codes to 0, when a prompt is quantized and when a bf16 window is."""
    import torch
    H, n, G = 2, 6, 32 if W == 8 else W
    rng = np.random.default_rng(W + bits)
    from oracle.numerics import from_fp16_bits
    from oracle.qevict_oracle import quantize_window
    kw, vw = (syn.bf16_bits_to_f32(syn.f32_to_bf16_bits(rng.standard_normal((n, H, W, 128)).astype(np.float32)))
              for _ in range(2))
    nan_k, nan_v = (rng.random((n, H, W, 128)) < 0.04 for _ in range(2))
    nan_k[:, :, 0] = False                          # every group keeps a number
    nan_v[..., ::16] = False
    # for the oracle the NaN is its group's minimum: code 0, the same extremes
    fill_k = np.where(nan_k, np.where(nan_k, np.inf, kw).min(2, keepdims=True), kw)
    g = lambda a: a.reshape(n, H, W, 128 // G, G)   # noqa: E731
    fill_v = np.where(g(nan_v), np.where(g(nan_v), np.inf, g(vw)).min(4, keepdims=True), g(vw)).reshape(vw.shape)

    def dev(x, nan):
        x = np.where(nan, np.float32(np.nan), x).transpose(1, 0, 2, 3).reshape(1, H, n * W, 128)
        return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).cuda().bfloat16()

    c = _edge_cache(W, bits, dev(kw, nan_k), dev(vw, nan_v), 2)
    try:
        for w in range(2):
            c.quantize_window(0, 0, w)
        for w in range(n):
            e = quantize_window(fill_k[w].astype(np.float64), fill_v[w].astype(np.float64), bits, G)
            ex = c.export_window(0, 0, w)
            for a, name, kc, ks in (("k", "codes_k", "kc", ("ks", "kz")), ("v", "codes_v", "vc", ("vs", "vz"))):
                m = from_fp16_bits(ex["meta_" + a])
                assert np.array_equal(m[:, 0], e[ks[0]]) and np.array_equal(m[:, 1], e[ks[1]]), (a, w)
                nan = (nan_k if a == "k" else nan_v)[w]
                assert np.array_equal(ex[name][~nan], e[kc].astype(np.uint8)[~nan]), (a, w)
                assert not ex[name][nan].any(), (a, w)
    finally:
        c.close()
