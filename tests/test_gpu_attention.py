"""GPU parity of the attention launch on its own: the tap behind it against the oracle's attention on
the q, k, v the GPU itself produced (the tap in front of it), so nothing that entered earlier counts."""
import numpy as np
import pytest

import synth_inputs as S
from oracle import activeflow_oracle as O
from paper_2504_08378_amd import binding as B
from paper_2504_08378_amd import model as M
from gpu_util import ctx, layer_taps, to_dev, to_host  # noqa: F401

pytestmark = pytest.mark.gpu


def _run(ctx, heads, kv_heads, hd, K, V, kv_len, splits=0):
    shape = S.ModelShape("attention", 1, 64, heads, kv_heads, hd, 64)
    rng = np.random.default_rng(heads * 1000 + kv_heads * 10 + kv_len)
    w = S.layer_weights(3, shape, 0)
    for m in ("Wq", "Wk", "Wv"):
        w[m] = (rng.standard_normal(w[m].shape) * 0.3).astype(np.float16)
    h = rng.standard_normal(64).astype(np.float16)
    st = M.DeviceStack(ctx, shape, [M.DeviceLayer(ctx, shape, w)], [(K.copy(), V.copy())], K.shape[1])
    hin = to_dev(h)
    out = to_dev(np.zeros_like(h))
    ctx.set_option(B.AF_OPT_TUNE_ATTN_SPLITS, splits)
    try:
        st.layer(0, hin, out, kv_len, kv_len, M.select_cfg(B.AF_SEL_TOPK, (64, heads * hd, 64, 64)))
        ctx.synchronize()
    finally:
        ctx.set_option(B.AF_OPT_TUNE_ATTN_SPLITS, 0)
    taps = layer_taps(ctx, shape)
    qkv = taps["qkv"]
    q, k, v = (qkv[a * hd: b * hd].reshape(-1, hd)
               for a, b in ((0, heads), (heads, heads + kv_heads), (heads + kv_heads, heads + 2 * kv_heads)))
    Kr, Vr = K.copy(), V.copy()
    Kr[:, kv_len] = O.round_f16(O.rope(k, kv_len, 10000.0))
    Vr[:, kv_len] = v
    Kd, Vd = to_host(st.K[0]), to_host(st.V[0])
    assert np.array_equal(Vd[:, kv_len], v)
    # a rotated key is rounded once from fp32 products: at most the neighbouring value
    assert np.all(np.abs(Kd[:, kv_len].astype(np.float64) - Kr[:, kv_len]) <= 2.0 ** -10 * np.maximum(np.abs(Kr[:, kv_len]), 2.0 ** -4))
    Kr[:, kv_len] = Kd[:, kv_len]
    return taps["attn"], lambda: O.attention_decode(O.rope(q, kv_len, 10000.0), Kr, Vr, kv_len + 1).reshape(-1)


def _cache(kv_heads, cap, hd, kv_len, seed):
    rng = np.random.default_rng(seed)
    K, V = (rng.standard_normal((kv_heads, cap, hd)).astype(np.float16) for _ in range(2))
    K[:, kv_len:], V[:, kv_len:] = np.nan, np.nan  # nothing behind the cache may leak in
    return K, V


@pytest.mark.parametrize("heads,kv_heads,hd", [(2, 2, 128), (4, 2, 64), (8, 1, 128), (9, 1, 64), (16, 1, 128), (6, 2, 128)])
@pytest.mark.parametrize("kv_len,splits", [(0, 0), (0, 3), (1, 0), (31, 1), (32, 0), (33, 2), (64, 2), (127, 1), (128, 1),
                                           (129, 1), (300, 0), (300, 17), (1500, 1), (1500, 33)])
def test_heads_keys_and_splits(ctx, heads, kv_heads, hd, kv_len, splits):
    """Steps of 32 keys and rounds of 128 with a remainder, empty splits, the new token alone in a step,
    groups of query heads of every size (more than eight take two workgroups)."""
    K, V = _cache(kv_heads, kv_len + 5, hd, kv_len, kv_len + hd)
    got, ref = _run(ctx, heads, kv_heads, hd, K, V, kv_len, splits)
    # fp32 sums and one rounding to fp16
    assert O.rel_err(got, O.round_f16(ref())) <= 2e-3


@pytest.mark.parametrize("splits", [1, 4])
def test_infinities_stay_where_they_are(ctx, splits):
    """An infinite value reaches its own dimension only; a key with an infinite component takes all the
    weight or has none (its score is +inf or -inf), and its head alone sees it."""
    heads, hd, kv_len = 2, 128, 200
    K, V = _cache(heads, kv_len + 1, hd, kv_len, 5)
    plain, _ = _run(ctx, heads, heads, hd, K, V, kv_len, splits)
    Vi = V.copy()
    Vi[0, 77, 9] = np.inf
    got, _ = _run(ctx, heads, heads, hd, K, Vi, kv_len, splits)
    assert np.isposinf(got[9])
    keep = np.arange(heads * hd) != 9
    assert np.array_equal(got[keep], plain[keep])
    finite = 0
    for sign in (1.0, -1.0):
        Ki = K.copy()
        Ki[1, 50, 3] = sign * np.inf
        got, ref = _run(ctx, heads, heads, hd, Ki, V, kv_len, splits)
        assert np.array_equal(got[:hd], plain[:hd])
        if np.all(np.isfinite(got[hd:].astype(np.float32))):
            finite += 1
            assert O.rel_err(got, O.round_f16(ref())) <= 2e-3
        else:
            assert np.all(np.isnan(got[hd:].astype(np.float32)))
    assert finite == 1
