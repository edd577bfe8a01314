"""GPU parity of the attention launch on its own: the tap behind it against the oracle's attention on
the q, k, v the GPU itself produced (the tap in front of it), so nothing that entered earlier counts."""
import ctypes

import numpy as np
import pytest

import synth_inputs as S
from oracle import activeflow_oracle as O
from paper_2504_08378_amd import binding as B
from paper_2504_08378_amd import model as M
from gpu_util import ctx, layer_taps, to_dev, to_host  # noqa: F401

pytestmark = pytest.mark.gpu


def _run(ctx, heads, kv_heads, hd, K, V, kv_len, splits=0):
    attn, q, Kr, Vr = _run_parts(ctx, heads, kv_heads, hd, K, V, kv_len, splits)
    return attn, lambda: O.attention_decode(O.rope(q, kv_len, 10000.0), Kr, Vr, kv_len + 1).reshape(-1)


def _run_parts(ctx, heads, kv_heads, hd, K, V, kv_len, splits=0, q_scale=0.3, seed=0, edit=None):
    shape = S.ModelShape("attention", 1, 64, heads, kv_heads, hd, 64)
    rng = np.random.default_rng(heads * 1000 + kv_heads * 10 + kv_len + 7 * seed)
    w = S.layer_weights(3, shape, 0)
    for m in ("Wq", "Wk", "Wv"):
        w[m] = (rng.standard_normal(w[m].shape) * q_scale).astype(np.float16)
    h = rng.standard_normal(64).astype(np.float16)
    if edit is not None:
        edit(w, h)
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
    return taps["attn"], q, Kr, Vr


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


@pytest.mark.parametrize("heads,kv_heads,hd,kv_len", [(72, 8, 128, 3100), (16, 16, 64, 3100), (16, 16, 64, 3000)])
def test_long_caches_share_rows_among_eight_heads(ctx, heads, kv_heads, hd, kv_len):
    """Caches on both sides of the line from which a workgroup takes eight query heads and not four."""
    K, V = _cache(kv_heads, kv_len + 5, hd, kv_len, kv_len + hd)
    got, ref = _run(ctx, heads, kv_heads, hd, K, V, kv_len)
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


def _partials(ctx, heads, hd, splits):
    """The key splits' fp32 results of the last launch: [head][split][maximum, sum, values].  They lie right in
    front of the first inter-operator tensor."""
    taps = []
    for i in range(7):
        p = ctypes.c_void_p()
        assert B.lib().af_layer_tap(ctx._h, i, ctypes.byref(p)) == 0
        taps.append(p.value - ctx.workspace.data_ptr())
    off = min(taps) - 4 * (1 << 18) * ctx.max_batch
    part = to_host(ctx.workspace[off: off + 4 * heads * splits * (hd + 2)]).view(np.float32)
    return part.astype(np.float64).reshape(heads, splits, hd + 2)


def _pairwise(x, axis):
    x = np.moveaxis(x, axis, 0)
    while len(x) > 1:
        x = np.concatenate([x, np.zeros_like(x[:1])]) if len(x) % 2 else x
        x = x[0::2] + x[1::2]
    return x[0]


@pytest.mark.parametrize("heads,kv_heads,hd", [(16, 16, 128), (32, 4, 128), (16, 4, 64)])
@pytest.mark.parametrize("kv_len,splits", [(16, 2), (64, 2), (500, 4), (2000, 2)])
def test_results_before_rounding_carry_fp32(ctx, heads, kv_heads, hd, kv_len, splits):
    """q, the weights and the sums are held in 32 bits: the results before their rounding to fp16 are as close to
    64 bits as fp32 arithmetic with one rounding per operation and sums in pairs, the most accurate order (0.66 to
    0.87 of its error measured; the bound leaves room for other inputs).  Operands of 22 bits and weights whose
    exponent carries a factor gave 2.0 to 2.6 times its error."""
    err, plain = [], []
    for seed in range(4):
        K, V = _cache(kv_heads, kv_len + 1, hd, kv_len, kv_len + hd + 100 * seed)
        _, q, Kr, Vr = _run_parts(ctx, heads, kv_heads, hd, K, V, kv_len, splits, 0.05, seed)
        part = _partials(ctx, heads, hd, splits)
        w = np.exp2(part[:, :, 0] - part[:, :, 0].max(1, keepdims=True))
        got = (w[..., None] * part[:, :, 2:]).sum(1) / (w * part[:, :, 1]).sum(1)[:, None]
        Kr, Vr = (np.repeat(a[:, : kv_len + 1], heads // kv_heads, 0) for a in (Kr, Vr))

        def attend(t):
            ang = kv_len * 10000.0 ** (-2.0 * np.arange(hd // 2) / hd)
            cs, sn = (f(ang).astype(np.float32).astype(t) for f in (np.cos, np.sin))
            a, b = q[:, : hd // 2].astype(t), q[:, hd // 2:].astype(t)
            x = np.concatenate([a * cs - b * sn, b * cs + a * sn], 1) * (t(1) / np.sqrt(t(hd)))
            s = _pairwise(Kr.astype(t) * x[:, None], 2)
            e = np.exp(s - s.max(1, keepdims=True))
            return _pairwise(e[..., None] * Vr.astype(t), 1) / _pairwise(e, 1)[:, None]

        exact = attend(np.float64)
        err.append(np.linalg.norm(got - exact) / np.linalg.norm(exact))
        plain.append(np.linalg.norm(attend(np.float32) - exact) / np.linalg.norm(exact))
    assert np.mean(err) <= 1.3 * np.mean(plain), (np.mean(err), np.mean(plain))


@pytest.mark.parametrize("splits", [1, 4])
@pytest.mark.parametrize("score,result", [(-25.0, np.inf), (-40.0, np.inf), (-70.0, np.inf), (-200.0, np.nan)])
def test_infinite_value_of_a_small_weight(ctx, splits, score, result):
    """However small the weight, an infinite value times it is infinite; times a weight of zero (e^-200 in fp32)
    it is NaN.  The other dimensions do not see it."""
    heads, hd, kv_len = 2, 128, 200
    K, V = _cache(heads, kv_len + 1, hd, kv_len, 6)
    K[:, :kv_len] = 0
    plain, q, _, _ = _run_parts(ctx, heads, heads, hd, K, V, kv_len, splits)
    x = O.rope(q, kv_len, 10000.0)[0]
    K[0, 77] = x * (score * np.sqrt(hd) / np.dot(x, x))
    plain, _, _, _ = _run_parts(ctx, heads, heads, hd, K, V, kv_len, splits)
    V[0, 77, 9] = np.inf
    got, _, _, _ = _run_parts(ctx, heads, heads, hd, K, V, kv_len, splits)
    assert np.array_equal(got[9: 10], np.array([result], np.float16), equal_nan=True)
    keep = np.arange(heads * hd) != 9
    assert np.array_equal(got[keep], plain[keep])


@pytest.mark.parametrize("splits", [1, 4])
def test_infinite_key_behind_a_small_query(ctx, splits):
    """A query component far below the smallest fp16, times an infinite key: the score is infinite and not NaN,
    so the key with -inf has no weight and nothing else changes."""
    heads, hd, kv_len = 2, 128, 200

    def small(w, h):  # component 3 of head 1 is two or three of the smallest fp16, its partner zero
        w["Wq"][hd + 3] = 0
        w["Wq"][hd + 3 + hd // 2] = 0
        w["Wq"][hd + 3, np.argmax(np.abs(h))] = 2.0 ** -24

    K, V = _cache(heads, kv_len + 1, hd, kv_len, 7)
    _, q, _, _ = _run_parts(ctx, heads, heads, hd, K, V, kv_len, splits, edit=small)
    x = O.rope(q, kv_len, 10000.0)[1, 3]
    assert 0 < abs(x) / np.sqrt(hd) * np.log2(np.e) < 2.0 ** -25
    K[1, 50, 3] = -np.sign(x) * np.inf
    got, q, Kr, Vr = _run_parts(ctx, heads, heads, hd, K, V, kv_len, splits, edit=small)
    ref = O.attention_decode(O.rope(q, kv_len, 10000.0), Kr, Vr, kv_len + 1).reshape(-1)
    assert np.all(np.isfinite(got.astype(np.float32)))
    assert O.rel_err(got, O.round_f16(ref)) <= 2e-3


@pytest.mark.parametrize("heads,kv_heads,hd", [(4, 2, 128), (6, 1, 128), (3, 3, 64), (16, 2, 64)])
@pytest.mark.parametrize("kv_len", [0, 1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 80, 97, 126, 127, 128])
def test_short_caches(ctx, heads, kv_heads, hd, kv_len):
    """Fewer than 128 cached keys go to a kernel of their own (up to 63 in one form, from 64 in another): against the oracle, and against
    the other kernel (one split asked for), both within half a unit in the last place plus fp32's error of
    the same result, so at most the neighbouring fp16 value apart."""
    K, V = _cache(kv_heads, kv_len + 3, hd, kv_len, kv_len + hd)
    got, ref = _run(ctx, heads, kv_heads, hd, K, V, kv_len)
    assert O.rel_err(got, O.round_f16(ref())) <= 2e-3
    other, _ = _run(ctx, heads, kv_heads, hd, K, V, kv_len, 1)
    a, b = got.astype(np.float64), other.astype(np.float64)
    assert np.all(np.abs(a - b) <= 2.0 ** -10 * np.maximum(np.abs(b), 2.0 ** -14) + 1e-6)


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("kv_len", [17, 63, 64, 127])
def test_short_caches_special_values(ctx, hd, kv_len):
    """An infinite value reaches its own dimension only; a key of -inf has no weight; a NaN key makes its head NaN;
    rows behind the cache are read and not used."""
    heads, rep = 4, 2
    K, V = _cache(heads // rep, kv_len + 2, hd, kv_len, 11)
    K[:, kv_len:] = np.nan
    V[:, kv_len:] = np.nan
    plain, q, Kr, Vr = _run_parts(ctx, heads, heads // rep, hd, K, V, kv_len)
    assert np.all(np.isfinite(plain.astype(np.float32)))
    V1 = V.copy(); V1[0, 5, 3] = np.inf
    got = _run_parts(ctx, heads, heads // rep, hd, K, V1, kv_len)[0].reshape(heads, hd)
    keep = np.ones((heads, hd), bool); keep[:rep, 3] = False
    assert np.all(got[:rep, 3] == np.inf) and np.array_equal(got[keep], plain.reshape(heads, hd)[keep])
    K1 = K.copy(); K1[1, 7, 2] = np.nan
    got = _run_parts(ctx, heads, heads // rep, hd, K1, V, kv_len)[0].reshape(heads, hd)
    assert np.all(np.isnan(got[rep:].astype(np.float32))) and np.array_equal(got[:rep], plain.reshape(heads, hd)[:rep])
    x = O.rope(q, kv_len, 10000.0)[0]
    K2 = K.copy(); K2[0, 9, 4] = -np.sign(x[4]) * np.inf
    got, q, Kr, Vr = _run_parts(ctx, heads, heads // rep, hd, K2, V, kv_len)
    one = O.attention_decode(O.rope(q, kv_len, 10000.0), Kr, Vr, kv_len + 1)[0]
    assert np.all(np.isfinite(got[:hd].astype(np.float32))) and O.rel_err(got[:hd], O.round_f16(one)) <= 2e-3
