"""GPU parity: af_select_gemv_f16 (producer + selection + gathered GEMV in one launch)
against the oracle's separate steps.  The selection input of each case is computed by the
oracle's own arithmetic on the same fp16 bits, so index sets are compared bit-for-bit where
the producer is the identity; behind a norm / SwiGLU producer the GPU's own x is used to
check the set from the definition and the oracle's set may differ only at the k-th magnitude."""
import numpy as np
import pytest
import torch

import synth_inputs as S
from oracle import activeflow_oracle as O
from paper_2504_08378_amd import binding as B
from gpu_util import ctx, to_dev, to_host  # noqa: F401

pytestmark = pytest.mark.gpu
TOL = 2e-3


def _wx(out, n, seed):
    W = S.weight_matrix(seed, out, n, "fused", out, n)
    x = S.activation(seed, S.channel_scales(seed, n, "fused"), "fused", 0)
    return W, x


def _run(ctx, Wt, src, n, **kw):
    xo = torch.zeros(n, dtype=torch.float16, device="cuda")
    io = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    co = torch.zeros(1, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()  # the context's stream does not wait for these fills
    y = ctx.select_gemv_f16(Wt, src, x_out=xo, idx_out=io, count_out=co, **kw)
    ctx.synchronize()
    c = int(to_host(co)[0])
    return to_host(y), to_host(xo), to_host(io)[:c], c


@pytest.mark.parametrize("out,n,k", [(136, 64, 32), (520, 1000, 377), (4096, 4096, 2048),
                                     (1032, 11008, 5504), (2056, 5120, 1536), (264, 28672, 14336)])
def test_identity_producer_topk_is_bit_exact(ctx, out, n, k):
    W, x = _wx(out, n, out + n)
    Wt = ctx.pack_inmajor_f16(to_dev(W))
    y, _, idx, c = _run(ctx, Wt, to_dev(x), n, sel_mode=B.AF_SEL_TOPK, k=k, y_kind=B.AF_F32)
    ref_idx = O.select_topk(x, k)
    assert c == k and np.array_equal(idx, ref_idx)
    assert O.rel_err(y, O.sparse_gemv(W, x, ref_idx)) <= 1e-4


def test_threshold_dense_and_empty(ctx):
    W, x = _wx(520, 2048, 5)
    Wt = ctx.pack_inmajor_f16(to_dev(W)); xd = to_dev(x)
    mags = np.sort(np.abs(x.astype(np.float64)))
    for t in (-1.0, 0.0, float(mags[1024]), 0.37, 3.0, 1e9, float("inf")):
        y, _, idx, c = _run(ctx, Wt, xd, 2048, sel_mode=B.AF_SEL_THRESHOLD, t=t, y_kind=B.AF_F32)
        ref_idx = O.select_threshold(x, t)
        assert c == len(ref_idx) and np.array_equal(idx, ref_idx), t
        assert O.rel_err(y, O.sparse_gemv(W, x, ref_idx)) <= 1e-4, t
    y = ctx.select_gemv_f16(Wt, xd, sel_mode=B.AF_SEL_DENSE, y_kind=B.AF_F32)
    ctx.synchronize()
    assert O.rel_err(to_host(y), O.sparse_gemv(W, x, np.arange(2048))) <= 1e-4
    res = S.activation(5, S.channel_scales(5, 520, "r"), "r", 0)
    y, _, idx, c = _run(ctx, Wt, xd, 2048, sel_mode=B.AF_SEL_TOPK, k=0, residual=to_dev(res))
    assert c == 0 and np.array_equal(y, res)
    # special values: NaN ranks highest for top-k and never passes a threshold
    z = x.copy(); z[7] = np.nan; z[9] = np.inf; z[11] = -np.inf
    _, _, idx, c = _run(ctx, Wt, to_dev(z), 2048, sel_mode=B.AF_SEL_TOPK, k=3)
    assert idx.tolist() == [7, 9, 11]
    _, _, idx, c = _run(ctx, Wt, to_dev(z), 2048, sel_mode=B.AF_SEL_THRESHOLD, t=1e4)
    assert idx.tolist() == O.select_threshold(z, 1e4).tolist() == [9, 11]


def _topk_property(x16, idx, k):
    key = (np.asarray(x16).view(np.uint16) & 0x7FFF).astype(np.int64)
    assert len(idx) == k and np.all(np.diff(idx) > 0)
    sel = np.zeros(len(key), bool); sel[idx] = True
    if k == 0 or k == len(key):
        return
    lo, hi = key[sel].min(), key[~sel].max()
    assert lo >= hi
    if lo == hi:
        assert np.nonzero(sel & (key == lo))[0].max() < np.nonzero(~sel & (key == lo))[0].min()


@pytest.mark.parametrize("n,out", [(256, 264), (4096, 12288), (5120, 1032)])
def test_rmsnorm_producer(ctx, n, out):
    W, h = _wx(out, n, n + 1)
    g = S.norm_gain(3, n, "fused")
    x_ref = O.round_f16(O.rmsnorm(h, g, 1e-5))
    k = n // 2
    Wt = ctx.pack_inmajor_f16(to_dev(W))
    y, x_gpu, idx, c = _run(ctx, Wt, to_dev(h), n, producer=B.AF_PRO_RMSNORM, gain=to_dev(g),
                            eps=1e-5, sel_mode=B.AF_SEL_TOPK, k=k, y_kind=B.AF_F32)
    assert O.rel_err(x_gpu, x_ref) <= TOL
    _topk_property(x_gpu, idx, k)
    ref_idx = O.select_topk(x_ref, k)
    if np.array_equal(x_gpu.view(np.uint16), x_ref.view(np.uint16)):
        assert np.array_equal(idx, ref_idx)
    # the GEMV itself, judged on the GPU's own x and set
    assert O.rel_err(y, O.sparse_gemv(W, x_gpu, idx)) <= 1e-4


def test_silumul_producer(ctx):
    n, out = 11008, 520
    W, _ = _wx(out, n, 77)
    sc = S.channel_scales(77, 2 * n, "gu")
    gu = (S.activation(77, sc, "gu", 0).astype(np.float32) * 0.3).astype(np.float16)
    x_ref = O.round_f16(O.silu(gu[:n]) * gu[n:].astype(np.float64))
    Wt = ctx.pack_inmajor_f16(to_dev(W))
    k = O.keep_count(n, 50)
    y, x_gpu, idx, c = _run(ctx, Wt, to_dev(gu), n, producer=B.AF_PRO_SILUMUL,
                            sel_mode=B.AF_SEL_TOPK, k=k, y_kind=B.AF_F32)
    assert O.rel_err(x_gpu, x_ref) <= TOL
    _topk_property(x_gpu, idx, k)
    assert O.rel_err(y, O.sparse_gemv(W, x_gpu, idx)) <= 1e-4


def test_argument_errors(ctx):
    W, x = _wx(64, 64, 1)
    Wt = ctx.pack_inmajor_f16(to_dev(W)); xd = to_dev(x)
    for kw, code in ((dict(producer=9), -1), (dict(sel_mode=5), -1), (dict(k=65), -1),
                     (dict(producer=B.AF_PRO_RMSNORM), -2), (dict(sel_mode=B.AF_SEL_THRESHOLD, t=float("nan")), -1)):
        with pytest.raises(B.AfError) as e:
            ctx.select_gemv_f16(Wt, xd, **kw)
        assert e.value.status == code, kw


# ---- threshold selection per channel range (no index list asked for) ---------------------
def _run_noidx(ctx, Wt, src, n, **kw):
    xo = torch.zeros(n, dtype=torch.float16, device="cuda")
    y = ctx.select_gemv_f16(Wt, src, x_out=xo, sel_mode=B.AF_SEL_THRESHOLD, y_kind=B.AF_F32, **kw)
    ctx.synchronize()
    return to_host(y), to_host(xo)


@pytest.mark.parametrize("out,n", [(136, 64), (520, 1000), (4096, 4096), (1032, 11008),
                                   (2056, 5120), (264, 28672), (22016, 4096), (8, 32768)])
def test_range_threshold_identity_producer(ctx, out, n):
    W, x = _wx(out, n, out + n)
    Wt = ctx.pack_inmajor_f16(to_dev(W)); xd = to_dev(x)
    mags = np.sort(np.abs(x.astype(np.float64)))
    for t in (-1.0, 0.0, float(mags[n // 2]), float(mags[(7 * n) // 10]), 1e9):
        y, xo = _run_noidx(ctx, Wt, xd, n, t=t)
        assert np.array_equal(xo.view(np.uint16), x.view(np.uint16))
        ref_idx = O.select_threshold(x, t)
        assert O.rel_err(y, O.sparse_gemv(W, x, ref_idx)) <= 1e-4, (t, len(ref_idx))


def test_range_threshold_special_values_and_residual(ctx):
    n, out = 2048, 520
    W, x = _wx(out, n, 5)
    z = x.copy(); z[7] = np.nan; z[9] = np.inf; z[11] = -np.inf; z[2040] = np.nan
    W2 = W.copy(); W2[:, [9, 11]] = 0     # keep the reference finite: Inf channels meet zero weights
    Wt = ctx.pack_inmajor_f16(to_dev(W2))
    # NaN never passes; Inf passes any finite threshold (and multiplies a zero weight -> NaN in
    # IEEE arithmetic, on both sides), so compare on a vector with the Infs removed as well
    z2 = z.copy(); z2[[9, 11]] = 0
    y, _ = _run_noidx(ctx, Wt, to_dev(z2), n, t=0.5)
    ref_idx = O.select_threshold(z2, 0.5)
    assert 7 not in ref_idx and 2040 not in ref_idx
    # the oracle multiplies the masked vector out densely (NaN * 0 = NaN), so its input is the
    # same vector with the unselected NaN channels cleared
    z3 = z2.copy(); z3[[7, 2040]] = 0
    assert O.rel_err(y, O.sparse_gemv(W2, z3, ref_idx)) <= 1e-4
    res = S.activation(5, S.channel_scales(5, out, "r"), "r", 0)
    y = ctx.select_gemv_f16(Wt, to_dev(x), sel_mode=B.AF_SEL_THRESHOLD, t=1e9, residual=to_dev(res))
    ctx.synchronize()
    assert np.array_equal(to_host(y), res)            # nothing passes: y is the residual


@pytest.mark.parametrize("producer", [B.AF_PRO_NONE, B.AF_PRO_RMSNORM, B.AF_PRO_SILUMUL])
@pytest.mark.parametrize("n,out,split,share", [
    (8, 8, 1, 0.5), (1016, 136, 1, 0.5), (1024, 136, 1, 1.0), (1032, 136, 1, 0.02),   # up to 64 channels a wave, one more
    (2048, 264, 1, 0.5), (2056, 520, 3, 0.9), (4096, 136, 1, 0.4), (4104, 136, 1, 0.4),  # 128, 256, and wider shares
    (3000, 8200, 7, 0.3), (3000, 14000, 5, 0.0),                                      # wider tiles, ragged splits, none kept
])
def test_range_threshold_shares(ctx, n, out, split, share, producer):
    """Every class of a wave's share against the oracle's product over the channels that pass, with x the
    GPU's own (the tap); a NaN never passes."""
    W, h = _wx(out, n, n + split)
    src, gain = h, None
    if producer == B.AF_PRO_SILUMUL:
        src = np.concatenate([h, h[::-1]])
    elif producer == B.AF_PRO_RMSNORM:
        gain = S.norm_gain(3, n, "shares")
    else:
        src = h.copy()
        src[n // 2] = np.nan
    t = 0.0
    Wt = ctx.pack_inmajor_f16(to_dev(W))
    ctx.set_option(B.AF_OPT_TUNE_SPLIT, split)
    try:
        args = dict(producer=producer, gain=None if gain is None else to_dev(gain), eps=1e-5)
        _, x = _run_noidx(ctx, Wt, to_dev(src), n, t=1e9, **args)
        mag = np.sort(np.abs(x[np.isfinite(x)].astype(np.float64)))[::-1]
        keep = int(share * len(mag))
        t = -1.0 if share == 1.0 else (float(mag[keep]) if keep < len(mag) else 0.0)
        if share == 0.0:
            t = float(mag[0])
        y, x2 = _run_noidx(ctx, Wt, to_dev(src), n, t=t, **args)
    finally:
        ctx.set_option(B.AF_OPT_TUNE_SPLIT, 0)
    assert np.array_equal(x.view(np.uint16), x2.view(np.uint16))
    idx = O.select_threshold(x, t)
    assert len(idx) == 0 if share == 0.0 else len(idx) > 0
    # the oracle multiplies the masked vector out densely (NaN * 0 = NaN)
    ref = O.sparse_gemv(W, np.nan_to_num(x, nan=0.0), idx)
    assert O.rel_err(y, ref) <= 1e-4 if len(idx) else not np.any(y)


@pytest.mark.parametrize("n,out", [(256, 264), (4096, 12288), (5120, 1032), (8192, 10240)])
def test_range_threshold_rmsnorm_producer(ctx, n, out):
    W, h = _wx(out, n, n + 1)
    g = S.norm_gain(3, n, "fused")
    x_ref = O.round_f16(O.rmsnorm(h, g, 1e-5))
    t = float(np.sort(np.abs(x_ref.astype(np.float64)))[n // 2])
    Wt = ctx.pack_inmajor_f16(to_dev(W))
    y, x_gpu = _run_noidx(ctx, Wt, to_dev(h), n, producer=B.AF_PRO_RMSNORM, gain=to_dev(g), eps=1e-5, t=t)
    assert O.rel_err(x_gpu, x_ref) <= TOL
    # same bits as the list-building form of the kernel
    _, x_list, idx, c = _run(ctx, Wt, to_dev(h), n, producer=B.AF_PRO_RMSNORM, gain=to_dev(g),
                             eps=1e-5, sel_mode=B.AF_SEL_THRESHOLD, t=t, y_kind=B.AF_F32)
    assert np.array_equal(x_gpu.view(np.uint16), x_list.view(np.uint16))
    # the GEMV, judged on the GPU's own x: the set follows from the definition
    own = O.select_threshold(x_gpu, t)
    assert np.array_equal(idx, own)
    assert O.rel_err(y, O.sparse_gemv(W, x_gpu, own)) <= 1e-4
    assert abs(len(own) / n - 0.5) < 0.02


def test_range_threshold_silumul_producer(ctx):
    n, out = 11008, 520
    W, _ = _wx(out, n, 77)
    sc = S.channel_scales(77, 2 * n, "gu")
    gu = (S.activation(77, sc, "gu", 0).astype(np.float32) * 0.3).astype(np.float16)
    x_ref = O.round_f16(O.silu(gu[:n]) * gu[n:].astype(np.float64))
    t = float(np.sort(np.abs(x_ref.astype(np.float64)))[n // 2])
    Wt = ctx.pack_inmajor_f16(to_dev(W))
    y, x_gpu = _run_noidx(ctx, Wt, to_dev(gu), n, producer=B.AF_PRO_SILUMUL, t=t)
    assert O.rel_err(x_gpu, x_ref) <= TOL
    own = O.select_threshold(x_gpu, t)
    assert O.rel_err(y, O.sparse_gemv(W, x_gpu, own)) <= 1e-4


@pytest.mark.parametrize("name,out,n,producer", [("gateup", 22016, 4096, "rmsnorm"), ("down", 4096, 11008, "silumul"),
                                                 ("o", 4096, 4096, "none")])
def test_7b_shapes_fused_forms_sampled(ctx, name, out, n, producer):
    """The benchmark's full-size operators in the launch shapes the bench times: the fused top-k
    form and the fused threshold form (no index list), sampled output columns against the oracle
    on the x the GPU produced (the selection is then checked from the definition)."""
    W = S.weight_matrix(0, out, n, "7b-fused", name, threads=8)
    kw = {}
    if producer == "rmsnorm":
        src = S.activation(0, S.channel_scales(0, n, "7b-fused", name), "7b-fused", name)
        g = S.norm_gain(0, n, "7b-fused", name)
        kw = dict(producer=B.AF_PRO_RMSNORM, gain=to_dev(g), eps=1e-5)
        x_ref = O.round_f16(O.rmsnorm(src, g, 1e-5))
    elif producer == "silumul":
        sc = S.channel_scales(0, 2 * n, "7b-fused", name)
        src = (S.activation(0, sc, "7b-fused", name).astype(np.float32) * 0.3).astype(np.float16)
        kw = dict(producer=B.AF_PRO_SILUMUL)
        x_ref = O.round_f16(O.silu(src[:n]) * src[n:].astype(np.float64))
    else:
        src = S.activation(0, S.channel_scales(0, n, "7b-fused", name), "7b-fused", name)
        x_ref = src
    Wt = ctx.pack_inmajor_f16(to_dev(W)); sd = to_dev(src)
    rows = np.random.default_rng(1).choice(out, size=64, replace=False)
    k = O.keep_count(n, 50)
    # top-k, fused
    y, x_gpu, idx, c = _run(ctx, Wt, sd, n, sel_mode=B.AF_SEL_TOPK, k=k, y_kind=B.AF_F32, **kw)
    assert O.rel_err(x_gpu, x_ref) <= TOL
    _topk_property(x_gpu, idx, k)
    ref = O.sparse_gemv(W[rows], x_gpu, idx)
    assert np.max(np.abs(y[rows] - ref)) <= 1e-4 * np.sqrt(np.mean(ref ** 2))
    # threshold, fused, no index list: the set follows from the definition on the GPU's x
    t = float(np.sort(np.abs(x_gpu.astype(np.float64)))[n // 2])
    y, x2 = _run_noidx(ctx, Wt, sd, n, t=t, **kw)
    assert np.array_equal(x2.view(np.uint16), x_gpu.view(np.uint16))
    own = O.select_threshold(x_gpu, t)
    ref = O.sparse_gemv(W[rows], x_gpu, own)
    assert np.max(np.abs(y[rows] - ref)) <= 1e-4 * np.sqrt(np.mean(ref ** 2))


def _random_cases(count, seed=2024):
    """Seeded mix of operator shapes that reaches every launch-shape branch (narrow / medium / wide
    tiles, one split and many), ragged sizes, every producer and both selection kinds."""
    rng = np.random.default_rng(seed)
    cases = []
    for i in range(count):
        out = 8 * int(rng.integers(1, [40, 800, 1600, 3600][i % 4]))
        n = 8 * int(rng.integers(1, min(2048, max(8, (3 << 20) // out))))   # the fused form takes in % 8 == 0
        pro = ("none", "rmsnorm", "silumul")[int(rng.integers(0, 3))]
        keep = float(rng.choice([0.05, 0.3, 0.5, 0.8, 1.0]))
        cases.append((out, n, pro, keep, int(rng.integers(0, 3))))
    return cases


@pytest.mark.parametrize("out,n,pro,keep,form", _random_cases(28))
def test_random_shapes_every_form(ctx, out, n, pro, keep, form):
    """form 0: top-k with list, 1: threshold with list, 2: threshold by channel range."""
    seed = out * 131 + n
    W = S.weight_matrix(seed, out, n, "rand", out, n)
    kw = {}
    if pro == "rmsnorm":
        src = S.activation(seed, S.channel_scales(seed, n, "rand"), "rand", 0)
        g = S.norm_gain(seed, n, "rand")
        kw = dict(producer=B.AF_PRO_RMSNORM, gain=to_dev(g), eps=1e-5)
        x_ref = O.round_f16(O.rmsnorm(src, g, 1e-5))
    elif pro == "silumul":
        src = (S.activation(seed, S.channel_scales(seed, 2 * n, "rand"), "rand", 1).astype(np.float32)
               * 0.3).astype(np.float16)
        kw = dict(producer=B.AF_PRO_SILUMUL)
        x_ref = O.round_f16(O.silu(src[:n]) * src[n:].astype(np.float64))
    else:
        src = S.activation(seed, S.channel_scales(seed, n, "rand"), "rand", 0)
        x_ref = src
    Wt = ctx.pack_inmajor_f16(to_dev(W)); sd = to_dev(src)
    k = min(n, max(1, int(round(keep * n))))
    if form == 0:
        y, x_gpu, idx, c = _run(ctx, Wt, sd, n, sel_mode=B.AF_SEL_TOPK, k=k, y_kind=B.AF_F32, **kw)
        _topk_property(x_gpu, idx, k)
    else:
        mags = np.sort(np.abs(x_ref.astype(np.float64)))
        t = float(mags[n - k]) if k < n else 0.0
        if form == 1:
            y, x_gpu, idx, c = _run(ctx, Wt, sd, n, sel_mode=B.AF_SEL_THRESHOLD, t=t, y_kind=B.AF_F32, **kw)
            assert np.array_equal(idx, O.select_threshold(x_gpu, t))
        else:
            y, x_gpu = _run_noidx(ctx, Wt, sd, n, t=t, **kw)
            idx = O.select_threshold(x_gpu, t)
    assert O.rel_err(x_gpu, x_ref) <= TOL
    if pro == "none":
        assert np.array_equal(x_gpu.view(np.uint16), x_ref.view(np.uint16))
    assert O.rel_err(y, O.sparse_gemv(W, x_gpu, idx)) <= 1e-4


# ---- rows requested before the selection has run (long top-k streams) ------------------------
def _pattern(kind, n, rng):
    x = rng.laplace(size=n)
    if kind == "equal":            # every channel ties with the k-th: the first k are kept
        x = np.where(rng.random(n) < 0.5, 1.5, -1.5)
    elif kind == "few":            # three magnitudes, ties across all ranges
        x = rng.choice([0.5, -1.0, 2.0], size=n)
    elif kind == "ascending":      # everything that is kept lies in the last ranges
        x = np.sort(np.abs(x))
    elif kind == "descending":
        x = -np.sort(-np.abs(x))
    elif kind == "sparse":         # fewer non-zero channels than k
        x = np.where(rng.random(n) < 0.2, x, 0.0)
    return x.astype(np.float16)


@pytest.fixture
def early_rows(ctx):
    """Every launch of the test requests rows early; one that could not would be refused."""
    ctx.set_option(B.AF_OPT_TUNE_EARLY_ROWS, 2)
    yield
    ctx.set_option(B.AF_OPT_TUNE_EARLY_ROWS, 0)


# width classes of the source (4096 / 16384 / above, and one past each), tile widths 128 / 256 / 512,
# ragged tiles, ranges that do not divide
@pytest.mark.parametrize("n,out,share", [(4096, 4096, 0.9), (4096, 12288, 0.5), (4096, 22016, 0.3), (4104, 8184, 0.5),
                                         (4040, 6152, 0.97), (11008, 4096, 0.5), (16384, 2056, 0.4),
                                         (16392, 4096, 0.5), (32768, 1032, 0.99), (8192, 10240, 1.0)])
@pytest.mark.parametrize("kind", ["random", "equal", "few", "ascending", "descending", "sparse"])
def test_early_rows_are_exactly_the_kept_ones(ctx, early_rows, n, out, share, kind):
    rng = np.random.default_rng(n + out)
    x, k = _pattern(kind, n, rng), int(n * share)
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    Wt = (torch.randn((n, out), generator=g, device="cuda") * 0.02).half()
    ref_idx = O.select_topk(x, k)
    # a channel that is not kept must not be touched by its weights either
    dropped = np.setdiff1d(np.arange(n), ref_idx)
    if len(dropped):
        Wt[torch.from_numpy(dropped).cuda()] = float("inf")
    y, xo, idx, c = _run(ctx, Wt, to_dev(x), n, sel_mode=B.AF_SEL_TOPK, k=k, y_kind=B.AF_F32)
    assert c == k and np.array_equal(idx, ref_idx)
    assert np.array_equal(xo.view(np.uint16), x.view(np.uint16))
    rows = torch.from_numpy(ref_idx.astype(np.int64)).cuda()
    xs = torch.from_numpy(x[ref_idx].astype(np.float64)).cuda()
    ref = (Wt[rows].double() * xs[:, None]).sum(0).cpu().numpy()
    assert O.rel_err(y, ref) <= 1e-4  # the bound of the fp32 results above
    y2, *_ = _run(ctx, Wt, to_dev(x), n, sel_mode=B.AF_SEL_TOPK, k=k, y_kind=B.AF_F32)
    assert np.array_equal(y, y2)      # the order of the sums is fixed


@pytest.mark.parametrize("n,out,share", [(4096, 12288, 0.5), (4096, 22016, 0.7), (8192, 10240, 0.5)])
def test_early_rows_lose_no_precision(ctx, n, out, share):
    """fp32 results against 64 bits, with and without early rows.  Different orders of the same sums:
    the mean over eight inputs of thousands of columns each settles to about 1 %; the early rows in
    the same running sum as the rest measured 4 to 15 % worse."""
    k = int(n * share)
    err = {1: [], 2: []}
    g = torch.Generator(device="cuda")
    for seed in range(8):
        g.manual_seed(seed)
        W = (torch.randn((n, out), generator=g, device="cuda") * 0.02).half()
        x = to_dev(S.activation(seed, S.channel_scales(seed, n, "fused"), "fused", 0))
        kept = torch.sort(x.float().abs(), descending=True, stable=True).indices[:k]
        ref = (W[kept].double() * x[kept].double()[:, None]).sum(0)
        torch.cuda.synchronize()
        for early in err:
            ctx.set_option(B.AF_OPT_TUNE_EARLY_ROWS, early)
            try:
                y = ctx.select_gemv_f16(W, x, sel_mode=B.AF_SEL_TOPK, k=k, y_kind=B.AF_F32)
            finally:
                ctx.set_option(B.AF_OPT_TUNE_EARLY_ROWS, 0)
            ctx.synchronize()
            err[early].append(float((y.double() - ref).norm() / ref.norm()))
    assert np.mean(err[2]) <= 1.02 * np.mean(err[1]), err


def _median_times(ctx, launches, reps=9):
    """Medians over `reps` of the time of each captured sequence of launches, taken in turn."""
    graphs = []
    with torch.cuda.stream(ctx.stream):
        for launch in launches:
            launch()  # nothing is prepared under capture
            ctx.synchronize()
            ctx.capture_begin()
            launch()
            graphs.append(ctx.capture_end())
    times = [[] for _ in graphs]
    for rep in range(reps):
        for t, g in zip(times, graphs):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            with torch.cuda.stream(ctx.stream):
                a.record()
                ctx.graph_launch(g)
                ctx.graph_launch(g)
                b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
    for g in graphs:
        ctx.graph_destroy(g)
    return [float(np.median(t[1:])) for t in times]


@pytest.mark.parametrize("n,out,pro", [(4096, 22016, "rmsnorm"), (28672, 8192, "none")])
def test_kept_channels_that_lie_together_cost_no_time(ctx, n, out, pro):
    """Half of the channels 6 times as large as the others, once spread out and once as one half of the
    vector: the same rows' worth of work for every split.  With the splits cut as contiguous channel
    ranges the second took 1.10 to 1.25 times the first; the medians of one case repeat within 0.03."""
    rng = np.random.default_rng(5)
    v, scale = rng.laplace(size=n) * 0.2, np.where(np.arange(n) < n // 2, 6, 1)
    kw = {"producer": B.AF_PRO_RMSNORM, "gain": to_dev(np.ones(n, np.float16))} if pro == "rmsnorm" else {}
    Ws = [(torch.randn((n, out), device="cuda") * 0.02).half() for _ in range(6)]
    y = torch.empty(out, dtype=torch.float16, device="cuda")
    srcs = [to_dev((v * sc).astype(np.float16)) for sc in (rng.permutation(scale), scale)]

    def launches(src):
        for W in Ws * 4:
            ctx.select_gemv_f16(W, src, sel_mode=B.AF_SEL_TOPK, k=n // 2, y=y, **kw)
    even, together = _median_times(ctx, [lambda src=src: launches(src) for src in srcs])
    assert together <= 1.06 * even, (even, together)


@pytest.mark.parametrize("n,out,share,pro", [(4096, 12288, 0.2, "rmsnorm"), (2048, 12288, 0.5, "none"),
                                             (16384, 6144, 0.1, "silumul"), (28672, 6144, 0.2, "silumul")])
def test_early_rows_are_left_out_where_they_cost_time(ctx, n, out, share, pro):
    """The built-in rule against early rows switched off.  By the bytes of a workgroup alone these four
    had them and took 1.05 to 1.12 times as long; without them both are the same launch."""
    k = int(n * share)
    kw = {}
    x = S.activation(1, S.channel_scales(1, n, "fused"), "fused", 0)
    if pro == "rmsnorm":
        kw = {"producer": B.AF_PRO_RMSNORM, "gain": to_dev(np.ones(n, np.float16))}
    elif pro == "silumul":
        kw, x = {"producer": B.AF_PRO_SILUMUL}, np.concatenate([np.full(n, 3, np.float16), x])
    src, y = to_dev(x), torch.empty(out, dtype=torch.float16, device="cuda")
    io, co = (torch.empty(m, dtype=torch.int32, device="cuda") for m in (n, 1))
    Ws = [(torch.randn((n, out), device="cuda") * 0.02).half() for _ in range(4)]
    torch.cuda.synchronize()

    def launches(early):
        ctx.set_option(B.AF_OPT_TUNE_EARLY_ROWS, early)
        try:
            for W in Ws * 6:
                ctx.select_gemv_f16(W, src, sel_mode=B.AF_SEL_TOPK, k=k, y=y, idx_out=io, count_out=co, **kw)
        finally:
            ctx.set_option(B.AF_OPT_TUNE_EARLY_ROWS, 0)
    off, rule = _median_times(ctx, [lambda e=e: launches(e) for e in (1, 0)])
    assert rule <= 1.03 * off, (off, rule)


# Every width class with every producer, forced onto the early rows: one channel group up to the widest
# input, splits that leave waves without channels, launches of fewer workgroups than list pieces,
# ragged tiles, padded rows, all three tile widths.
EARLY_SHAPES = [(8, 8, 0, 0), (136, 264, 3, 0), (1000, 520, 1, 8), (2048, 2048, 0, 0), (4088, 1032, 7, 0), (4096, 12288, 4, 0),
                (4104, 7176, 0, 24), (11008, 4096, 8, 0), (16384, 520, 16, 0), (16392, 1032, 0, 8), (32768, 520, 5, 0),
                (28672, 22016, 0, 0)]


@pytest.mark.parametrize("n,out,split,pad", EARLY_SHAPES)
@pytest.mark.parametrize("pro,kind", [(p, k) for p in ("none", "rmsnorm", "silumul") for k in ("random", "few", "half")]
                         + [("none", "special")])
def test_early_rows_forced(ctx, n, out, split, pad, pro, kind):
    rng = np.random.default_rng(n * 7 + out)
    if kind == "half":
        v = rng.laplace(size=n) * np.where(np.arange(n) < n // 2, 6, 1)
    elif kind == "special":
        v = rng.laplace(size=n)
        v[rng.random(n) < 0.3] *= 1e-7           # subnormal halves
        v[rng.integers(0, n, 5)] = np.nan
        v[rng.integers(0, n, 5)] = np.inf
        v[rng.integers(0, n, 5)] = -np.inf
    else:
        v = _pattern(kind, n, rng).astype(np.float64)
    v = v.astype(np.float16)
    kw, src = {}, v
    if pro == "rmsnorm":
        kw = {"producer": B.AF_PRO_RMSNORM, "gain": to_dev(np.ones(n, np.float16))}
    elif pro == "silumul":
        kw, src = {"producer": B.AF_PRO_SILUMUL}, np.concatenate([np.full(n, 3, np.float16), v])
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    Wt = (torch.randn((n, out + pad), generator=g, device="cuda") * 0.02).half()
    res = to_dev(S.activation(n, S.channel_scales(n, out, "r"), "r", 0))
    for share in (0.2, 0.7):
        k = max(1, int(n * share))
        got = {}
        for early in (1, 2):
            ctx.set_option(B.AF_OPT_TUNE_EARLY_ROWS, early)
            ctx.set_option(B.AF_OPT_TUNE_SPLIT, split)
            try:
                got[early] = _run(ctx, Wt, to_dev(src), n, sel_mode=B.AF_SEL_TOPK, k=k, out=out, residual=res, **kw)
            finally:
                ctx.set_option(B.AF_OPT_TUNE_EARLY_ROWS, 0)
                ctx.set_option(B.AF_OPT_TUNE_SPLIT, 0)
        (y1, x1, i1, c1), (y2, x2, i2, c2) = got[1], got[2]
        assert c1 == c2 == k and np.array_equal(x1.view(np.uint16), x2.view(np.uint16))
        assert np.array_equal(i2, O.select_topk(x2, k)) and np.array_equal(i1, i2)
        if kind != "special":
            rows = torch.from_numpy(i2.astype(np.int64)).cuda()
            xs = torch.from_numpy(x2[i2].astype(np.float64)).cuda()
            ref = (Wt[rows, :out].double() * xs[:, None]).sum(0) + res.double()
            assert O.rel_err(y2, ref.cpu().numpy()) <= TOL  # one rounding to fp16


def test_early_rows_refused_where_they_cannot_run(ctx):
    W, x = _wx(264, 2048, 3)
    Wt = ctx.pack_inmajor_f16(to_dev(W))
    ctx.set_option(B.AF_OPT_TUNE_EARLY_ROWS, 2)
    try:
        ctx.set_option(B.AF_OPT_TUNE_WAVES, 4)
        with pytest.raises(B.AfError):
            ctx.select_gemv_f16(Wt, to_dev(x), sel_mode=B.AF_SEL_TOPK, k=1024)
        ctx.set_option(B.AF_OPT_TUNE_WAVES, 0)
        ctx.select_gemv_f16(Wt, to_dev(x), sel_mode=B.AF_SEL_THRESHOLD, t=0.5)  # no early rows there
    finally:
        ctx.set_option(B.AF_OPT_TUNE_WAVES, 0)
        ctx.set_option(B.AF_OPT_TUNE_EARLY_ROWS, 0)
    ctx.synchronize()


@pytest.mark.parametrize("producer", [B.AF_PRO_RMSNORM, B.AF_PRO_SILUMUL])
@pytest.mark.parametrize("n,out,split", [(4096, 1032, 1), (4104, 136, 1), (8192, 264, 1), (8200, 6400, 3), (28672, 136, 5)])
def test_given_rows_ahead_of_x(ctx, n, out, split, producer):
    """Rows that are known (here all of them) are requested before x is built: one and several staging
    passes, all three counts of source vectors, both sides of the tile, a ragged split."""
    W, h = _wx(out, n, n + out)
    src = np.concatenate([h, h[::-1]]) if producer == B.AF_PRO_SILUMUL else h
    gain = to_dev(S.norm_gain(3, n, "given")) if producer == B.AF_PRO_RMSNORM else None
    xo = torch.zeros(n, dtype=torch.float16, device="cuda")
    Wt, srcd = ctx.pack_inmajor_f16(to_dev(W)), to_dev(src)
    ctx.set_option(B.AF_OPT_TUNE_SPLIT, split)
    try:
        y = ctx.select_gemv_f16(Wt, srcd, producer=producer, gain=gain, x_out=xo, sel_mode=B.AF_SEL_DENSE, y_kind=B.AF_F32)
        ctx.synchronize()
    finally:
        ctx.set_option(B.AF_OPT_TUNE_SPLIT, 0)
    assert O.rel_err(to_host(y), O.sparse_gemv(W, to_host(xo), np.arange(n))) <= 1e-4


@pytest.mark.parametrize("producer", [B.AF_PRO_RMSNORM, B.AF_PRO_SILUMUL])
@pytest.mark.parametrize("lx", [16, 32, 64])
@pytest.mark.parametrize("n,out,split", [(8, 8, 1), (136, 264, 1), (504, 136, 3), (520, 520, 1), (1032, 1032, 2), (5000, 264, 40)])
def test_few_given_rows_ahead_of_x(ctx, n, out, split, lx, producer):
    """The same where the rule would not: workgroups with fewer rows than are requested ahead, or a few more."""
    W, h = _wx(out, n, n + out)
    src = np.concatenate([h, h[::-1]]) if producer == B.AF_PRO_SILUMUL else h
    gain = to_dev(S.norm_gain(3, n, "given")) if producer == B.AF_PRO_RMSNORM else None
    xo = torch.zeros(n, dtype=torch.float16, device="cuda")
    Wt, srcd = ctx.pack_inmajor_f16(to_dev(W)), to_dev(src)
    ctx.set_option(B.AF_OPT_TUNE_SPLIT, split)
    ctx.set_option(B.AF_OPT_TUNE_LX, lx)
    ctx.set_option(B.AF_OPT_TUNE_EARLY_ROWS, 2)
    try:
        y = ctx.select_gemv_f16(Wt, srcd, producer=producer, gain=gain, x_out=xo, sel_mode=B.AF_SEL_DENSE, y_kind=B.AF_F32)
        ctx.synchronize()
    finally:
        for opt in (B.AF_OPT_TUNE_SPLIT, B.AF_OPT_TUNE_LX, B.AF_OPT_TUNE_EARLY_ROWS):
            ctx.set_option(opt, 0)
    assert O.rel_err(to_host(y), O.sparse_gemv(W, to_host(xo), np.arange(n))) <= 1e-4


@pytest.mark.parametrize("lx", [16, 64])
def test_given_rows_ahead_of_x_of_matrices_picked_on_the_device(ctx, lx):
    """Two output slots, each with the matrix that a device array names."""
    n, out, picked = 1032, 264, (2, 0)
    cases = [_wx(out, n, 50 + e) for e in range(3)]
    bank = torch.stack([ctx.pack_inmajor_f16(to_dev(W)) for W, _ in cases])
    x = cases[0][1]
    xo = torch.zeros(n, dtype=torch.float16, device="cuda")
    gain, srcd = to_dev(S.norm_gain(3, n, "given")), to_dev(x)
    sel = torch.tensor(picked, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    ctx.set_option(B.AF_OPT_TUNE_LX, lx)
    ctx.set_option(B.AF_OPT_TUNE_EARLY_ROWS, 2)
    try:
        y = ctx.select_gemv_experts_f16(bank, sel, 2, srcd, B.AF_PRO_RMSNORM, gain=gain, x_out=xo, sel_mode=B.AF_SEL_DENSE,
                                        y_kind=B.AF_F32)
        ctx.synchronize()
    finally:
        ctx.set_option(B.AF_OPT_TUNE_LX, 0)
        ctx.set_option(B.AF_OPT_TUNE_EARLY_ROWS, 0)
    ref = np.concatenate([O.sparse_gemv(cases[e][0], to_host(xo), np.arange(n)) for e in picked])
    assert O.rel_err(to_host(y).reshape(-1), ref) <= 1e-4
