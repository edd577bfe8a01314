"""GPU test of af_sparse_gemv_f16_noalloc (the entry point for callers that cannot allocate):
through the C ABI, on a context that owns no workspace, two calls in a row (the second on a
smaller input) must give the bits af_sparse_gemv_f16 gives, and stay within 2e-3 of the oracle.
Collected last on purpose (the file name sorts behind the other tests)."""
import numpy as np
import pytest
import torch

import synth_inputs as S
from oracle import activeflow_oracle as O
from paper_2504_08378_amd import binding as B
from gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu
TOL = 2e-3


def _case(out, n, seed):
    W = S.weight_matrix(seed, out, n, "noalloc", out, n)
    x = S.activation(seed, S.channel_scales(seed, n, "noalloc"), "noalloc", 0)
    return W, x


def test_noalloc_matches_workspace_entry_point_twice():
    ref_ctx = B.Context(0)
    ctx = B.Context(0, with_workspace=False)
    try:
        # the plain entry point refuses a context without workspace; the new one does not need it
        W0, x0 = _case(8, 8, 1)
        with pytest.raises(B.AfError) as e:
            ctx.sparse_gemv_f16(ref_ctx.pack_inmajor_f16(to_dev(W0)), to_dev(x0))
        assert e.value.status == -4
        # first call: several tiles, several splits, ragged tail; second call: smaller input
        for (out, n, k, kind, with_res) in [(4104, 2048, 1031, B.AF_F16, True),
                                            (520, 777, 300, B.AF_F32, False),
                                            (11008 * 2, 512, 256, B.AF_F16, False),
                                            (136, 100, 0, B.AF_F16, True)]:
            W, x = _case(out, n, out + n)
            idx = O.select_topk(x, k)
            res = S.activation(7, S.channel_scales(7, out, "res"), "res", 0) if with_res else None
            Wt = ref_ctx.pack_inmajor_f16(to_dev(W))
            ref_ctx.synchronize()
            xd, idxd = to_dev(x), to_dev(idx if k else np.zeros(1, np.int32))
            resd = None if res is None else to_dev(res)
            dt = torch.float16 if kind == B.AF_F16 else torch.float32
            y_ref = torch.zeros(out, dtype=dt, device="cuda")
            y_new = torch.full((out,), 7.0, dtype=dt, device="cuda")   # made before the call
            torch.cuda.synchronize()   # the contexts' streams do not wait for these fills
            ref_ctx.sparse_gemv_f16(Wt, xd, idxd, nidx=k, y=y_ref, y_kind=kind, residual=resd, out=out)
            ref_ctx.synchronize()
            # torch's allocator counts every device allocation it makes: the call must add none
            before = torch.cuda.memory_stats()["allocation.all.allocated"]
            ctx.sparse_gemv_f16_noalloc(Wt, xd, idxd, nidx=k, y=y_new, y_kind=kind, residual=resd, out=out)
            ctx.synchronize()
            assert torch.cuda.memory_stats()["allocation.all.allocated"] == before
            a, b = to_host(y_new), to_host(y_ref)
            assert np.array_equal(a.view(np.uint16 if kind == B.AF_F16 else np.uint32),
                                  b.view(np.uint16 if kind == B.AF_F16 else np.uint32)), (out, n, k)
            ref = O.sparse_gemv(W, x, idx)
            if res is not None:
                ref = ref + res.astype(np.float64)
            assert O.rel_err(a, ref) <= (TOL if kind == B.AF_F16 else 1e-4), (out, n, k)
    finally:
        ctx.close()
        ref_ctx.close()


def test_noalloc_limits_and_errors():
    ctx = B.Context(0, with_workspace=False)
    try:
        W, x = _case(8, 8, 3)
        Wt = to_dev(np.ascontiguousarray(W.T))
        L = B.lib()
        import ctypes as C
        y = torch.zeros(8, dtype=torch.float16, device="cuda")
        # out beyond the stated maximum: refused with its own status, nothing launched
        rc = L.af_sparse_gemv_f16_noalloc(ctx._h, C.c_void_p(Wt.data_ptr()), 8, B.AF_NOALLOC_MAX_OUT + 8,
                                          B.AF_NOALLOC_MAX_OUT + 8, C.c_void_p(to_dev(x).data_ptr()), None, 0,
                                          None, C.c_void_p(y.data_ptr()), B.AF_F16, None)
        assert rc == B.AF_ENOALLOC_LIMIT
        assert "limit" in B.strerror(rc)
        rc = L.af_sparse_gemv_f16_noalloc(ctx._h, None, 8, 8, 8, C.c_void_p(to_dev(x).data_ptr()), None, 0,
                                          None, C.c_void_p(y.data_ptr()), B.AF_F16, None)
        assert rc == -2
    finally:
        ctx.close()
