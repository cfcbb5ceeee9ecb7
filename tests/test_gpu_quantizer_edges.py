"""GPU parity of the quantizers' width- and type-specific kernels at the edges of their ranges."""
import numpy as np
import pytest
import torch

from oracle import bitnet_a48 as O
from paper_2411_04965_amd import binding as B
from paper_2411_04965_amd import synth as S
from tests.gpu_util import EPS, decode_int8, dev, host

pytestmark = pytest.mark.gpu


def _rows(M, K, seed):
    """Heavy-tailed rows, rows of a few distinct values, all zeros, mostly zeros, one value, and tiny values."""
    rng = np.random.default_rng(seed)
    x = S.gauss_outlier(M, K, max(1, K // 64), 20.0, seed)
    x[1::6] = np.round(x[1::6] * 8) * np.float32(0.0137)
    x[2::6] = 0.0
    x[3::6] *= rng.random((len(x[3::6]), K)) < 0.2
    x[4::6] = -0.75
    x[5::6] *= 1e-39
    return x.astype(np.float32)


@pytest.mark.parametrize("K", [4, 252, 256, 260, 512, 516, 1000, 1024, 1028])
def test_topk_float32_rows(K):
    """Float32 rows on both sides of the one-wave kernel's widest row, topk from 1 to K; bit for bit the oracle's codes,
    and the general kernel's (which a call that asks for the index list takes), infinities among the rows too."""
    M = 37
    x = _rows(M, K, S.seed_for(8, K))
    for topk in sorted({1, 2, K // 4 or 1, K // 2, K - 1, K}):
        print("[case] topk f32 K=%d topk=%d" % (K, topk), flush=True)
        q_ref, d_ref, _ = O.quant_topk_int8(x, topk, EPS)
        r = B.quantize_act(dev(x), B.BL_ACT_TOPK_INT8_ABSMAX, topk, EPS, want_rowsum=True)
        assert np.array_equal(host(r["scale"]), d_ref)
        assert np.array_equal(decode_int8(host(r["q"]), M, K), q_ref)
        assert np.array_equal(host(r["rowsum"]), q_ref.sum(1, dtype=np.int32))
        y = x.copy()
        y[::4, K // 2] = np.inf
        for eps in (EPS, 0.0):
            a = B.quantize_act(dev(y), B.BL_ACT_TOPK_INT8_ABSMAX, topk, eps, want_rowsum=True)
            b = B.quantize_act(dev(y), B.BL_ACT_TOPK_INT8_ABSMAX, topk, eps, want_rowsum=True, want_sel=True)
            for k in ("q", "rowsum"):
                assert torch.equal(a[k], b[k])
            assert torch.equal(a["scale"].view(torch.int32), b["scale"].view(torch.int32))
