"""GPU parity of the quantizers' width- and type-specific kernels at the edges of their ranges."""
import numpy as np
import pytest
import torch

from oracle import bitnet_a48 as O
from paper_2411_04965_amd import binding as B
from paper_2411_04965_amd import synth as S
from tests.test_gpu_parity import _rows_around_the_shortcut
from tests.gpu_util import EPS, decode_fp4, decode_fp4_mx, decode_int8, dev, host

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


@pytest.mark.parametrize("T,H,D", [(1, 3, 32), (5, 7, 96), (3, 5, 160)])
def test_kv_cache_widths(T, H, D):
    """The cache's two code widths in one launch: heads in rows of 16 lanes (D <= 128) and one per wave (wider), head
    counts that split a workgroup, the first token alone and with others, reads from position 0 and from 1."""
    print("[case] kv widths T=%d H=%d D=%d" % (T, H, D), flush=True)
    X = S.heavy(T, H * D, S.seed_for(8, T + H + D)).reshape(T, H, D)
    raw, d = O.kv_cache_pack(X, EPS)
    vals = O.kv_cache_unpack(raw, d, T, H, D)
    cache, scales = B.kv_cache_new(T, H, D, "cuda")
    B.kv_cache_append(dev(X.reshape(T, H * D)).reshape(T, H, D), 0, cache, scales, EPS)
    assert np.array_equal(cache.cpu().numpy(), raw)
    assert np.array_equal(host(scales), d)
    for pos0 in range(min(T, 2)):
        out = B.kv_cache_read(cache, scales, pos0, T - pos0, H, D, torch.float32)
        assert np.array_equal(host(out), vals[pos0:])


@pytest.mark.parametrize("be", [1, 2, 3, 4, 100, 127, 200, 253, 254])
def test_fp4_every_bfloat16(be):
    """Every bfloat16 value of the 17 binades up to a block's maximum, both signs, under every mantissa of that maximum:
    codes and scales bit for bit, at both ends of the exponent range and inside it."""
    print("[case] fp4 values be=%d" % be, flush=True)
    top = be * 128 + np.arange(128)                         # bit patterns of the maxima
    vals = np.arange(max(0, (be - 16) * 128), be * 128 + 128)
    blocks = []
    for t in top:
        v = vals[vals <= t]
        v = np.concatenate([v, v | 0x8000])
        v = np.concatenate([v, np.zeros(-len(v) % 31, v.dtype)]).reshape(-1, 31)
        blocks.append(np.concatenate([np.full((len(v), 1), t | (0x8000 if t & 1 else 0)), v], axis=1))
    bits = np.concatenate(blocks).astype(np.uint32)
    bits = bits[:len(bits) // 96 * 96].reshape(-1, 96 * 32)  # rows of 96 blocks
    x = (bits << 16).view(np.float32)
    M, K = x.shape
    c_ref, e_ref = O.quant_fp4(x)
    r = B.quantize_act(dev(x, torch.bfloat16), B.BL_ACT_FP4_E2M1_B32_MX)
    codes, e = decode_fp4_mx(host(r["q"]), host(r["scale"]), M, K)
    assert np.array_equal(e, e_ref + 127)
    assert np.array_equal(codes, c_ref)


@pytest.mark.parametrize("M,K", [(1, 8), (2, 24), (3, 136), (33, 504), (35, 520), (65, 1000), (31, 3200)])
def test_fp4_mx_edges(M, K):
    """Row pairs and wave edges, zero blocks; infinities and NaN give what the kernel for row-major codes gives."""
    print("[case] fp4 mx M=%d K=%d" % (M, K), flush=True)
    Kp = (K + 255) // 256 * 256
    x = S.snap_bf16(S.heavy(M, K, S.seed_for(8, M + K)))
    x[M // 2, :min(K, 64)] = 0.0
    pad = np.zeros((M, Kp), np.float32)
    pad[:, :K] = x
    c_ref, e_ref = O.quant_fp4(pad)
    r = B.quantize_act(dev(x, torch.bfloat16), B.BL_ACT_FP4_E2M1_B32_MX)
    codes, e = decode_fp4_mx(host(r["q"]), host(r["scale"]), M, Kp)
    assert np.array_equal(e, e_ref + 127) and np.array_equal(codes, c_ref)
    x[0, ::5] = np.inf
    x[M - 1, 1::7] = np.nan
    r = B.quantize_act(dev(x, torch.bfloat16), B.BL_ACT_FP4_E2M1_B32_MX)
    codes, e = decode_fp4_mx(host(r["q"]), host(r["scale"]), M, Kp)
    r = B.quantize_act(dev(x, torch.bfloat16), B.BL_ACT_FP4_E2M1_B32)
    assert np.array_equal(e, host(r["scale"]).reshape(M, Kp // 32))
    assert np.array_equal(codes, decode_fp4(host(r["q"]), M, Kp))


@pytest.mark.parametrize("K", [4, 260, 2048, 2052, 5460, 8192])
def test_topk_shortcut_eight_waves(K):
    """Eight waves per token, rows of up to 8192 channels: the shortcut for mostly-zero rows one count below, at and above its
    boundary, and rows with no value in reach of it, bit for bit the oracle's codes."""
    M, n_big = 33, max(1, K // 5)
    x = _rows_around_the_shortcut(M, K, n_big, S.seed_for(8, K)) if K >= 16 else S.snap_bf16(S.heavy(M, K, 1))
    x[5] = 0.0
    x[6] *= 2.0 ** -126                                     # maximum within 8 binades of the smallest number
    for topk in sorted({1, max(1, n_big - 1), n_big, min(K, n_big + 1), K // 2, K}):
        print("[case] topk shortcut K=%d topk=%d" % (K, topk), flush=True)
        q_ref, d_ref, _ = O.quant_topk_int8(x, topk, EPS)
        r = B.quantize_act(dev(x, torch.bfloat16), B.BL_ACT_TOPK_INT8_ABSMAX, topk, EPS)
        assert np.array_equal(host(r["scale"]), d_ref)
        assert np.array_equal(decode_int8(host(r["q"]), M, K), q_ref)
