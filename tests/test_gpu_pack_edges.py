"""GPU parity of pack_ternary where its kernels and their dispatch have edges: rows of any length, both sides of the rule between
the two K-major kernels, weights on either side of the rounding boundary, scales outside the range of the comparison."""
import numpy as np
import pytest
import torch

from oracle import bitnet_a48 as O
from paper_2411_04965_amd import binding as B
from paper_2411_04965_amd import synth as S
from tests.gpu_util import EPS, decode_w_gemm, decode_w_kmajor, decode_w_mx2, decode_w_mx4, decode_w_rows, dev, host

pytestmark = pytest.mark.gpu

F32, BF16 = torch.float32, torch.bfloat16
DECODE = {B.BL_W_GEMM: decode_w_gemm, B.BL_W_KMAJOR: decode_w_kmajor, B.BL_W_MX4: decode_w_mx4, B.BL_W_ROWS: decode_w_rows,
          B.BL_W_MX2: decode_w_mx2}


def check(W, layout, dtype=F32, eps=EPS, ref=None):
    T, alpha = ref or O.ternarize(W, eps)
    packed, a = B.pack_ternary(dev(W, dtype), eps, layout)
    assert host(a)[0] == alpha
    assert np.array_equal(DECODE[layout](host(packed), *W.shape), T)
    assert np.array_equal(host(B.unpack_ternary(packed, *W.shape, layout)), T)


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("layout", sorted(DECODE))
@pytest.mark.parametrize("N,K", [(1, 1), (17, 101), (33, 514), (530, 1003)])
def test_rows_of_any_length(N, K, layout, dtype):
    print("[case] pack N=%d K=%d layout=%d %s" % (N, K, layout, dtype), flush=True)
    W = S.latent_weights(N, K, S.seed_for(7, N + K))
    check(S.snap_bf16(W) if dtype == BF16 else W, layout, dtype)


# K-major blocks of 64 channels x 512 outputs: 99 / 100 (rows of whole groups of four), 256 / 257 (other rows; 256 CUs)
@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("N,K", [(4608, 704), (5120, 640), (8192, 1021), (512, 16447)])
def test_kmajor_rule(N, K, dtype):
    print("[case] pack K-major N=%d K=%d %s" % (N, K, dtype), flush=True)
    W = S.latent_weights(N, K, S.seed_for(7, N + K))
    check(S.snap_bf16(W) if dtype == BF16 else W, B.BL_W_KMAJOR, dtype)


def boundary(N, K, t):
    """Weights whose mean is t: mostly +-t, and every 32nd one just below t/2, t/2 or just above it, next to a +-3t/2."""
    half = np.float32(t / 2)
    special = [np.nextafter(half, np.float32(0)), half, np.nextafter(half, np.float32(np.inf))]
    W = np.full(N * K, t, dtype=np.float32)
    W[1::2] *= -1
    for i, b in enumerate(range(0, N * K - 32, 32)):
        sign = 1 if i & 1 else -1
        W[b + i % 23] = sign * special[i % 3]
        W[b + i % 23 + 1] = sign * np.float32(1.5) * t
    return W.reshape(N, K), special


# the comparison holds from 2^-100 to 2^100; outside, the quotient of eq. 2 is formed
@pytest.mark.parametrize("layout", sorted(DECODE))
@pytest.mark.parametrize("e", [-127, -110, -101, -100, -99, -6, 0, 99, 100, 101, 126])
def test_rounding_boundary(e, layout):
    """The float32 neighbours of half the scale: t/2 and less are 0 (half to even), the next number above is 1, at any scale."""
    print("[case] pack boundary 2^%d layout=%d" % (e, layout), flush=True)
    for m in (1.0, 1.0 + 2.0 ** -23, 1.5, 2.0 - 2.0 ** -23):
        t = np.float32(np.ldexp(m, e))
        for K in (203, 204):
            W, special = boundary(35, K, t)
            T, alpha = O.ternarize(W, 0.0)
            assert alpha == t
            for s, c in zip(special, (0, 0, 1)):
                assert (np.abs(T[np.abs(W) == s]) == c).all()
            check(W, layout, eps=0.0, ref=(T, alpha))
