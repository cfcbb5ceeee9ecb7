"""Straight-through backward: every tile size of its contraction kernel, at sizes where tiles, rows and steps end raggedly,
against float64 products of the same operands."""
import pytest
import torch

from paper_2411_04965_amd import binding as B

pytestmark = pytest.mark.gpu


def _operands(M, N, K, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn((M, K), generator=g, device="cuda").bfloat16()
    w = 0.02 * torch.randn((N, K), generator=g, device="cuda")
    dy = (1e-3 * torch.randn((M, N), generator=g, device="cuda")).bfloat16()
    wb, alpha = B.pack_ternary(w, layout=B.BL_W_KMAJOR)
    T = B.unpack_ternary(wb, N, K, B.BL_W_KMAJOR).double()
    qa = B.quantize_act(x, B.BL_ACT_INT4_ABSMEAN)
    q = B.unpack_act(qa["q"], B.BL_ACT_INT4_ABSMEAN, M, K).double()
    dyd = (dy.float() * qa["scale"][:, None]).bfloat16().double()      # the rounding that the definition asks for
    return dy, wb, alpha, T, qa, q, dyd


# (on 256 CUs) dX: 64 x 64, 64 x 128, 128 x 128 and 256 x 256 tiles; dW of the last three shapes: 128 x 128, 64 x 64, 256 x 256
@pytest.mark.parametrize("M,N,K", [(65, 70, 130), (1030, 130, 1090), (2110, 1030, 2001), (3600, 70, 3900), (40, 3900, 3600)])
def test_every_tile(M, N, K):
    print("[case] ste tiles M=%d N=%d K=%d" % (M, N, K), flush=True)
    dy, wb, alpha, T, qa, q, dyd = _operands(M, N, K, M + N + K)
    dx, dw = B.bitlinear_backward(dy, qa["q"], qa["scale"], B.BL_ACT_INT4_ABSMEAN, K, wb, alpha, dx_dtype=torch.float32)
    u = 2.0 ** -24
    # float32 sums of exact products: n roundings of at most u times the sum of magnitudes each (dX: one more for alpha)
    ref, mag = dy.double() @ T * alpha.double(), dy.double().abs() @ T.abs() * alpha.double()
    assert bool(((dx.double() - ref).abs() <= (N + 1) * u * mag).all())
    ref, mag = dyd.t().contiguous() @ q, dyd.abs().t().contiguous() @ q.abs()
    assert bool(((dw.double() - ref).abs() <= M * u * mag).all())
    db, _ = B.bitlinear_backward(dy, qa["q"], qa["scale"], B.BL_ACT_INT4_ABSMEAN, K, wb, alpha, want_dw=False)
    assert torch.equal(db, dx.bfloat16())


def test_rows_beyond_32_bit_offsets():
    """A contraction of 2^22 + 70 tokens: offsets inside a tile no longer fit 32 bits.  Errors of float32 sums add up like
    a random walk here, about u sqrt(M) = 1.2e-4 of the result; four times that."""
    M, N, K = (1 << 22) + 70, 66, 70
    print("[case] ste wide M=%d N=%d K=%d" % (M, N, K), flush=True)
    dy, wb, alpha, T, qa, q, dyd = _operands(M, N, K, 5)
    _, dw = B.bitlinear_backward(dy, qa["q"], qa["scale"], B.BL_ACT_INT4_ABSMEAN, K, wb, alpha, want_dx=False)
    ref = torch.zeros((N, K), dtype=torch.float64, device="cuda")
    for i in range(0, M, 1 << 20):
        ref += dyd[i:i + (1 << 20)].t().contiguous() @ q[i:i + (1 << 20)]
    assert float((dw.double() - ref).norm() / ref.norm()) < 5e-4
