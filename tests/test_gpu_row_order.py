"""GPU parity of the products on codes in row order, as callers that quantize themselves pass them: every kernel of that dispatch, also
at sizes for which the linears take fragment order; and the gate/up front at sizes beyond the fragment-order products, in one launch."""
import pytest
import torch

from paper_2411_04965_amd import binding as B
from tests.test_gpu_prefill_tiles import product

pytestmark = pytest.mark.gpu
BF16, F32 = torch.bfloat16, torch.float32

# up to 16 tokens: the streaming kernel, and where the codes do not fit its LDS whole tiles of 16 outputs and K split over blocks
SIZES = [(9, 12288, 4096), (16, 2050, 1000), (12, 4096, 4096), (5, 2064, 5460), (3, 1040, 2048), (16, 300, 8192), (1, 17, 8),
         (16, 2050, 11008), (16, 300, 11008), (9, 33, 20480),
         # 17 to 32: codes in LDS, one slice of K and several, one to four output tiles per block
         (17, 37, 256), (32, 70, 300), (24, 5460, 2048), (32, 4097, 4104), (31, 1030, 11008), (32, 12290, 4096), (20, 17000, 520),
         # 33 to 64: 64 x 64 and 64 x 128 tiles in one turn and in two, both sides of the rule on long K
         (33, 70, 200), (33, 1027, 1300), (57, 5460, 2048), (64, 16452, 520), (63, 32901, 257), (64, 260, 4200), (40, 70, 6401), (39, 70, 7168),
         (64, 2048, 6656), (64, 2049, 6500), (33, 2048, 7937), (47, 512, 7600), (64, 513, 7680), (64, 2560, 9216), (40, 2561, 9000),
         (64, 5120, 10241), (57, 5121, 9985), (35, 4916, 20480), (50, 6144, 13500), (33, 333, 32768), (64, 6144, 24577),
         # more: 64 x 64, 64 x 128 and 128 x 128 tiles, 128 x 128 with persistent blocks for short K and few outputs
         (65, 63, 200), (191, 1021, 257), (130, 516, 700), (256, 5000, 777), (200, 4100, 520), (250, 9001, 300), (3000, 389, 256)]


@pytest.mark.parametrize("M,N,K", SIZES)
def test_products(M, N, K):
    """Both code formats, bfloat16 rows alone, both output types with accumulators, bit for bit."""
    print("[case] row order M=%d N=%d K=%d" % (M, N, K), flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + N)
    X = torch.randn((M, K), generator=g, device="cuda").to(BF16)
    W = 0.02 * torch.randn((N, K), generator=g, device="cuda")
    p, a = B.pack_ternary(W)
    for mode, topk in ((B.BL_ACT_TOPK_INT8_ABSMAX, max(1, K // 2)), (B.BL_ACT_INT4_ABSMEAN, 0)):
        acc_ref, y_ref = product(X, W, mode, topk)
        qa = B.quantize_act(X, mode, topk=topk)
        assert torch.equal(B.bitlinear_gemm(qa["q"], qa["scale"], mode, M, K, p, a, N), y_ref.to(BF16))
        for dt in (BF16, F32):
            y, acc = B.bitlinear_gemm(qa["q"], qa["scale"], mode, M, K, p, a, N, y_dtype=dt, want_acc=True)
            assert torch.equal(y, y_ref.to(dt)) and torch.equal(acc, acc_ref.int())


# gate and up where the fragment-order products end, on 256 CUs: the streaming kernel on codes (up to 8 float32 tokens of long rows, 16
# tokens with many outputs), codes in LDS (17 to 32 tokens; short rows, and longer ones), 64-token tiles (33 to 64 tokens, likewise)
@pytest.mark.parametrize("M,N,K,dtype", [(8, 700, 8192, F32), (3, 1001, 5000, F32), (1, 37, 4100, F32), (16, 49200, 264, BF16),
                                         (32, 20001, 1000, BF16), (17, 30000, 256, F32), (24, 32902, 1288, BF16), (64, 8210, 1000, BF16),
                                         (40, 16000, 200, F32), (64, 12305, 1288, BF16), (48, 16392, 2056, BF16)])
def test_gate_up_one_launch(M, N, K, dtype):
    print("[case] gate/up, other kernels M=%d N=%d K=%d %s" % (M, N, K, dtype), flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + N)
    X = torch.randn((M, K), generator=g, device="cuda").to(dtype)
    W = 0.02 * torch.randn((N, K), generator=g, device="cuda")
    Wu = 0.02 * torch.randn((N, K), generator=g, device="cuda")
    g4, u4 = product(X, W, B.BL_ACT_INT4_ABSMEAN)[1], product(X, Wu, B.BL_ACT_INT4_ABSMEAN)[1]
    p, a = B.pack_ternary(W)
    pu, au = B.pack_ternary(Wu)
    h = B.bitlinear_a4_gate_up(X, p, a, pu, au, N, want=("H",))["H"]
    assert torch.equal(h, (u4 * g4.clamp_min(0.0).square()).to(BF16))
