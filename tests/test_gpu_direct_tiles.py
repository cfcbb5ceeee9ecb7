"""GPU parity of the products whose waves load both operands in fragment order (up to 256 bfloat16 tokens, BL_W_GEMM weights):
every tile of the dispatch, token tiles of 1 to 16 rows, ragged outputs, K tiles fewer than waves and rounds that do not come out
even."""
import pytest
import torch

from paper_2411_04965_amd import binding as B
from tests.test_gpu_prefill_tiles import product

pytestmark = pytest.mark.gpu
BF16 = torch.bfloat16

# on 256 CUs these reach (INT8 / INT4 / gate-up; token tiles x output tiles): 1x1 1x1 1x2, 2x6 2x6 2x6, 2x8 2x4 3x6, 1x2 1x2 -,
# 1x4 1x3 1x6, - 1x4 1x4, 1x6 2x3 -, - 1x6 2x4, 2x4 - 2x2, 1x3 - -, 3x4 - -, and with the last four 2x3, 2x2 and 4x3, 2x2
CASES = [(9, 3210, 2056), (256, 5460, 776), (129, 5460, 2056), (9, 6141, 1288), (200, 8200, 200), (100, 2053, 1288),
         (47, 6141, 1288), (200, 5460, 1288), (256, 3210, 264), (256, 2053, 1288), (129, 8200, 776),
         (1, 17, 8), (2, 15, 264), (16, 1, 4104), (17, 33, 2048), (31, 1027, 5464), (33, 130, 11008), (255, 31, 3200)]
EXTRA = [(81, 4073, 776), (81, 2707, 8200), (177, 4078, 2056), (255, 1560, 520)]


@pytest.mark.parametrize("M,N,K", CASES + EXTRA)
def test_tiles(M, N, K):
    """Both linears and the gate/up front: bfloat16 and float32 outputs and accumulators, bit for bit (integer sums below 2^24
    are exact in the float32 reference; the rescale is the same two float32 products)."""
    print("[case] direct tiles M=%d N=%d K=%d" % (M, N, K), flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + N)
    X = torch.randn((M, K), generator=g, device="cuda").to(BF16)
    W = 0.02 * torch.randn((N, K), generator=g, device="cuda")
    Wu = 0.02 * torch.randn((N, K), generator=g, device="cuda")
    p, a = B.pack_ternary(W)
    pu, au = B.pack_ternary(Wu)
    topk = max(1, K // 2)
    acc8, y8 = product(X, W, B.BL_ACT_TOPK_INT8_ABSMAX, topk)
    assert torch.equal(B.bitlinear_a8_sparse(X, topk, p, a, N), y8.to(BF16))
    y, acc = B.bitlinear_a8_sparse(X, topk, p, a, N, y_dtype=torch.float32, want_acc=True)
    assert torch.equal(y, y8) and torch.equal(acc, acc8.int())
    acc4, y4 = product(X, W, B.BL_ACT_INT4_ABSMEAN)
    u4 = product(X, Wu, B.BL_ACT_INT4_ABSMEAN)[1]
    assert torch.equal(B.bitlinear_a4(X, p, a, N), y4.to(BF16))
    y, acc = B.bitlinear_a4(X, p, a, N, y_dtype=torch.float32, want_acc=True)
    assert torch.equal(y, y4) and torch.equal(acc, acc4.int())
    h = B.bitlinear_a4_gate_up(X, p, a, pu, au, N, want=("H",))["H"]
    assert torch.equal(h, (u4 * y4.clamp_min(0.0).square()).to(BF16))


def test_guard_bytes():
    """Nothing is written past the codes' space of the workspace or the outputs when the last token tile is ragged."""
    M, N, K = 35, 50, 520
    X = torch.randn((M, K), device="cuda").to(BF16)
    p, a = B.pack_ternary(0.02 * torch.randn((N, K), device="cuda"))
    for mode in (B.BL_ACT_INT4_ABSMEAN, B.BL_ACT_TOPK_INT8_ABSMAX):
        n = B.lib().bitlinear_workspace_bytes(mode, M, N, K)
        ws = torch.full((n + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
        y = torch.full((M * N + 64,), 7.0, dtype=BF16, device="cuda")
        if mode == B.BL_ACT_INT4_ABSMEAN:
            B.bitlinear_a4(X, p, a, N, ws=ws[:n], out=y[:M * N])
        else:
            B.bitlinear_a8_sparse(X, K // 2, p, a, N, ws=ws[:n], out=y[:M * N])
        assert (ws[n:] == 0x5A).all() and (y[M * N:] == 7.0).all()
