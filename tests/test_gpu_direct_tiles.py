"""GPU parity of the products whose waves load both operands in fragment order (up to 256 tokens, BL_W_GEMM weights): every tile of
the dispatch and both sides of its lines, token tiles of 1 to 16 rows, ragged outputs, K tiles fewer than waves and rounds that do not
come out even; bfloat16 and float32 tokens."""
import pytest
import torch

from paper_2411_04965_amd import binding as B
from tests.test_gpu_prefill_tiles import product

pytestmark = pytest.mark.gpu
BF16 = torch.bfloat16

# on 256 CUs these reach (token tiles x output tiles of INT8, of INT4, of gate and up; - = another kernel)
CASES = [(33, 5269, 200),                         # 1x2 1x2 -
         (45, 4282, 520),                         # 1x2 1x2 1x4
         (200, 6789, 1288),                       # 2x4 2x4 2x4
         (31, 1776, 200),                         # 1x1 1x1 1x2
         (31, 5376, 776),                         # 1x3 1x3 1x6
         (31, 10981, 1288),                       # 1x6 2x3 2x6
         (129, 3436, 1288),                       # 1x4 1x4 3x6
         (177, 3989, 2056),                       # 2x6 2x6 2x4
         (180, 2699, 776),                        # 2x2 2x2 2x4
         (72, 9575, 776),                         # 1x6 1x6 1x6
         (65, 10064, 1288),                       # 2x8 2x4 2x4
         (17, 6414, 264),                         # 1x2 1x2 2x2
         (177, 4062, 776), (81, 8168, 776),       # 2x3 2x3 2x4, 3x4 1x4 2x4
         (1, 17, 8), (2, 15, 264), (16, 1, 4104), (9, 3210, 2056), (31, 1027, 5464), (33, 130, 11008), (255, 31, 3200), (256, 3210, 264),
         # weights that the quantizer's launch touches: lines that do not divide by eight XCDs, one matrix and two; and beyond the rule
         (9, 2049, 2312), (64, 4099, 2056), (40, 24600, 264), (57, 17000, 520), (250, 6300, 300),
         # either side of the lines: outputs of a turn of the other kernels (33 to 64 and 17 to 32 tokens), token tiles in pairs with short
         # and with longer rows, one K tile, nine to sixteen K tiles at up to 32 tokens, beyond a turn of 64 x 128 tiles
         (33, 32760, 264), (33, 32776, 264), (17, 65528, 264), (17, 65544, 264), (48, 16376, 1000), (48, 16392, 1000), (97, 12288, 1288),
         (97, 12296, 1288), (90, 5464, 256), (90, 5460, 200), (28, 45056, 2312), (28, 45060, 2312), (88, 16384, 3400), (88, 16392, 3400)]


# float32 tokens and rows of any length: the general INT4 quantizer, the one-wave Top_k quantizer of up to 512 and 1024 channels
OTHER = [(16, 512, 256, torch.float32), (64, 1000, 1000, torch.float32), (33, 130, 1021, torch.float32), (1, 16, 4, torch.float32),
         (47, 700, 512, torch.float32), (17, 70, 516, torch.float32), (200, 300, 4097, torch.float32), (17, 70, 300, BF16),
         (9, 100, 262, BF16), (40, 333, 4099, BF16)]


@pytest.mark.parametrize("M,N,K,dtype", [c + (BF16,) for c in CASES] + OTHER)
def test_tiles(M, N, K, dtype):
    """Both linears and the gate/up front: bfloat16 and float32 outputs and accumulators, bit for bit (integer sums below 2^24
    are exact in the float32 reference; the rescale is the same two float32 products)."""
    print("[case] direct tiles M=%d N=%d K=%d %s" % (M, N, K, dtype), flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + N)
    X = torch.randn((M, K), generator=g, device="cuda").to(dtype)
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


def _special_rows(M, K, seed):
    """Rows in turn: zeros, one value, few values with ties everywhere, mostly zeros, an infinity, both infinities, NaN, subnormals, largest
    finite values, ordinary ones."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn((M, K), generator=g, device="cuda")
    x[0::10] = 0.0
    x[1::10] = -0.75
    x[2::10] = torch.round(x[2::10] * 2.0) * 0.5
    x[3::10] *= torch.rand(x[3::10].shape, generator=g, device="cuda") < 0.1
    x[4::10, K // 2] = float("inf")
    x[5::10, 0] = float("inf")
    x[5::10, K - 1] = float("-inf")
    x[6::10, K // 3] = float("nan")
    x[7::10] *= 1e-39
    x[8::10] = x[8::10].sign() * 3.0e38
    return x


@pytest.mark.parametrize("M", [9, 16, 35, 64, 200, 256])
@pytest.mark.parametrize("K,dtype", [(520, BF16), (4104, BF16), (5460, BF16), (9000, BF16), (1021, BF16), (516, torch.float32),
                                     (1024, torch.float32), (2050, torch.float32)])
def test_special_rows(M, K, dtype):
    """Codes stored in fragment order against the same quantizers' codes in row order: accumulators, outputs and scales."""
    print("[case] special rows M=%d K=%d %s" % (M, K, dtype), flush=True)
    N = 130
    X = _special_rows(M, K, M + K).to(dtype)
    p, a = B.pack_ternary(torch.randn((N, K), generator=torch.Generator(device="cuda").manual_seed(K), device="cuda"))
    for mode, topks in ((B.BL_ACT_INT4_ABSMEAN, (0,)), (B.BL_ACT_TOPK_INT8_ABSMAX, (1, K // 2, K))):
        for topk in topks:
            qa = B.quantize_act(X, mode, topk=topk)
            y_ref, acc_ref = B.bitlinear_gemm(qa["q"], qa["scale"], mode, M, K, p, a, N, y_dtype=torch.float32, want_acc=True)
            ws = B.workspace(mode, M, N, K, "cuda")
            if mode == B.BL_ACT_INT4_ABSMEAN:
                y, acc = B.bitlinear_a4(X, p, a, N, y_dtype=torch.float32, want_acc=True, ws=ws)
            else:
                y, acc = B.bitlinear_a8_sparse(X, topk, p, a, N, y_dtype=torch.float32, want_acc=True, ws=ws)
            assert torch.equal(acc, acc_ref)
            assert ((y == y_ref) | (y.isnan() & y_ref.isnan())).all()
            at = (qa["q"].numel() + 255) // 256 * 256
            assert torch.equal(ws[at:at + 4 * M].view(torch.int32), qa["scale"].view(torch.int32))


@pytest.mark.parametrize("M", [2, 33])
@pytest.mark.parametrize("N", [70, 72])
def test_nan_scale(M, N):
    """A weight scale that is NaN, of any payload, gives NaN outputs whatever the length of the rows."""
    print("[case] nan M=%d N=%d" % (M, N), flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + N)
    X = torch.randn((M, 264), generator=g, device="cuda").to(BF16)
    p, a = B.pack_ternary(torch.randn((N, 264), generator=g, device="cuda"))
    for bits in (0x7FC00000, 0x7FFFFFFF, -1):
        nan = torch.full((1,), bits, dtype=torch.int32, device="cuda").view(torch.float32)
        assert B.bitlinear_a4(X, p, nan, N).isnan().all() and B.bitlinear_a8_sparse(X, 100, p, nan, N).isnan().all()
