"""GPU parity of the many-token GEMMs at the edges of their tiles: output rows of any length (every remainder of the
16-byte stores), tokens around tile edges, and sizes on both sides of the dispatch rules."""
import numpy as np
import pytest
import torch

from oracle import bitnet_a48 as O
from paper_2411_04965_amd import binding as B
from paper_2411_04965_amd import synth as S
from tests.gpu_util import EPS, dev, host, pack

pytestmark = pytest.mark.gpu
BF16 = torch.bfloat16


@pytest.mark.parametrize("M,N,K", [(70, 129, 256), (129, 131, 300), (1030, 1026, 256), (1030, 1027, 256), (1025, 1028, 256),
                                   (1030, 1029, 256), (65, 255, 256), (300, 1031, 512)])
def test_rows_of_any_length(M, N, K):
    """bfloat16 rows whose length is no multiple of 8: both linears and the gate/up front, bit for bit."""
    print("[case] rows M=%d N=%d K=%d" % (M, N, K), flush=True)
    X = S.heavy(M, K, S.seed_for(6, M + N))
    W = S.latent_weights(N, K, S.seed_for(6, N + K))
    Wu = S.latent_weights(N, K, S.seed_for(6, N + K + 1))
    Xd = dev(X, BF16)
    ref = O.bitlinear_a4(X, W, EPS, "bf16")["y"]
    g, u = O.bitlinear_a4(X, W, EPS, "f32")["y"], O.bitlinear_a4(X, Wu, EPS, "f32")["y"]
    for layout in (B.BL_W_GEMM, B.BL_W_MX2, B.BL_W_MX4):
        p, a = pack(W, layout)
        assert np.array_equal(host(B.bitlinear_a4(Xd, p, a, N, EPS, layout=layout)), ref)
        if layout != B.BL_W_GEMM:
            pu, au = pack(Wu, layout)
            h = B.bitlinear_a4_gate_up(Xd, p, a, pu, au, N, EPS, layout, want=("H",))["H"]
            assert np.array_equal(host(h), O.relu2_glu(g, u))
    p, a = pack(W)
    ref8 = O.bitlinear_a8_sparse(X, W, K // 2, EPS, "bf16")["y"]
    assert np.array_equal(host(B.bitlinear_a8_sparse(Xd, K // 2, p, a, N, EPS)), ref8)


def product(X, W, mode, topk=0):
    """The product stage on codes from the library's own quantizers (which have their own tests), in plain torch: integer
    sums are below 2^24 and so exact in float32."""
    M, K = X.shape
    p, a = B.pack_ternary(W)
    qa = B.quantize_act(X, mode, topk=topk)
    acc = B.unpack_act(qa["q"], mode, M, K).float() @ B.unpack_ternary(p, W.shape[0], K).float().T
    return acc, (acc * qa["scale"][:, None]) * a


# (tokens, outputs, channels) that reach each tile of the many-token GEMMs on 256 CUs, with ragged edges, one K step (fewer
# than K groups), odd and even numbers of steps: 64 x 64, 64 x 128 with one and two K groups, 128 x 128, 256 x 256 (integer codes of up to
# 256 tokens go through the fragment-order products here, and through these tiles in test_gpu_row_order.py)
TILES = [(65, 63, 200), (191, 1021, 257), (130, 516, 700), (449, 3211, 1025), (833, 2045, 300), (641, 4091, 520), (1153, 2052, 777),
         (4090, 4091, 300), (4097, 4100, 520), (2900, 6141, 256)]


@pytest.mark.parametrize("M,N,K", TILES)
def test_tiles(M, N, K):
    """Every tile and number format, bfloat16 and float32 outputs and accumulators, bit for bit."""
    print("[case] tiles M=%d N=%d K=%d" % (M, N, K), flush=True)
    g = torch.Generator(device="cuda").manual_seed(M)
    X = torch.randn((M, K), generator=g, device="cuda").to(BF16)
    W = 0.02 * torch.randn((N, K), generator=g, device="cuda")
    Wu = 0.02 * torch.randn((N, K), generator=g, device="cuda")
    acc8, y8 = product(X, W, B.BL_ACT_TOPK_INT8_ABSMAX, K // 2)
    acc4, y4 = product(X, W, B.BL_ACT_INT4_ABSMEAN)
    u4 = product(X, Wu, B.BL_ACT_INT4_ABSMEAN)[1]
    p, a = B.pack_ternary(W)
    assert torch.equal(B.bitlinear_a8_sparse(X, K // 2, p, a, N), y8.to(BF16))
    y, acc = B.bitlinear_a8_sparse(X, K // 2, p, a, N, y_dtype=torch.float32, want_acc=True)
    assert torch.equal(y, y8) and torch.equal(acc, acc8.int())
    assert torch.equal(B.bitlinear_a4(X, p, a, N), y4.to(BF16))
    y, acc = B.bitlinear_a4(X, p, a, N, want_acc=True)
    assert torch.equal(y, y4.to(BF16)) and torch.equal(acc, acc4.int())
    p, a = B.pack_ternary(W, layout=B.BL_W_MX2)
    pu, au = B.pack_ternary(Wu, layout=B.BL_W_MX2)
    assert torch.equal(B.bitlinear_a4(X, p, a, N, layout=B.BL_W_MX2), y4.to(BF16))
    y, acc = B.bitlinear_a4(X, p, a, N, layout=B.BL_W_MX2, y_dtype=torch.float32, want_acc=True)
    assert torch.equal(y, y4) and torch.equal(acc, acc4.int())
    h = B.bitlinear_a4_gate_up(X, p, a, pu, au, N, layout=B.BL_W_MX2, want=("H",))["H"]
    assert torch.equal(h, (u4 * y4.clamp_min(0.0).square()).to(BF16))


# both sides of 32 tokens; K of one step and of an odd number; outputs past one turn of the smallest tile and of the next one (fragment
# order, except the two widest; the kernels behind it: test_gpu_row_order.py)
@pytest.mark.parametrize("M,N,K,mul", [(32, 70, 300, 1.0), (33, 70, 200, 1.0), (33, 1027, 1300, 1e-36), (57, 5460, 2048, 1.0),
                                       (64, 16452, 520, 1.0), (63, 32901, 257, 1.0), (64, 260, 4200, 1.0)])
def test_decode_tokens(M, N, K, mul):
    """33 to 64 tokens in the two-bit tile layout, the gate/up front among them, bit for bit; with tiny activations too, whose
    scales have no binades to spare."""
    print("[case] decode tiles M=%d N=%d K=%d mul=%g" % (M, N, K, mul), flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + N)
    X = (mul * torch.randn((M, K), generator=g, device="cuda")).to(BF16)
    W = 0.02 * torch.randn((N, K), generator=g, device="cuda")
    Wu = 0.02 * torch.randn((N, K), generator=g, device="cuda")
    acc8, y8 = product(X, W, B.BL_ACT_TOPK_INT8_ABSMAX, K // 2)
    acc4, y4 = product(X, W, B.BL_ACT_INT4_ABSMEAN)
    u4 = product(X, Wu, B.BL_ACT_INT4_ABSMEAN)[1]
    p, a = B.pack_ternary(W)
    pu, au = B.pack_ternary(Wu)
    assert torch.equal(B.bitlinear_a8_sparse(X, K // 2, p, a, N), y8.to(BF16))
    y, acc = B.bitlinear_a8_sparse(X, K // 2, p, a, N, y_dtype=torch.float32, want_acc=True)
    assert torch.equal(y, y8) and torch.equal(acc, acc8.int())
    assert torch.equal(B.bitlinear_a4(X, p, a, N), y4.to(BF16))
    y, acc = B.bitlinear_a4(X, p, a, N, y_dtype=torch.float32, want_acc=True)
    assert torch.equal(y, y4) and torch.equal(acc, acc4.int())
    h = B.bitlinear_a4_gate_up(X, p, a, pu, au, N, want=("H",))["H"]
    assert torch.equal(h, (u4 * y4.clamp_min(0.0).square()).to(BF16))


# more than 32 tokens: both sides of the rule on long K (INT8 codes: from 26 K tiles on, from 29 below 40 tokens, with outputs up
# to 2048, 512 per K tile beyond 28 or 30, 5120 or 6144; INT4 codes: from 30 on with 512, or 512 per tile beyond 31 and 176 per tile
# beyond 20), one and two turns of the chip.  The linears take fragment order at most of these; the rule itself is tested on codes in row
# order (test_gpu_row_order.py)
@pytest.mark.parametrize("M,N,K", [(40, 70, 6401), (39, 70, 7168), (64, 2048, 6656), (64, 2049, 6500), (33, 2048, 7937), (47, 512, 7600),
                                   (64, 513, 7680), (64, 2560, 9216), (40, 2561, 9000), (64, 5120, 10241), (57, 5121, 9985),
                                   (35, 4916, 20480), (50, 6144, 13500), (33, 333, 32768), (64, 6144, 24577)])
def test_decode_tokens_long_k(M, N, K):
    """33 to 64 tokens with K split over blocks and without, bit for bit."""
    print("[case] decode long K M=%d N=%d K=%d" % (M, N, K), flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + N)
    X = torch.randn((M, K), generator=g, device="cuda").to(BF16)
    W = 0.02 * torch.randn((N, K), generator=g, device="cuda")
    p, a = B.pack_ternary(W)
    for mode, call in ((B.BL_ACT_TOPK_INT8_ABSMAX, lambda **kw: B.bitlinear_a8_sparse(X, K // 2, p, a, N, **kw)),
                       (B.BL_ACT_INT4_ABSMEAN, lambda **kw: B.bitlinear_a4(X, p, a, N, **kw))):
        acc_ref, y_ref = product(X, W, mode, K // 2)
        assert torch.equal(call(), y_ref.to(BF16))
        y, acc = call(y_dtype=torch.float32, want_acc=True)
        assert torch.equal(y, y_ref) and torch.equal(acc, acc_ref.int())


# (tokens, outputs, channels) for which the persistent kernels' blocks walk on to a second tile, on 256 CUs, with rows whose length is
# no multiple of 8 in bfloat16 and a multiple of 4 in float32: 256 x 256 tiles (416 of them), 128 x 128 tiles for short K and few
# outputs (645 with three steps of K for INT8 codes, 645 and 96 with one step)
@pytest.mark.parametrize("M,N,K", [(8190, 3197, 300), (8190, 3196, 777), (16500, 515, 700), (16500, 516, 513), (16500, 517, 256),
                                   (16500, 516, 255), (3000, 389, 256)])
def test_blocks_walk_on(M, N, K):
    """Persistent blocks with ragged rows, both code formats, bfloat16 and float32 outputs and accumulators, bit for bit."""
    print("[case] walk M=%d N=%d K=%d" % (M, N, K), flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + N)
    X = torch.randn((M, K), generator=g, device="cuda").to(BF16)
    W = 0.02 * torch.randn((N, K), generator=g, device="cuda")
    p, a = B.pack_ternary(W)
    for mode, call in ((B.BL_ACT_TOPK_INT8_ABSMAX, lambda **kw: B.bitlinear_a8_sparse(X, K // 2, p, a, N, **kw)),
                       (B.BL_ACT_INT4_ABSMEAN, lambda **kw: B.bitlinear_a4(X, p, a, N, **kw))):
        acc_ref, y_ref = product(X, W, mode, K // 2)
        assert torch.equal(call(), y_ref.to(BF16))
        for dt in (BF16, torch.float32):
            y, acc = call(y_dtype=dt, want_acc=True)
            assert torch.equal(y, y_ref.to(dt)) and torch.equal(acc, acc_ref.int())
    for layout in (B.BL_W_MX2, B.BL_W_MX4):
        p2, a2 = B.pack_ternary(W, layout=layout)
        assert torch.equal(B.bitlinear_a4(X, p2, a2, N, layout=layout), y_ref.to(BF16))


@pytest.mark.parametrize("layout", [B.BL_W_MX2, B.BL_W_MX4])
@pytest.mark.parametrize("M,N,K", [(8190, 3197, 300), (8190, 3196, 777), (300, 517, 256)])
def test_block_float_outputs(M, N, K, layout):
    """The block-float GEMMs in every output form, blocks that walk on to a second tile among them: INT4 codes bit for bit; FP4 codes,
    whose two output types round the same float32 sums, against each other."""
    print("[case] block float M=%d N=%d K=%d layout=%d" % (M, N, K, layout), flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + N)
    X = torch.randn((M, K), generator=g, device="cuda").to(BF16)
    W = 0.02 * torch.randn((N, K), generator=g, device="cuda")
    acc_ref, y_ref = product(X, W, B.BL_ACT_INT4_ABSMEAN)
    p, a = B.pack_ternary(W, layout=layout)
    for dt in (BF16, torch.float32):
        assert torch.equal(B.bitlinear_a4(X, p, a, N, layout=layout, y_dtype=dt), y_ref.to(dt))
        y, acc = B.bitlinear_a4(X, p, a, N, layout=layout, y_dtype=dt, want_acc=True)
        assert torch.equal(y, y_ref.to(dt)) and torch.equal(acc, acc_ref.int())
    y = B.bitlinear_a4(X, p, a, N, layout=layout, act_fp4=True, y_dtype=torch.float32)
    assert torch.equal(B.bitlinear_a4(X, p, a, N, layout=layout, act_fp4=True), y.to(BF16))


# 33 to 64 tokens: gate and up, on 256 CUs all through the fragment-order products (other kernels: test_gpu_row_order.py)
@pytest.mark.parametrize("M,N,K", [(33, 70, 1025), (64, 4096, 1200), (50, 4097, 1200), (64, 4090, 1024), (64, 1021, 4096), (47, 2688, 4001)])
def test_decode_gate_up(M, N, K):
    """Gate and up with eq. 5 in the same launch, bit for bit."""
    print("[case] gate/up M=%d N=%d K=%d" % (M, N, K), flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + N)
    X = torch.randn((M, K), generator=g, device="cuda").to(BF16)
    W = 0.02 * torch.randn((N, K), generator=g, device="cuda")
    Wu = 0.02 * torch.randn((N, K), generator=g, device="cuda")
    g4, u4 = product(X, W, B.BL_ACT_INT4_ABSMEAN)[1], product(X, Wu, B.BL_ACT_INT4_ABSMEAN)[1]
    p, a = B.pack_ternary(W)
    pu, au = B.pack_ternary(Wu)
    h = B.bitlinear_a4_gate_up(X, p, a, pu, au, N, want=("H",))["H"]
    assert torch.equal(h, (u4 * g4.clamp_min(0.0).square()).to(BF16))
