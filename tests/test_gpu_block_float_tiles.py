"""GPU parity of the block-float products on 64-token tiles: both arrangements of the waves, one and two K groups, the gate/up form
with 64 and with 128 outputs per block, ragged tokens and outputs, one K step and odd numbers of them, both sides of the rules."""
import pytest
import torch

from paper_2411_04965_amd import binding as B
from tests.test_gpu_prefill_tiles import product

pytestmark = pytest.mark.gpu
BF16 = torch.bfloat16


# on 256 CUs: 64 x 128 tiles in one turn with 2 x 2 waves (the first four; the fourth at the longest rows), with two K groups (the next two),
# with 1 x 4 waves (the next two: many tokens with few outputs, a third turn of 64 x 256 nearly empty), 64 x 256 (the next nine, among them
# sizes on the other side of the last rule and at the one against 256 x 256), 256 x 256 (the last).  Gate and up: 64 outputs per block in the
# first six, then 128, or 256 x 256 tiles in (1000, 4103), (1500, 3071), (6001, 3069) and (6500, 2700)
@pytest.mark.parametrize("M,N,K", [(65, 1, 256), (66, 129, 200), (130, 2000, 777), (100, 517, 3584), (100, 517, 3585), (97, 300, 4100),
                                   (16500, 100, 300), (912, 8829, 2056), (912, 8829, 3073), (300, 12000, 264), (289, 8229, 1300),
                                   (1000, 4103, 520), (1000, 2700, 1024), (1500, 3071, 1024), (700, 4099, 2050), (6001, 3069, 300),
                                   (6500, 2700, 1024), (1500, 6141, 300)])
def test_tiles(M, N, K):
    print("[case] block-float tiles M=%d N=%d K=%d" % (M, N, K), flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + N)
    X = torch.randn((M, K), generator=g, device="cuda").to(BF16)
    W = 0.02 * torch.randn((N, K), generator=g, device="cuda")
    Wu = 0.02 * torch.randn((N, K), generator=g, device="cuda")
    acc_ref, y_ref = product(X, W, B.BL_ACT_INT4_ABSMEAN)
    u_ref = product(X, Wu, B.BL_ACT_INT4_ABSMEAN)[1]
    p, a = B.pack_ternary(W, layout=B.BL_W_MX2)
    pu, au = B.pack_ternary(Wu, layout=B.BL_W_MX2)
    assert torch.equal(B.bitlinear_a4(X, p, a, N, layout=B.BL_W_MX2), y_ref.to(BF16))
    y, acc = B.bitlinear_a4(X, p, a, N, layout=B.BL_W_MX2, y_dtype=torch.float32, want_acc=True)
    assert torch.equal(y, y_ref) and torch.equal(acc, acc_ref.int())
    h = B.bitlinear_a4_gate_up(X, p, a, pu, au, N, layout=B.BL_W_MX2, want=("H",))["H"]
    assert torch.equal(h, (u_ref * y_ref.clamp_min(0.0).square()).to(BF16))
