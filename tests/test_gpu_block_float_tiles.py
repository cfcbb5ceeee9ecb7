"""GPU parity of the block-float products on 64-token tiles: both arrangements of the waves, one and two K groups, the gate/up form
with 64 and with 128 outputs per block, ragged tokens and outputs, one K step and odd numbers of them."""
import pytest
import torch

from paper_2411_04965_amd import binding as B
from tests.test_gpu_prefill_tiles import product

pytestmark = pytest.mark.gpu
BF16 = torch.bfloat16


# on 256 CUs: 64 x 128 (the first four; the fourth with two K groups), 64 x 256 (the next three), then sizes at the rule against
# 256 x 256 tiles, either side.  Gate and up: 64 outputs per block up to (130, 2000), 128 from (300, 12000) on
@pytest.mark.parametrize("M,N,K", [(65, 1, 256), (66, 129, 200), (130, 2000, 777), (97, 300, 4100), (300, 12000, 264), (289, 8229, 1300),
                                   (1000, 4103, 520), (1000, 2700, 1024), (1500, 3071, 1024), (1500, 6141, 300), (700, 4099, 2050)])
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
