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
