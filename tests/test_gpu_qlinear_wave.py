"""GPU parity of the layer on small grids (one output tile per workgroup, the contraction split over its
waves) against the fp64 oracle, at the edges of its tiles: M around 16, 32 and 64 rows and the counts
at which the tile shape changes, ragged N, and K of fewer chunks of 128 than waves, one round of them, and
remainders."""

import numpy as np
import pytest
import torch

import oracle
import paper_2607_02461_amd as oq
from paper_2607_02461_amd import workloads
from tests.gpu_util import check_gemm, gemm_scale, qlinear_oracle_bf16

pytestmark = pytest.mark.gpu

DEV = "cuda"

# (M, N, K): 16-row tiles (1 x 1 and, from 180 tiles on, 1 x 4), 32-row tiles (2 x 2, 2 x 4), 64-row
# tiles with eight waves (up to one tile per compute unit) and with four
SHAPES = [(1, 77, 128), (15, 1000, 384), (16, 12289, 256), (17, 640, 1024), (32, 11530, 256), (33, 3001, 1152),
          (64, 12288, 384), (65, 6400, 1280), (200, 3070, 640), (450, 4099, 512)]


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("ba,bw", [(4, 4), (3, 3), (2, 2), (6, 4), (4, 3), (3, 2), (6, 2)])
@pytest.mark.parametrize("epilogue", ["plain", "bias"])
def test_small_grids(M, N, K, ba, bw, epilogue):
    xc, wc = workloads.random_codes(M, K, ba, M + K), workloads.random_codes(N, K, bw, N + K)
    xs, wr = workloads.random_norms(M, M, 0), workloads.random_norms(N, N, 1).to(torch.bfloat16)
    bias = torch.linspace(-3, 3, N).to(torch.bfloat16) if epilogue == "bias" else None
    cba, cbw = oq.lloydmax_codebook(ba, K), oq.lloydmax_codebook(bw, K)
    xp = torch.from_numpy(oracle.pack_codes(oracle.to_labels(xc.numpy(), ba), ba)).to(DEV)
    wp = torch.from_numpy(oracle.pack_codes(oracle.to_labels(wc.numpy(), bw), bw)).to(DEV)
    out = torch.full((M, N + 3), float("nan"), device=DEV)
    Y = oq.orbit_qlinear_ex(cba, xp, xs.to(DEV), cbw, wp, wr.to(DEV), bias=bias.to(DEV) if bias is not None else None,
                            out=out[:, :N])
    again = oq.orbit_qlinear_ex(cba, xp, xs.to(DEV), cbw, wp, wr.to(DEV),
                                bias=bias.to(DEV) if bias is not None else None)
    torch.cuda.synchronize()
    assert torch.equal(Y, again) and bool(torch.isnan(out[:, N:]).all())
    ref = qlinear_oracle_bf16(xc.numpy(), xs.double().numpy(), ba, wc.numpy(), wr.double().numpy(), bw, K)
    la = oracle.bf16_round(oracle.lloydmax_codebook(ba, K).levels)
    lw = oracle.bf16_round(oracle.lloydmax_codebook(bw, K).levels)
    scale = gemm_scale(xc.numpy(), xs.double().numpy(), la, wc.numpy(), wr.double().numpy(), lw)
    slack = 0.0
    if bias is not None:
        # one fp32 rounding of a sum of at most |ref| + 3
        slack = 2.0 ** -23 * (np.abs(ref) + 3.0)
        ref = ref + bias.double().numpy()[None, :]
    check_gemm(f"small grid M={M} N={N} K={K} W{bw}A{ba} {epilogue}", Y.cpu().numpy(), ref, scale, K, slack=slack)
