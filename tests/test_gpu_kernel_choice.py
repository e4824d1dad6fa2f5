"""Which kernel a layer's rows run on, at the sizes where the choice is close: read off the recorded call."""

import pytest
import torch

import paper_2607_02461_amd as oq
from paper_2607_02461_amd.launches import launches

pytestmark = pytest.mark.gpu

DEV = "cuda"


def kernels(M, N, K, ba, bw, workspace=False):
    cba, cbw = oq.lloydmax_codebook(ba, K), oq.lloydmax_codebook(bw, K)
    xp, wp = (torch.zeros((r, K * b // 8), dtype=torch.uint8, device=DEV) for r, b in ((M, ba), (N, bw)))
    xs, wr = torch.zeros(M, device=DEV), torch.zeros(N, dtype=torch.bfloat16, device=DEV)
    out = torch.empty((M, N), device=DEV)
    if not workspace:
        return [r.kernel.split("<")[0] for r in launches(lambda: oq.orbit_qlinear(cba, xp, xs, cbw, wp, wr, out=out))]
    ws = torch.empty(oq.orbit_qlinear_workspace_size(M, N, K), dtype=torch.uint8, device=DEV)
    return [r.kernel.split("<")[0] for r in launches(lambda: oq.orbit_qlinear_ws(cba, xp, xs, cbw, wp, wr, ws, out=out))]


# microseconds on 128 x 128 tiles, wave tiles and large tiles are beside each layer
@pytest.mark.parametrize("M,N,K,ba,bw,workspace,kernel", [
    # short contractions, where a wave tile's fixed cost decides
    (1319, 5120, 640, 2, 4, False, "lut_gemm_kernel"),     # 20.2, 27.4
    (1183, 9216, 384, 4, 4, False, "lut_gemm_kernel"),     # 24.3, 35.2, 21.7
    (559, 9216, 640, 6, 4, False, "lut_gemm_kernel"),      # 24.5, 30.8
    (64, 3072, 640, 4, 4, False, "lut_gemm_wave"),
    # a long contraction of few outputs in many splits, whose reduction decides
    (156, 385, 13824, 4, 4, True, "lut_gemm_wave"),        # 44.8, 18.0
    (1, 223, 13824, 4, 4, True, "lut_gemm_wave"),          # 33, 10
    # 6-bit codes on 64 x 64 wave tiles against the split kernel
    (365, 9584, 3072, 6, 4, True, "lut_gemm_kernel"),      # 54.2, 59.7
    (271, 9216, 12288, 6, 3, True, "lut_gemm_kernel"),     # 138, 156
    # and 4-bit ones
    (1388, 3072, 5120, 4, 4, True, "lut_gemm_wave"),       # 79.9, 68.8
    # K no multiple of 128: never on wave tiles
    (1, 3072, 3136, 4, 4, False, "lut_gemm_kernel"),
    # one partial round of large tiles
    (4429, 3072, 3072, 3, 3, False, "lut_gemm_big"),       # 129, -, 85
])
def test_kernel_of_a_layer(M, N, K, ba, bw, workspace, kernel):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the expected kernels are those of 256 compute units")
    ran = kernels(M, N, K, ba, bw, workspace)
    assert ran[0] == kernel, ran
    assert ran[1:] == (["lut_gemm_reduce"] if workspace and kernel == "lut_gemm_kernel" else [])
