"""The list of a call's kernel launches: names taken from the mangled ones, and a captured call that runs nothing."""

import pytest
import torch

import paper_2607_02461_amd as oq
from paper_2607_02461_amd.launches import launches, short_name


@pytest.mark.parametrize("mangled,short", [
    ("_ZN5orbit12_GLOBAL__N_115lut_gemm_kernelILi4ELi3ELb1EEEvNS_10GemmParamsE", "lut_gemm_kernel<4,3,true>"),
    ("_ZN5orbit12_GLOBAL__N_115lut_gemm_reduceENS_10GemmParamsEi", "lut_gemm_reduce"),
    ("_ZN5orbit12_GLOBAL__N_113lut_gemm_waveILi6ELi4ELi2ELi4ELi2EEEvNS_10GemmParamsE", "lut_gemm_wave<6,4,2,4,2>"),
    ("_Z4fillILin1ELb0EEvPf", "fill<-1,false>"),
    ("plain", "plain"),
])
def test_short_name(mangled, short):
    assert short_name(mangled) == short


@pytest.mark.gpu
def test_launches_are_listed_and_not_run():
    K = 1024
    plan, cb = oq.rpbh_plan(K, 128, 0), oq.lloydmax_codebook(4, K)
    X = torch.randn((33, K), device="cuda").to(torch.bfloat16)
    codes = torch.full((33, K // 2), 0xA5, dtype=torch.uint8, device="cuda")
    norms = torch.full((33,), -1.0, device="cuda")

    def call():
        oq.rpbh_quantize_act(plan, cb, X, 1e-10, codes, norms)

    ran = launches(call)
    torch.cuda.synchronize()
    assert len(ran) == 1 and "quantize" in ran[0].kernel and ran[0].grid[0] >= 1
    assert bool((codes == 0xA5).all()) and bool((norms == -1.0).all())
    call()
    torch.cuda.synchronize()
    assert bool((norms > 0).all())
