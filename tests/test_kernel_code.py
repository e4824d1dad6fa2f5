"""What the compiler made of the kernels, read off the built library: properties that the sources rely on and that
no result shows."""

import re

from tests.code_objects import disassembly, kernel_metadata, mfma_hazards


def test_wave_kernel_keeps_its_loop_in_registers():
    # every instance of the small-grid kernel: nothing spilled, and room for two workgroups of eight waves on a
    # compute unit (128 of a SIMD's 512 registers per wave) with the 32 x 64 tile
    kernels = {n: k for n, k in kernel_metadata().items() if n.startswith("lut_gemm_wave<")}
    assert len(kernels) == 72
    for name, k in kernels.items():
        assert k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0, f"{name} spills"
        assert k[".max_flat_workgroup_size"] == 512, name
        if re.match(r"lut_gemm_wave<\d,\d,2,4,", name):
            assert k[".vgpr_count"] <= 128, f"{name} takes {k['.vgpr_count']} registers"
    # the 32 x 64 tile has two chunks of codes in flight wherever they fit those registers
    assert {n for n in kernels if re.match(r"lut_gemm_wave<\d,\d,2,4,1", n)} == {"lut_gemm_wave<6,3,2,4,1>", "lut_gemm_wave<6,4,2,4,1>"}


def test_hazards_are_seen():
    acc = ["v[0:3]", "v[8:11]", "v[12:15]", "v[0:3]"]
    mfma = ("v_mfma_f32_16x16x32_bf16", acc)
    assert mfma_hazards([("v_mov_b32_e32", ["v3", "0"]), ("s_nop", ["1"]), mfma]) == []
    assert len(mfma_hazards([("v_mov_b32_e32", ["v3", "0"]), ("s_nop", ["0"]), mfma])) == 1       # the accumulator
    assert len(mfma_hazards([("v_perm_b32", ["v9", "v20", "v21", "v22"]), mfma])) == 1            # a fragment
    assert len(mfma_hazards([("v_permlane32_swap_b32_e32", ["v20", "v12"]), mfma])) == 1
    assert mfma_hazards([mfma, mfma, ("s_nop", ["15"]), ("v_mul_f32_e32", ["v20", "v0", "v21"])]) == []
    assert len(mfma_hazards([mfma, ("s_nop", ["9"]), ("v_mul_f32_e32", ["v20", "v3", "v21"])])) == 1
    assert len(mfma_hazards([mfma, ("global_store_dwordx4", ["v[30:31]", "v[0:3]", "off"])])) == 1


def test_large_kernel_keeps_the_wait_states_of_its_mfmas():
    # its MFMAs are inline asm, whose wait states the compiler does not see to
    kernels = {n: c for n, c in disassembly().items() if n.startswith("lut_gemm_big<")}
    assert len(kernels) == 12
    for name, code in kernels.items():
        assert sum(i[0] == "v_mfma_f32_16x16x32_bf16" for i in code) >= 4 * 64, name
        assert mfma_hazards(code) == [], name


def test_adaln_kernel_fits_the_workgroups_its_launcher_counts_on():
    # workgroups of four waves on a compute unit, one wave of each per SIMD of 512 registers
    kernels = {n: k for n, k in kernel_metadata().items() if n.startswith("adaln_int4_linear_kernel<")}
    fit = {"<1,1>": 6, "<1,2>": 6, "<2,1>": 3, "<2,2>": 3, "<4,1>": 4, "<4,2>": 3}
    assert {n[n.index("<"):] for n in kernels} == set(fit)
    for name, k in kernels.items():
        assert k[".vgpr_spill_count"] == 0, name
        assert 512 // ((k[".vgpr_count"] + 7) // 8 * 8) == fit[name[name.index("<"):]], f"{name} takes {k['.vgpr_count']}"
