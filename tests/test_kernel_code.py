"""What the compiler made of the kernels, read off the built library: properties that the sources rely on and that
no result shows."""

import re

from tests.code_objects import kernel_metadata


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
