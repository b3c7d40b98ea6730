"""Workgroups that fit a compute unit together, from the built library's metadata."""
import os

import pytest

from _code_objects import kernels, library, tool

LDS_BYTES, REGISTERS, SIMDS = 160 * 1024, 512, 4


@pytest.mark.skipif(not os.path.exists(tool("llvm-readelf")), reason="no llvm-readelf in this image")
def test_fp32_tiles_leave_room_for_a_second_wave(tmp_path):
    # A tile's fill and its store are waited out unless another wave of the same SIMD
    # has MFMAs to run: two workgroups of four waves a CU, or one of eight
    found = {k: v for k, v in kernels(library(), tmp_path).items() if "15gemm_f32_kernelI" in k}
    assert len(found) >= 11 * 4
    for name, k in found.items():
        waves = k["max_flat_workgroup_size"] // 64
        by_registers = REGISTERS // k["vgpr_count"] * SIMDS // waves
        by_lds = LDS_BYTES // k["group_segment_fixed_size"]
        assert min(by_registers, by_lds) * waves >= 2 * SIMDS, (name, k)
        assert k["private_segment_fixed_size"] == 0, (name, k)
