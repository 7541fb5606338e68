"""Register budgets that a change of a shared function can move (the noise of
every FP64 kernel is inlined).  CPU only: hipcc cross-compiles."""
import os

import pytest

from test_build_resources import HIPCC, resource_report


def test_wlc_wave_kernel_keeps_the_registers_its_lds_leaves_it():
    """At most 3 chains of 257 beads or more fit the LDS of a compute unit:
    registers for more than 4 wavefronts a SIMD only cost reads in flight."""
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    (r,) = [r for n, r in resource_report("dm_plain.hip").items() if "wlc_wave_kernel" in n]
    assert int(r["Occupancy"]) <= 4
    assert int(r["ScratchSize"]) == 0


def test_paired_fp64_tiles_fit_two_workgroups_of_8_wavefronts():
    """The last template argument asks for it: 4 wavefronts a SIMD."""
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    lean = [r for n, r in resource_report("dm_modes64.hip").items()
            if "modes64_kernel" in n and "Lb0ELb0ELi0ELb1E" in n]
    assert len(lean) == 1 and int(lean[0]["Occupancy"]) == 4
    assert int(lean[0]["ScratchSize"]) <= 16
