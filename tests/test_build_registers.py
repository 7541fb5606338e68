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
