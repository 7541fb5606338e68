"""Split-BF16 chains of 386..448 beads (14 row tiles per half: the streamed
tables' blocks of 4 row tiles end in one of 3) against the oracle.  Over 10
steps from the straight chain the reduced path stays within 1e-5 of the
contour length of FP64 (split products 2^-17 of the bonds), as at the other
lengths."""
import numpy as np
import pytest
import torch

import oracle
from paper_1411_3487_amd import Context, inputs, NU_DSDNA as NU, T_STAR_DSDNA as TS

pytestmark = pytest.mark.gpu

B_FAC = 1.0 / (1.0 - 2.0 * NU)


@pytest.mark.parametrize("M", [386, 416, 448])
@pytest.mark.parametrize("mode", ["streamed", "auto"])
def test_lengths_of_fourteen_row_tiles(M, mode):
    torch.cuda.set_device(0)
    B, n = 7, 10
    pos = inputs.straight_chains(B, M, B_FAC, seed=M, random_orientation=True)
    with Context(pos, seed=5, precision="bf16x3") as ctx:
        ctx.set_params([M], [100.0], T_star=TS, nu=NU, table_mode=mode)
        ctx.step_modes(n)
        got = ctx.positions()
    R = oracle.step_modes(oracle.modes_from_positions(pos), NU, TS, 100.0, n, seed=5)
    err = np.abs(got - oracle.positions_from_modes(R)).max() / ((M - 1) * B_FAC)
    assert err < 1e-5, err
