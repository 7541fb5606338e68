"""Monte Carlo sweeps against the oracle around the numbers of bonds at which
the kernel holds another bond per lane (64 bonds each) and at the longest
chain it takes.

Both sides add the same proposals to the amplitudes, so states agree to
rounding (1e-12 of the largest amplitude) unless a decision differs, and the
energies, formed differently, agree to about 1e-12 of T*: for 1e5 proposals a
differing decision has a chance of 1e-7.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1411_3487_amd import Context, inputs, NU_DSDNA as NU, T_STAR_DSDNA as TS

pytestmark = pytest.mark.gpu

B_FAC = 1.0 / (1.0 - 2.0 * NU)


@pytest.mark.parametrize("M,scale", [(22, 3.0), (23, 3.0), (64, 0.0), (65, 3.0), (66, 3.0),
                                     (129, 3.0), (130, 3.0), (193, 1.0), (194, 3.0), (257, 3.0),
                                     (258, 3.0), (386, 3.0), (514, 3.0), (770, 3.0), (1026, 3.0),
                                     (1365, 3.0)])
def test_mc_matches_oracle_at_every_register_shape(M, scale):
    torch.cuda.set_device(0)
    B, n = 3, 2
    pos = inputs.straight_chains(B, M, B_FAC, seed=M, random_orientation=True, jitter=0.05)
    with Context(pos, seed=6, precision="fp64") as ctx:
        ctx.set_params([M], [1.0], T_star=TS, nu=NU)
        R0 = ctx.modes()
        acc = ctx.step_mc(n, scale) + ctx.step_mc(1, scale)
        got = ctx.modes()
    want, want_acc = oracle.mc_sweeps(R0, NU, TS, scale, n + 1, seed=6)
    assert acc == want_acc.sum()
    assert np.abs(got - want).max() <= 1e-12 * np.abs(want).max()
