"""The inextensible limit of chains of 2 beads, which have no neighbouring
tension and a kernel of their own, against the oracle: a bare chain, full and
ragged groups of a wavefront, both forms of the step, fixed cycles and cycles
that stop at convergence.  Bound 1e-10 of the chain length as for the other
lengths; a cycle that stops at 1e-12 moves a bond by no more than that in
each of the 100 steps after it."""
import numpy as np
import pytest
import torch

import oracle
from paper_1411_3487_amd import Context
from paper_1411_3487_amd.inputs import unit_chains

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("midpoint", [True, False])
@pytest.mark.parametrize("tol", [0.0, 1e-12])
@pytest.mark.parametrize("B", [1, 4, 17, 1025])
def test_pairs_match_oracle(B, tol, midpoint):
    torch.cuda.set_device(0)
    T, dt, n = 0.2, 2e-3, 100
    pos = unit_chains(B, 2, 3)
    with Context(pos, seed=21, precision="fp64") as ctx:
        ctx.step_wlc(n, dt, T, iters=12, tol=tol, midpoint=midpoint)
        got = ctx.positions()
    want = oracle.step_wlc(pos, T, dt, n, iters=12, seed=21, midpoint=midpoint)
    assert np.abs(got - want).max() < (1e-10 if tol == 0.0 else 3e-10)
