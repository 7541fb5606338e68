"""The inextensible limit against the oracle where the register kernel changes
shape: chains that fill 16, 32 or 64 lanes of four bonds exactly, one bond
more or less, groups without a chain at the end of a launch, and a cycle that
stops at convergence chain by chain.  Bound 1e-10 of the chain length as for
the other lengths (rounding of 1e-16 per step, 100 steps, amplified by the
tension solve by less than 1e3)."""
import numpy as np
import pytest
import torch

import oracle
from paper_1411_3487_amd import Context
from paper_1411_3487_amd.inputs import unit_chains

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("midpoint", [True, False])
@pytest.mark.parametrize("B,M", [(1, 5), (5, 6), (17, 33), (3, 63), (4, 64), (3, 127), (9, 128),
                                 (2, 129), (5, 130), (3, 255), (6, 256), (2, 257)])
def test_wlc_matches_oracle_around_the_lane_groups(B, M, midpoint):
    torch.cuda.set_device(0)
    T, dt, n = 0.2, 2e-3, 100
    pos = unit_chains(B, M, M + 1)
    with Context(pos, seed=21, precision="fp64") as ctx:
        ctx.step_wlc(n, dt, T, iters=8, midpoint=midpoint)
        got = ctx.positions()
    want = oracle.step_wlc(pos, T, dt, n, iters=8, seed=21, midpoint=midpoint)
    assert np.abs(got - want).max() / (M - 1) < 1e-10


@pytest.mark.parametrize("M", [30, 90, 200])
def test_wlc_chains_of_a_wavefront_converge_apart(M):
    """A straight chain next to crumpled ones: each stops its own cycle, so
    the result does not depend on the chains beside it."""
    torch.cuda.set_device(0)
    T, dt, n = 1.0 / 114.4, 1e-3, 50
    pos = unit_chains(6, M, M)
    pos[2] = unit_chains(1, M, 7, T_bar=1e-4)[0]
    with Context(pos, seed=8, precision="fp64") as ctx:
        ctx.step_wlc(n, dt, T, iters=16, tol=1e-7)
        got = ctx.positions()
    for c in range(6):
        # the same chain with copies of itself in the other groups: chain c
        # keeps its noise
        same = np.repeat(pos[c:c + 1], 6, axis=0)
        with Context(same, seed=8, precision="fp64") as ctx:
            ctx.step_wlc(n, dt, T, iters=16, tol=1e-7)
            assert np.array_equal(ctx.positions()[c], got[c])
