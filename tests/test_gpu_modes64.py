"""The persistent FP64 stepper against the oracle at the edges of its tiles:
the first and last chains of 5- and 16-chain tiles, lengths around the 16-row
half tiles and the limits of each kernel shape, even and odd, with shear, and
ensembles of many lengths in one launch (with one beyond its range, which
takes the dense steps).

Tolerance relative to the contour length: the oracle forms zeta_p by the
subtraction zeta^l_p - (1 - 2 nu) 4 s^2, off by up to 4 * 2^-53 from the
library's product, so E_p differs by 4 * 2^-53 dtau per step and 20 steps of
dtau = 100 by 9e-13; rounding adds a few 1e-14.  1e-11 holds both.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1411_3487_amd import Context, inputs, NU_DSDNA as NU, T_STAR_DSDNA as TS

pytestmark = pytest.mark.gpu

B_FAC = 1.0 / (1.0 - 2.0 * NU)
TOL = 1e-11
STEPS = 20


@pytest.fixture(scope="module", autouse=True)
def _device():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    torch.cuda.set_device(0)
    yield
    torch.cuda.synchronize()


def check(got, pos, ids, M, dtau, seed, gdot=0.0, nonlinear=True):
    R = oracle.modes_from_positions(pos)
    R = oracle.step_modes(R, NU, TS, dtau, STEPS, seed=seed, chain_ids=ids, gamma_dot=gdot,
                          nonlinear=nonlinear)
    err = np.abs(got - oracle.positions_from_modes(R)).max() / ((M - 1) * B_FAC)
    assert err < TOL, (M, err)


@pytest.mark.parametrize("B,M,dtau", [
    (1, 2, 1.0), (4, 3, 1.0), (5, 31, 10.0), (6, 32, 10.0), (5, 33, 10.0), (9, 64, 10.0),
    (11, 65, 10.0), (16, 97, 10.0), (5, 128, 50.0), (6, 129, 50.0), (7, 256, 100.0),
    (6, 257, 100.0), (4, 511, 100.0), (6, 512, 100.0), (2, 513, 100.0),
    (2, 514, 100.0)])
def test_five_chain_tiles(B, M, dtau):
    pos = inputs.straight_chains(B, M, B_FAC, seed=M, random_orientation=True)
    gdot = 1e-4 if B % 2 else 0.0
    with Context(pos, seed=M + 1, precision="fp64") as ctx:
        ctx.set_params([M], [dtau], T_star=TS, nu=NU, gamma_dot=gdot)
        ctx.step_modes(STEPS)
        got = ctx.positions()
    check(got, pos, np.arange(B), M, dtau, M + 1, gdot)


@pytest.mark.parametrize("M", [130, 255, 256])
@pytest.mark.parametrize("gdot,nonlinear", [(0.0, True), (1e-4, True), (1e-4, False)])
def test_sixteen_chain_tiles(M, gdot, nonlinear):
    # more than two rounds of 5-chain tiles on 256 compute units, less than
    # one of 16-chain tiles; 10 chains in the last tile
    B, dtau = 2570, 50.0
    pos = inputs.straight_chains(B, M, B_FAC, seed=M, random_orientation=True)
    with Context(pos, seed=9, precision="fp64") as ctx:
        ctx.set_params([M], [dtau], T_star=TS, nu=NU, gamma_dot=gdot, nonlinear=nonlinear)
        ctx.step_modes(STEPS)
        got = ctx.positions()
    ids = np.array([0, 1, 15, 16, 31, 1000, 2559, 2560, 2568, 2569])
    check(got[ids], pos[ids], ids, M, dtau, 9, gdot, nonlinear)


@pytest.mark.parametrize("B,M,gdot", [(4090, 128, 0.0), (3700, 96, 1e-4), (6300, 64, 1e-4),
                                      (8190, 30, 0.0)])
def test_sixteen_chain_tiles_of_short_chains(B, M, gdot):
    pos = inputs.straight_chains(B, M, B_FAC, seed=M, random_orientation=True)
    with Context(pos, seed=9, precision="fp64") as ctx:
        ctx.set_params([M], [10.0], T_star=TS, nu=NU, gamma_dot=gdot)
        ctx.step_modes(STEPS)
        got = ctx.positions()
    ids = np.array([0, 15, 16, 17, 2000, B - 17, B - 2, B - 1])
    check(got[ids], pos[ids], ids, M, 10.0, 9, gdot)


@pytest.mark.parametrize("lens", [[2, 33, 64, 65], [20, 100, 130, 257, 400, 513, 514]])
def test_many_lengths_in_one_launch(lens):
    beads = np.random.default_rng(1).permutation(np.repeat(np.array(lens, dtype=np.int32), 6))
    chains = inputs.mixed_chains(beads, B_FAC, seed=3)
    dtau = 10.0
    with Context(chains, seed=4, precision="fp64") as ctx:
        ctx.set_params(lens, [dtau] * len(lens), T_star=TS, nu=NU, sample_every=7, use_graphs=True)
        ctx.step_modes(STEPS)
        got = ctx.positions()
    for M in lens:
        ids = np.flatnonzero(beads == M)
        check(np.stack([got[c] for c in ids]), np.stack([chains[c] for c in ids]), ids, M, dtau, 4)
