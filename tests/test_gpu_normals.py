"""The FP64 normals the GPU draws, against the oracle's (C library log, sqrt,
cos and sin on the same Philox words), through one step of free modes:
R' = E R + W z, so z = (R' - E R) / W.

Tolerance: the device normal is within 4e-16 and the library pair within
8e-16 of the exact one relative to its radius, which is at most
sqrt(66 ln 2) = 6.77; the update rounds its products and sum (4 units of R'),
and E of the tables and of this file may differ by a few units (8 of E R).
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1411_3487_amd import Context, inputs, NU_DSDNA as NU, T_STAR_DSDNA as TS

pytestmark = pytest.mark.gpu

B_FAC = 1.0 / (1.0 - 2.0 * NU)


@pytest.mark.parametrize("B,M,seed", [(300, 64, 5), (150, 65, 1 << 40), (200, 31, 77)])
def test_fp64_normals_match_the_oracle(B, M, seed):
    torch.cuda.set_device(0)
    dtau = 10.0
    pos = inputs.straight_chains(B, M, B_FAC, seed=1, random_orientation=True)
    pos -= pos.mean(axis=2, keepdims=True)
    with Context(pos, seed=seed, precision="fp64") as ctx:
        ctx.set_params([M], [dtau], T_star=TS, nu=NU, nonlinear=False)
        R0 = ctx.modes()
        ctx.step_modes(1)
        R1 = ctx.modes()
    s2 = np.sin(np.pi * np.arange(M) / (2 * M)) ** 2
    z = 16 * NU * s2 * s2
    E = np.exp(-z * dtau)
    W = np.full(M, np.sqrt(2 * TS * dtau))
    W[1:] = np.sqrt(-TS * np.expm1(-2 * z[1:] * dtau) / z[1:])
    got = (R1 - E * R0) / W
    want = np.array([[np.concatenate([oracle.gauss4(seed, q, c, 0, a, oracle.TAG_MODE)
                                      for q in range((M + 3) // 4)])[:M]
                      for a in range(3)] for c in range(B)])
    tol = 12e-16 * 6.77 + 2.0 ** -53 * (4 * np.abs(R1) + 8 * np.abs(E * R0)) / W
    assert np.all(np.abs(got - want) <= tol)
