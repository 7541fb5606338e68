"""Positions written to a device array in the caller's chain order, against
the oracle's transform of the same amplitudes, at lengths around the 32 x 32
tiles of the general product, the multiples of 16 that take the other one, and
ragged ensembles.  A sum of M products of magnitude |phi R| rounds to M 2^-53 of
their absolute sum; the tables add a few units in the last place."""
import numpy as np
import pytest
import torch

import oracle
from paper_1411_3487_amd import Context, inputs, NU_DSDNA as NU, T_STAR_DSDNA as TS

pytestmark = pytest.mark.gpu

B_FAC = 1.0 / (1.0 - 2.0 * NU)


@pytest.mark.parametrize("lens,B", [([2], 1), ([31], 11), ([33], 10), ([63], 300), ([65], 21),
                                    ([129, 48, 257], 37), ([64, 130, 31, 512], 25), ([515], 3)])
def test_device_positions(lens, B):
    torch.cuda.set_device(0)
    beads = inputs.mixed_lengths(B, lens, seed=1)
    chains = inputs.mixed_chains(beads, B_FAC, seed=2, jitter=0.1)
    have = sorted(set(int(m) for m in beads))
    with Context(chains, seed=2, precision="fp64", stream=torch.cuda.current_stream()) as ctx:
        ctx.set_params(have, [10.0] * len(have), T_star=TS, nu=NU)
        ctx.step_modes(3)
        R = ctx.modes()
        dst = torch.full((int(3 * beads.sum()),), np.nan, dtype=torch.float64, device="cuda")
        ctx.positions_to_device(dst.data_ptr())
        got = dst.cpu().numpy()
        host = ctx.positions()
    at = 0
    for c, M in enumerate(beads):
        r = np.asarray(R[c])[None]
        want = oracle.positions_from_modes(r)[0]
        scale = np.abs(r).sum() * np.sqrt(2.0 / M)
        piece = got[at:at + 3 * M].reshape(3, M)
        assert np.abs(piece - want).max() <= (M + 8) * 2.0 ** -53 * scale
        assert np.array_equal(piece, host[c])
        at += 3 * M
