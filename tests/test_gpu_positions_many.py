"""More chains than the 65536 workgroups of a second grid dimension hold 32
columns each for (699050): positions in, amplitudes
and positions out of 700000 chains of 3 beads.  Two products of 3 terms each round to 3 2^-53 of their absolute sum, at most sqrt(3) times the
chain's sum of magnitudes; the tables add a few units in the last place."""
import numpy as np
import pytest
import torch

from paper_1411_3487_amd import Context

pytestmark = pytest.mark.gpu


def test_positions_of_700000_chains():
    torch.cuda.set_device(0)
    B, M = 700000, 3
    pos = np.random.default_rng(0).standard_normal((B, 3, M)) + 4.0 * np.arange(M)
    with Context(pos, seed=2, precision="fp64", stream=torch.cuda.current_stream()) as ctx:
        dst = torch.full((B, 3, M), np.nan, dtype=torch.float64, device="cuda")
        ctx.positions_to_device(dst.data_ptr())
        got = dst.cpu().numpy()
    scale = np.abs(pos).sum(axis=2, keepdims=True)
    assert np.all(np.abs(got - pos) <= 2 * (M + 8) * 2.0 ** -53 * np.sqrt(3.0) * scale)
