"""A chain without a finite state leaves the other chains of its FP64 tile as
they are, under shear too: the same bits as beside a healthy chain.  One chain
has all beads at one point (bonds of length 0, no force direction), another
holds NaN, its centre of mass included."""
import numpy as np
import pytest
import torch

from paper_1411_3487_amd import Context, inputs, NU_DSDNA as NU, T_STAR_DSDNA as TS

pytestmark = pytest.mark.gpu

B_FAC = 1.0 / (1.0 - 2.0 * NU)


@pytest.fixture(scope="module", autouse=True)
def _device():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    torch.cuda.set_device(0)
    yield
    torch.cuda.synchronize()


# 5-chain tiles: noise wavefronts at two lengths, one and two row tiles a
# wavefront; without noise wavefronts; tiles of 16 chains
@pytest.mark.parametrize("B,M", [(5, 33), (10, 128), (5, 200), (5, 300), (1300, 65), (2570, 140)])
@pytest.mark.parametrize("gdot", [0.0, 1e-3])
@pytest.mark.parametrize("fill", [0.0, np.nan], ids=["point", "nan"])
def test_neighbours_of_a_bad_chain(B, M, gdot, fill):
    pos = inputs.straight_chains(B, M, B_FAC, seed=M, random_orientation=True)
    bad = pos.copy()
    bad[2] = bad[B - 1] = fill
    out = []
    for p in (pos, bad):
        with Context(p, seed=7, precision="fp64") as ctx:
            ctx.set_params([M], [20.0], T_star=TS, nu=NU, gamma_dot=gdot)
            ctx.step_modes(5)
            out.append(ctx.modes())
    others = np.delete(np.arange(B), [2, B - 1])
    assert np.all(np.isfinite(out[0]))
    assert not np.isfinite(out[1][2]).all() and not np.isfinite(out[1][B - 1]).all()
    assert np.array_equal(out[0][others], out[1][others])
