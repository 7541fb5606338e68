"""FP64 trajectories do not depend on how chains are batched: the first chains
of a large ensemble (tiles of 16 chains), of a middling one (tiles of 5 with
streamed tables) and of a small one (tiles of 5, noise wavefronts and held
tables where the chains are short) hold the same bits, at lengths with every
16-chain shape."""
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


@pytest.mark.parametrize("kw", [{}, {"gamma_dot": 1e-4}, {"gamma_dot": 1e-4, "nonlinear": False}],
                         ids=["rest", "shear", "linear"])
@pytest.mark.parametrize("B,M", [(8190, 30), (6300, 64), (3700, 96), (4090, 128), (2570, 131),
                                 (2570, 256)])
def test_same_bits_in_every_tile(B, M, kw):
    pos = inputs.straight_chains(B, M, B_FAC, seed=M, random_orientation=True)
    out = []
    for n in (B, 1300, 22):
        with Context(pos[:n], seed=7, precision="fp64") as ctx:
            ctx.set_params([M], [20.0], T_star=TS, nu=NU, **kw)
            ctx.step_modes(13)
            out.append(ctx.modes()[:22])
    assert np.all(np.isfinite(out[0]))
    assert np.array_equal(out[0], out[2])
    assert np.array_equal(out[1], out[2])
