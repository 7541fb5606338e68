"""Tiles of 16 chains (split-BF16): the same bits as the 5-chain shapes, at
chain counts around a tile and lengths at the ends of both row-tile counts,
with shear, free modes, and sampled blocks replayed as graphs."""
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


def run(pos, M, mode, steps=(7, 5), **kw):
    """Modes, accumulators and the shape after two calls of step_modes."""
    with Context(pos, seed=3, precision="bf16x3") as ctx:
        ctx.set_params([M], [50.0], T_star=TS, nu=NU, table_mode=mode, **kw)
        for n in steps:
            ctx.step_modes(n)
        return ctx.modes(), ctx.accumulators()[0], int(ctx.tiling()[0]["split"])


@pytest.mark.parametrize("M", [130, 192, 194, 256])
@pytest.mark.parametrize("B,kw", [
    (2561, {}), (2576, {"gamma_dot": 1e-5}), (2575, {"nonlinear": False, "gamma_dot": 1e-5}),
    (2580, {"sample_every": 3, "use_graphs": True})])
def test_same_bits_as_five_chain_tiles(M, B, kw):
    pos = inputs.straight_chains(B, M, B_FAC, seed=M, random_orientation=True)
    got, acc, split = run(pos, M, "auto", **kw)
    assert split == 3, "the shortest schedule on 256 compute units"
    want, wacc, split = run(pos, M, "resident", **kw)
    assert split == 0
    assert np.array_equal(got, want)
    for k in acc:
        assert np.array_equal(acc[k], wacc[k]), k


def test_two_lengths_share_the_launch():
    beads = np.repeat(np.array([160, 256], dtype=np.int32), [2000, 1900])
    beads = np.random.default_rng(0).permutation(beads)
    chains = inputs.mixed_chains(beads, B_FAC, seed=3)
    out = []
    for mode in ("auto", "resident"):
        with Context(chains, seed=4, precision="bf16x3") as ctx:
            ctx.set_params([160, 256], [50.0, 100.0], T_star=TS, nu=NU, table_mode=mode)
            ctx.step_modes(11)
            out.append(ctx.modes())
            assert all(int(t["split"]) == (3 if mode == "auto" else 0) for t in ctx.tiling())
    assert all(np.array_equal(a, b) for a, b in zip(*out))
