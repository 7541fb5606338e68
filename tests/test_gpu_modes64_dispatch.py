"""FP64 launches of sizes that few-chain tests do not reach: 5-chain tiles
without noise wavefronts at every width, ensembles whose lengths take several
launches (16-chain tiles beside 5-chain tiles of several widths), and the
allocation-free step of chains beyond the persistent stepper.  Sampled chains
against the oracle, 1e-11 of the contour length: E_p, formed by another
subtraction there, differs by 4 * 2^-53 dtau per step (9e-13 after 20 steps of
dtau = 100), rounding adds a few 1e-14."""
import numpy as np
import pytest
import torch

import oracle
from paper_1411_3487_amd import Context, inputs, _lib, NU_DSDNA as NU, T_STAR_DSDNA as TS

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


def check(got, pos, ids, dtau, seed, gdot=0.0, nonlinear=True):
    M = pos.shape[-1]
    R = oracle.step_modes(oracle.modes_from_positions(pos), NU, TS, dtau, STEPS, seed=seed,
                          chain_ids=ids, gamma_dot=gdot, nonlinear=nonlinear)
    err = np.abs(got - oracle.positions_from_modes(R)).max() / ((M - 1) * B_FAC)
    assert err < TOL, (M, err)


# more than one 5-chain tile per compute unit of 256, too few chains for tiles
# of 16; odd lengths whose last mode lies beyond their tiles (65, 129, 257)
@pytest.mark.parametrize("B,M,gdot,nonlinear", [
    (1281, 2, 0.0, True), (1283, 31, 1e-4, True), (2000, 33, 0.0, True), (2000, 64, 1e-4, True),
    (2000, 65, 1e-4, True), (2001, 65, 1e-4, False), (2500, 97, 0.0, True),
    (2500, 128, 1e-4, True), (2500, 129, 1e-4, True), (1400, 200, 1e-4, True),
    (1400, 257, 1e-4, True), (1300, 513, 1e-4, True)])
def test_five_chain_tiles_without_noise_wavefronts(B, M, gdot, nonlinear):
    pos = inputs.straight_chains(B, M, B_FAC, seed=M, random_orientation=True)
    with Context(pos, seed=5, precision="fp64") as ctx:
        ctx.set_params([M], [20.0], T_star=TS, nu=NU, gamma_dot=gdot, nonlinear=nonlinear)
        ctx.step_modes(STEPS)
        got = ctx.positions()
    ids = np.array([0, 4, 5, B // 2, B - 6, B - 1])
    check(got[ids], pos[ids], ids, 20.0, 5, gdot, nonlinear)


# 2600 x 256 on 16-chain tiles, and 541 (181) 5-chain tiles: four launches by
# width, with odd lengths in two of them (one launch of the widest)
@pytest.mark.parametrize("counts", [
    {256: 2600, 64: 700, 65: 400, 100: 505, 130: 600, 257: 200, 300: 300},
    {256: 2600, 33: 300, 128: 305, 200: 300}])
def test_lengths_in_several_launches(counts):
    lens = sorted(counts)
    beads = np.repeat(np.array(lens, dtype=np.int32), [counts[m] for m in lens])
    beads = np.random.default_rng(1).permutation(beads)
    chains = inputs.mixed_chains(beads, B_FAC, seed=3)
    out = []
    for graphs in (False, True):  # (20 steps: two replayed blocks)
        with Context(chains, seed=4, precision="fp64") as ctx:
            ctx.set_params(lens, [20.0] * len(lens), T_star=TS, nu=NU, gamma_dot=1e-4,
                           sample_every=10, use_graphs=graphs)
            ctx.step_modes(STEPS)
            out.append((ctx.positions(), ctx.accumulators()))
    got = out[0][0]
    assert all(np.array_equal(a, b) for a, b in zip(got, out[1][0]))
    for a, b in zip(out[0][1], out[1][1]):
        assert a["n_samples"] == b["n_samples"] == 2
        assert np.array_equal(a["modes"], b["modes"])
    for M in lens:
        ids = np.flatnonzero(beads == M)[[0, 5, 17, -17, -1]]
        check(np.stack([got[c] for c in ids]), np.stack([chains[c] for c in ids]), ids, 20.0, 4,
              1e-4)


@pytest.mark.parametrize("B,M,gdot,nonlinear", [(5, 514, 1e-4, True), (7, 528, 0.0, True),
                                                (3, 1025, 1e-4, False)])
def test_allocation_free_step_beyond_the_persistent_stepper(B, M, gdot, nonlinear):
    pos = inputs.straight_chains(B, M, B_FAC, seed=M, random_orientation=True)
    with Context(pos, seed=6, precision="fp64") as ctx:
        ctx.set_params([M], [100.0], T_star=TS, nu=NU, gamma_dot=gdot, nonlinear=nonlinear)
        R0 = ctx.modes()
    # chains 2 .. of the ensemble, in two calls
    R = torch.tensor(R0[2:], dtype=torch.float64, device="cuda").contiguous()
    lib = _lib.load()
    stream = torch.cuda.current_stream()
    for step0, n in ((0, 8), (8, STEPS - 8)):
        rc = lib.dm_step_modes_f64_static(R.data_ptr(), B - 2, M, TS, NU, 100.0, gdot,
                                          1 if nonlinear else 0, 6, 2, step0, n,
                                          stream.cuda_stream)
        assert rc == _lib.DM_OK, lib.dm_last_error(None).decode()
    torch.cuda.synchronize()
    got = oracle.positions_from_modes(R.cpu().numpy())
    check(got, pos[2:], np.arange(2, B), 100.0, 6, gdot, nonlinear)


@pytest.mark.parametrize("B,M,mode,split", [(1024, 128, "split", 1), (1024, 512, "split", 1),
                                            (1024, 256, "split8", 2), (1024, 512, "split8", 2)])
def test_split_tiles_of_reduced_precision_at_batched_sizes(B, M, mode, split):
    """The forms that only table_mode picks: the bits of the default shape."""
    pos = inputs.straight_chains(B, M, B_FAC, seed=1, random_orientation=True)
    out = []
    for m in (mode, "auto"):
        with Context(pos, seed=1, precision="bf16x3") as c:
            c.set_params([M], [100.0], T_star=TS, nu=NU, table_mode=m)
            assert int(c.tiling()[0]["split"]) == (split if m == mode else 4)
            c.step_modes(5)
            out.append(c.modes())
    assert np.array_equal(out[0], out[1])
