"""The sums over the chains in the accumulators (dm_observables, DM_OBS_ACCUM)
against the per-chain observables of the same sample, at chain counts around
the summing kernel's slices of 128 chains and 4 loads per thread, and for
ensembles of several lengths.  Both sides add the same FP64 numbers, so they
agree to n 2^-53 of the sum of magnitudes.
"""
import numpy as np
import pytest
import torch

from paper_1411_3487_amd import Context, inputs, DM_OBS_MODES, NU_DSDNA as NU, T_STAR_DSDNA as TS

pytestmark = pytest.mark.gpu

B_FAC = 1.0 / (1.0 - 2.0 * NU)


@pytest.fixture(scope="module", autouse=True)
def _device():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    torch.cuda.set_device(0)
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("counts", [{6: 1}, {6: 127}, {6: 128}, {7: 129}, {6: 511}, {6: 512},
                                    {9: 513}, {6: 1100}, {6: 130, 7: 3, 20: 600}])
def test_accumulators_are_the_sums_over_the_chains(counts):
    beads = np.concatenate([np.full(n, m, dtype=np.int32) for m, n in counts.items()])
    beads = np.random.default_rng(4).permutation(beads)
    chains = inputs.mixed_chains(beads, B_FAC, seed=5)
    lens = sorted(counts)
    with Context(chains, seed=3, precision="fp64") as ctx:
        ctx.set_params(lens, [10.0] * len(lens), T_star=TS, nu=NU, sample_every=4)
        ctx.step_modes(4)
        obs = ctx.chain_observables()
        m2 = ctx.observables(DM_OBS_MODES)
        acc = ctx.accumulators()
    off = np.concatenate([[0], np.cumsum(beads)])
    assert [a["M"] for a in acc] == lens
    for a in acc:
        M, n = int(a["M"]), counts[int(a["M"])]
        rows = np.flatnonzero(beads == M)
        assert a["n_chains"] == n and a["n_samples"] == 1
        tol = n * 2.0 ** -53
        for key, col in (("bond", 0), ("L2", 1), ("xspan", 14), ("bond2", 15)):
            want = obs[rows, col].sum()
            assert abs(a[key] - want) <= tol * np.abs(obs[rows, col]).sum(), key
        want = np.stack([m2[off[c]:off[c] + M] for c in rows]).sum(axis=0)
        assert np.all(np.abs(a["modes"] - want) <= tol * want)
