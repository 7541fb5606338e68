"""The observation kernel over length buckets of several row-tile counts in one
launch, and over more buckets than one launch takes: each chain against the
same chain observed alone in a context of one length (whose launch has the
row-tile count of its own), from the same uploaded state: the same arithmetic
per chain in both kernels, so the same bits."""
import numpy as np
import pytest
import torch

from paper_1411_3487_amd import Context, _lib, inputs, NU_DSDNA as NU, T_STAR_DSDNA as TS

pytestmark = pytest.mark.gpu

B_FAC = 1.0 / (1.0 - 2.0 * NU)


@pytest.fixture(scope="module", autouse=True)
def _device():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    torch.cuda.set_device(0)
    yield
    torch.cuda.synchronize()


def observed(pos, lens, prec):
    with Context(pos, seed=5, precision=prec) as ctx:
        ctx.set_params(lens, [10.0] * len(lens), T_star=TS, nu=NU, sample_every=1)
        return ctx.chain_observables(), ctx.observables(_lib.DM_OBS_MODES)


@pytest.mark.parametrize("prec", ["fp32", "bf16x3"])
@pytest.mark.parametrize("lens", [[4, 512], [2, 66, 130, 258, 322, 386, 450],
                                  [2, 4, 34, 64, 66, 96, 128, 130, 192, 256, 258, 384, 510, 512]])
def test_mixed_lengths_equal_single_lengths(lens, prec):
    counts = [1 + (7 * i) % 11 for i in range(len(lens))]
    parts = [inputs.straight_chains(n, M, B_FAC, seed=M, random_orientation=True)
             for n, M in zip(counts, lens)]
    parts = [p + 0.3 * np.random.default_rng(M).standard_normal(p.shape)
             for p, M in zip(parts, lens)]
    got, m2 = observed([c for p in parts for c in p], lens, prec)
    at = m = 0
    for p, n, M in zip(parts, counts, lens):
        want, wm2 = observed(p, [M], prec)
        assert np.array_equal(got[at:at + n], want), M
        assert np.array_equal(m2[m:m + n * M], wm2), M
        at, m = at + n, m + n * M
