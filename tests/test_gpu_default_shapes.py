"""The shapes that dm_set_params picks untimed, on the 256 compute units of an
MI355X: where a launch fills the chip once with resident tables and takes
several rounds of small-launch tiles, the coupled mode tiles decide."""
import pytest
import torch

from paper_1411_3487_amd import Context, NU_DSDNA as NU, T_STAR_DSDNA as TS

pytestmark = pytest.mark.gpu

RESIDENT, TILE16, SMALL1, SMALL2 = (1, 4, 0), (0, 1, 3), (0, 1, 4), (0, 2, 4)


# (measured, microseconds per 40 steps: small-launch tiles against resident
# tables, 3840 x 66: 160 and 149; 17920 x 128 at dtau = 100: 605 and 561;
# FP32 7680 x 66 at dtau = 100: 422 and 406, at dtau = 10: 423 and 446)
@pytest.mark.parametrize("prec,B,M,dtau,shape", [
    ("bf16x3", 2561, 66, 10.0, RESIDENT), ("bf16x3", 3840, 66, 10.0, RESIDENT),
    ("bf16x3", 3840, 128, 100.0, RESIDENT), ("bf16x3", 17920, 128, 100.0, RESIDENT),
    ("bf16x3", 5120, 256, 200.0, RESIDENT), ("fp32", 7680, 66, 100.0, RESIDENT),
    ("fp32", 14080, 194, 100.0, RESIDENT),
    ("fp32", 7680, 66, 10.0, SMALL2), ("fp32", 5121, 66, 100.0, SMALL1),
    ("bf16x3", 5120, 256, 10.0, SMALL2), ("bf16x3", 2560, 64, 10.0, SMALL2),
    ("bf16x3", 1280, 128, 10.0, SMALL1), ("bf16x3", 4096, 256, 100.0, TILE16),
    ("bf16x3", 20480, 192, 10.0, TILE16), ("bf16x3", 1024, 512, 100.0, SMALL1)])
def test_untimed_shape(prec, B, M, dtau, shape):
    torch.cuda.set_device(0)
    assert torch.cuda.get_device_properties(0).multi_processor_count == 256
    with Context(None, seed=1, precision=prec, beads=[M] * B) as ctx:
        ctx.set_params([M], [dtau], T_star=TS, nu=NU)
        t = ctx.tiling()[0]
        assert (int(t["resident"]), int(t["tpw"]), int(t["split"])) == shape
        ctx.step_modes(2)
