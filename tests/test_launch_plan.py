"""The default launches the host code decides on, without a GPU."""
import pytest

from paper_2007_01277_amd import hfuse as H
from tests import launch_plan as P

# narrow planes: a unit of the row paths covers few outputs, so a few hundred
# megabytes make millions of units
NARROW = [P.task(H.HF_UPSAMPLE, (65536, 64, 4, 4), (2,)), P.task(H.HF_UPSAMPLE, (1 << 20, 64, 1, 2), (2,)),
          P.task(H.HF_UPSAMPLE, (1 << 21, 100, 3, 3), (1,)), P.task(H.HF_UPSAMPLE, (1 << 17, 64, 3, 5), (3,), misalign=4),
          P.task(H.HF_MAXPOOL, (65536, 64, 8, 8), (3, 3, 2, 1)), P.task(H.HF_MAXPOOL, (1 << 20, 64, 3, 8), (3, 3, 2, 1)),
          P.task(H.HF_MAXPOOL, (1 << 20, 200, 3, 3), (3, 3, 1, 1), idx=True)]


@pytest.mark.parametrize("t", NARROW, ids=lambda t: f"{H.KIND_NAMES[t.kind]}-{t.n}x{t.c}x{t.h}x{t.w}")
@pytest.mark.parametrize("block,per_cu", [(256, 8), (512, 4), (1024, 2), (1024, 1)])
def test_a_launch_stays_below_2_to_the_32_lanes(t, block, per_cu):
    """hipLaunchKernel refuses more; in a fused launch the whole block counts, also
    where the body has one wavefront of it."""
    for waves in (1, 2, block // 64):
        g = P.wgs(t, waves, block, 256 * per_cu)
        assert 1 <= g and g * block < 1 << 32, (waves, g)
        assert g <= P.useful(t, waves)
