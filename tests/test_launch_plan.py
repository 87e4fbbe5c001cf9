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


def _extra(c, n, h, w):
    t = P.task(H.HF_BN_STATS, (n, c, h, w))
    return P.own_scratch(t) - H.hf_scratch_bytes(t)


def test_statistics_scratch_grows_by_a_line_per_channel_or_not_at_all():
    for c in (1, 16, 255, 2047, 2048):
        assert _extra(c, 64, 56, 56) == 128 * c
    for c in (2049, 65536, 131073, 174762, 200000):  # packed counters
        assert _extra(c, 1, 60, 60) == 0
    # whole channels count no arrivals
    for c, n, h, w in ((2048, 1, 7, 7), (16, 2, 32, 32), (2048, 8, 32, 32), (256, 8, 32, 32)):
        assert _extra(c, n, h, w) == 0
    assert _extra(255, 8, 32, 32) == 128 * 255


def test_a_task_that_fits_a_slot_s_mebibytes_never_grows_it():
    """Growing is impossible while a stream is captured: whatever needs no more
    whole MiB of hf_scratch_bytes than an earlier task must fit its slot."""
    tasks = [P.task(H.HF_LDS_HIST, (1 << 20,), (256,))]
    for c in (1, 100, 2047, 2048, 2049, 65537, 131073, 174762, 200000, 260000):
        for hw in (1, 32, 47, 64, 97, 1000):
            if c * hw * hw < 1 << 31:
                tasks.append(P.task(H.HF_BN_STATS, (1, c, hw, hw)))
    for a in tasks:
        slot = P.slot(P.own_scratch(a))
        mib = max(1, -(-H.hf_scratch_bytes(a) // (1 << 20))) << 20
        for b in tasks:
            if H.hf_scratch_bytes(b) <= mib:
                assert P.own_scratch(b) <= slot, (a.kind, a.c, a.h, b.kind, b.c, b.h)


@pytest.mark.parametrize("n", [1, 1000, 1 << 16, 1 << 20, 9_000_001, 1 << 26, (1 << 31) - 1])
@pytest.mark.parametrize("block,per_cu", [(256, 8), (512, 4), (1024, 2)])
def test_a_histogram_takes_four_wavefronts_per_cu(n, block, per_cu):
    """However many workgroups the launch has room for, each starts and merges."""
    t = P.task(H.HF_LDS_HIST, (n,), (256,))
    for waves in (1, 2, block // 64):
        g = P.wgs(t, waves, block, 256 * per_cu)
        assert 1 <= g <= min(P.useful(t, waves), 256 * per_cu)
        assert g <= max(256, -(-1024 // waves))
        if n >= 1 << 20:
            assert g * waves >= 1024 or g == 256 * per_cu


def test_upsample_takes_the_path_whose_lanes_the_planes_fill():
    """Rows: an even width whose chunks of 32 columns and bands of four rows keep half
    of a unit's lanes; places: rows long enough, or whole lines; else pointwise."""
    def path(h, w, s, misalign=0, planes=32):
        return P.upsample_path(P.task(H.HF_UPSAMPLE, (1, planes, h, w), (s,), misalign))

    for h, w in ((1, 2), (2, 2), (4, 4), (8, 8), (12, 12), (1, 96), (4096, 4)):
        assert path(h, w, 2) == 0, (h, w)
    for h, w in ((16, 16), (24, 24), (32, 32), (28, 28), (56, 56), (3, 96), (4, 64), (128, 128)):
        assert path(h, w, 2) == 2, (h, w)
    assert path(16, 16, 2, misalign=4) == 1  # one output column at a time
    assert path(16, 17, 2) == 1
    for s, short, full in ((3, 7, 8), (4, 5, 6), (5, 5, 6), (16, 5, 6)):
        assert path(9, short, s) == 0 and path(9, full, s) == 1, s
    assert path(9, 4, 8) == 1 and path(9, 2, 16) == 1  # whole lines
    assert path(9, 3, 8) == 0
    for s in (3, 4):  # past 2^22 the coordinates lose what the path by places assumes
        assert path((1 << 22) // s + 1, 8, s, planes=1) == 0


def test_short_upsample_units_are_taken_several_at_a_time():
    for shape, s in (((1000, 64, 6, 7), 1), ((1000, 64, 5, 5), 2), ((2000, 64, 4, 4), 2)):
        t = P.task(H.HF_UPSAMPLE, shape, (s,))
        outputs = shape[0] * shape[1] * shape[2] * shape[3] * s * s
        for block, per_cu in ((256, 8), (512, 4)):
            W = block // 64
            g = P.wgs(t, W, block, 256 * per_cu)
            assert g <= outputs / (192 * W) and g > 256 * per_cu
        assert P.wgs(t, 16, 1024, 512) <= 512  # their gaps are not covered: resident


def test_statistics_with_few_counter_lines_arrive_less_often():
    """Where arrivals share few lines of counters (the caller's scratch, or up to 64
    channels) between 8 and 16 wavefronts per CU, four units or more each past that;
    elsewhere the resident workgroups, up to 24 wavefronts per CU."""
    few = ((32, 16, 128, 128), (2, 3, 1024, 1024), (64, 64, 112, 112))
    many = ((64, 256, 56, 56), (16, 300, 33, 33), (256, 2048, 7, 7))
    for shape in few + many:
        for own in (True, False):
            t = P.task(H.HF_BN_STATS, shape, scratch=not own)
            for block, per_cu in ((256, 7), (512, 3), (1024, 1)):
                W = block // 64
                g = P.wgs(t, W, block, 256 * per_cu, own=own)
                most = min(256 * per_cu, P.useful(t, W))
                if own and shape in many:
                    assert g == min(most, 24 * 256 // W)
                else:
                    assert 1 <= g <= most and (g - 1) * W < 16 * 256
                    assert g * W >= 8 * 256 or g == most
    short = (8, 32, 16, 16)  # whole channels: no counters
    assert P.wgs(P.task(H.HF_BN_STATS, short, scratch=True), 4, 256, 1792, own=False) == \
        P.wgs(P.task(H.HF_BN_STATS, short), 4, 256, 1792)


@pytest.mark.parametrize("rows", [4099, 1 << 23])
@pytest.mark.parametrize("waves,block,per_cu", [(4, 256, 6), (1, 256, 6), (8, 512, 3), (2, 512, 2), (16, 1024, 1)])
def test_table_walks_get_wavefronts_for_one_pass_or_two(rows, waves, block, per_cu):
    res = 256 * per_cu
    for n in (0, 1, 31, 33, 1000, 8192, 20000, 49152, 50000, 65000, 98304, 98305, 130000, 131073, 150000, 262144, 1 << 24):
        t = P.task(H.HF_ETHASH, (n, 0, rows, 0))
        g = P.wgs(t, waves, block, res)
        assert 1 <= g <= res
        one = -(-n // 32)
        if one <= g * waves:  # one pass each
            assert g <= max(1, one)
        else:  # two passes, in no more iterations than the resident workgroups need
            assert g == min(res, -(-n // (64 * waves)))


def test_table_walks_load_the_simds_evenly():
    def g(n, waves, block, per_cu, rows=4099):
        return P.wgs(P.task(H.HF_ETHASH, (n, 0, rows, 0)), waves, block, 256 * per_cu)

    assert g(20000, 8, 512, 3) == 625       # a workgroup for each wavefront
    assert g(50000, 4, 256, 6) == 1024      # four per CU, not the six that fit
    assert g(50000, 8, 512, 3) == 512
    assert g(95000, 8, 512, 3) == 768       # four busy wavefronts in each of three
    assert g(130000, 4, 256, 6) == 508      # two passes where the seeds count ...
    assert g(130000, 4, 256, 6, 1 << 23) == 1024
    assert g(130000, 16, 1024, 1) == 256    # ... unless CUs would idle


def test_pooling_streams_from_four_rounds_of_workgroups_on():
    def g(n, block=256, per_cu=8):
        t = P.task(H.HF_MAXPOOL, (n, 64, 56, 56), (3, 3, 2, 1))
        return P.wgs(t, 4, block, 256 * per_cu), P.useful(t, 4)

    assert g(32)[0] == 2048 < g(32)[1]      # 1.75 rounds: resident
    assert g(128)[0] == 2048 * 7            # seven: one for every unit
    assert g(128, 1024, 1)[0] == 256
