"""The kernels' special paths against their general ones, bit for bit, at the
sizes where a tile, a band or a chunk ends.  A tensor that starts one element
into its allocation is misaligned for vector accesses, which sends the same task
down the general path."""
import numpy as np
import pytest
import torch

from paper_2007_01277_amd import hfuse as H
from paper_2007_01277_amd import inputs
from tests import gpu_cases as G

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    assert torch.cuda.is_available()
    H.hf_init()
    yield


def _out(shape, offset, dtype=torch.float32):
    n = int(np.prod(shape))
    return torch.full((n + offset,), 7, dtype=dtype, device="cuda")[offset:].view(shape)


def _run(make, block=256, grid=0):
    task, outs = make
    H.hf_run_solo(task, block, grid)
    torch.cuda.synchronize()
    return outs


@pytest.mark.parametrize("h", [1, 2, 3, 4, 5, 8, 9, 31])
@pytest.mark.parametrize("w", [2, 30, 34, 96, 130])
def test_upsample2_bands_equal_the_general_path(h, w):
    x = G.dev(inputs.normal_image((2, 3, h, w), 7 * h + w))
    res = []
    for off in (0, 1):
        o = _out((2, 3, 2 * h, 2 * w), off)
        res.append(_run((H.task_upsample(x, o, 2), o)))
    assert torch.equal(res[0], res[1])
    for block, grid in ((256, 1), (512, 3), (1024, 0)):  # resident wavefronts that take several units
        o = _out((2, 3, 2 * h, 2 * w), 0)
        assert torch.equal(_run((H.task_upsample(x, o, 2), o), block, grid), res[0]), (block, grid)


@pytest.mark.parametrize("n", [1, 15, 16, 4096, 70_001, 3_000_017])
@pytest.mark.parametrize("own", [False, True])
def test_histogram_merge_at_every_grid(n, own):
    """One workgroup (nothing to merge), up to and past the number of
    accumulators and of workgroups per accumulator, in the library's scratch
    and in the caller's (one accumulator)."""
    c = G.hist_case(n, seed=n)
    if not own:
        scr = torch.zeros(H.hf_scratch_bytes(c.task) // 4, dtype=torch.int32, device="cuda")
        c.task.scratch = scr.data_ptr()
    for grid in (0, 1, 2, 15, 16, 17, 64, 65, 100, 700):
        for block in (256, 1024):
            G.run_and_check(lambda: H.hf_run_solo(c.task, block, grid), [c])
    if not own:
        assert int(scr.abs().sum()) == 0


@pytest.mark.parametrize("cfg", [(1, 256, 0), (4, 512, 64), (15, 1024, 0)])
def test_fused_bodies_with_grids_of_their_own(cfg):
    """A kernel that streams (a workgroup per unit) next to one that runs
    resident, both ways round and with either of them the larger."""
    cases = [G.up_case((4, 32, 33, 64), 2, 1), G.pool_case((2, 16, 64, 128), seed=2), G.hist_case(200_003, seed=3),
             G.bn_case((2, 8, 20, 20), seed=4), G.mix_case(1 << 20, 3, seed=5, sample=512)]
    for ca in cases:
        for cb in cases:
            if ca is not cb:
                pr = H.make_pair(ca.task, cb.task)
                G.run_and_check(lambda: H.hf_run_fused_cfg(pr, H.hf_config(*cfg, 0)), [ca, cb])


@pytest.mark.parametrize("n", [4, 63, 64, 255, 256, 257, 1023, 1025, 5000])
@pytest.mark.parametrize("rounds", [0, 1, 2, 7])
def test_int_mix_steps_of_one_to_four_vectors(n, rounds):
    """One lane takes one, two, three or four vectors per step (few workgroups
    make the steps full), with and without a scalar tail."""
    c = G.mix_case(n, rounds, seed=n + rounds)
    for grid in (1, 2, 0):
        G.run_and_check(lambda: H.hf_run_solo(c.task, 256, grid), [c])


# kernel, stride, pad: every block width and stride class of im2col's general path
@pytest.mark.parametrize("k,s,p", [((1, 1), 1, 0), ((1, 1), 2, 0), ((2, 3), 1, 1), ((3, 3), 2, 1), ((4, 4), 1, 2),
                                   ((4, 4), 4, 0), ((5, 5), 1, 2), ((7, 7), 2, 3), ((3, 9), 2, 4), ((11, 17), 3, 8),
                                   ((2, 2), 5, 1)])
@pytest.mark.parametrize("shape", [(1, 1, 11, 16), (2, 3, 12, 17), (3, 1, 19, 28), (1, 2, 40, 65)])
def test_im2col_general_path(k, s, p, shape):
    for off in (0, 1):  # one element into its allocation: neither input nor output vector-aligned
        c = G.im2col_case(shape, k, s, p, seed=sum(shape) + off)
        if off:
            x, o = G.dev(inputs.normal_image(shape, sum(shape) + off), 1), c.bufs["outs"][0]
            o2 = _out(o.shape, 1)
            c.bufs["outs"] = [o2]
            c.bufs["in"] = x
            c.task = H.task_im2col(x, o2, k[0], k[1], s, p)
        for block, grid in ((256, 0), (1024, 0), (256, 1)):
            G.run_and_check(lambda: H.hf_run_solo(c.task, block, grid), [c])


def _coord32(o, s, length):
    """The kernel's source coordinate of outputs o, step by step in float32."""
    f = np.float32
    t = np.maximum((o.astype(f) + f(0.5)) * (f(1.0) / f(s)) - f(0.5), f(0.0))
    a = np.minimum(t.astype(np.uint32), length - 1).astype(np.int64)
    return a, np.minimum(a + 1, length - 1), t - a.astype(f)


def _upsample32(x, s):
    """The pointwise definition in float32, rounding after every operation."""
    n, c, h, w = x.shape
    y0, y1, ly = _coord32(np.arange(h * s), s, h)
    x0, x1, lx = _coord32(np.arange(w * s), s, w)

    def lerp(a, b, l):
        return a + l * (b - a)

    top = lerp(x[:, :, y0][..., x0], x[:, :, y0][..., x1], lx)
    bot = lerp(x[:, :, y1][..., x0], x[:, :, y1][..., x1], lx)
    return lerp(top, bot, ly[:, None])


@pytest.mark.parametrize("s", [1, 2, 3, 4, 5, 7, 8, 16])
@pytest.mark.parametrize("shape", [(1, 1, 1, 1), (2, 3, 5, 4), (1, 2, 9, 33), (3, 1, 2, 68), (1, 1, 65, 65)])
def test_upsample_by_places_has_the_pointwise_bits(s, shape):
    xh = inputs.normal_image(shape, 10 * s + shape[3])
    x = G.dev(xh)
    want = _upsample32(xh, s)
    for off in (0, 1):
        for block, grid in ((256, 0), (512, 1)):
            o = _out((shape[0], shape[1], shape[2] * s, shape[3] * s), off)
            got = _run((H.task_upsample(x, o, s), o), block, grid).cpu().numpy()
            assert np.array_equal(got, want), (off, block, grid)


@pytest.mark.parametrize("k,s", [((2, 2), 2), ((2, 2), 1), ((3, 3), 2), ((3, 3), 3)])
@pytest.mark.parametrize("shape", [(1, 1, 3, 3), (2, 3, 7, 9), (1, 2, 33, 129), (4, 5, 6, 64)])
@pytest.mark.parametrize("special", [False, True])
def test_maxpool_without_padding(k, s, shape, special):
    g = inputs.rng(shape[3] + s)
    x = np.round(g.standard_normal(shape)).astype(np.float32)  # ties
    if special:
        x[g.random(shape) < 0.1] = np.nan
        x[g.random(shape) < 0.1] = -np.inf
    for off in (0, 1):
        c = G.pool_case(shape, k, s, 0, offset=off, x=x)
        for block in (256, 1024):
            G.run_and_check(lambda: H.hf_run_solo(c.task, block), [c])


@pytest.mark.parametrize("hw", [1, 255, 256, 257, 512, 513, 700, 2048, 2049])
def test_bn_whole_channels_equal_cut_ones(hw):
    """256 channels of up to eight units (1024 elements each) are handed out whole,
    16 channels of more than two are cut: the same bits, at every grid."""
    x = G.dev(inputs.bn_input((4, 256, 1, hw), hw))

    def stats(xs, block, grid):
        o = [_out((xs.shape[1],), 0) for _ in range(2)]
        return _run((H.task_bn_stats(xs, *o), o), block, grid)

    parts = [stats(x[:, c:c + 16].contiguous(), 256, 0) for c in range(0, 256, 16)]
    want = [torch.cat(p) for p in zip(*parts)]
    for block, grid in ((256, 0), (512, 0), (1024, 0), (256, 1), (256, 3), (1024, 300)):
        got = stats(x, block, grid)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), (block, grid)


@pytest.mark.parametrize("shape", [(2, 1, 300, 301), (3, 16, 64, 64), (1, 2048, 97, 96), (1, 2049, 96, 97)])
def test_bn_counters_in_lines_and_packed(shape):
    """A line for each counter (the library's scratch, up to 2048 channels) and
    packed counters (the caller's) count the same arrivals and end at zero."""
    x = inputs.cuda_normal(shape, sum(shape))
    res = []
    for own in (True, False):
        o = [_out((shape[1],), 0) for _ in range(2)]
        t = H.task_bn_stats(x, *o)
        if not own:
            scr = torch.zeros(H.hf_scratch_bytes(t) // 4, dtype=torch.int32, device="cuda")
            t.scratch = scr.data_ptr()
        for block, grid in ((256, 0), (1024, 0), (512, 7)):  # each finds the scratch as the last left it
            for b in o:
                b.fill_(7)
            _run((t, o), block, grid)
            res.append([b.clone() for b in o])
        if not own:
            assert int(scr.abs().sum()) == 0
    for r in res[1:]:
        assert torch.equal(r[0], res[0][0]) and torch.equal(r[1], res[0][1])


@pytest.mark.parametrize("n", [1, 31, 32, 33, 63, 64, 65, 127, 129, 300, 1025])
def test_ethash_one_and_two_passes_per_wavefront(n):
    c = G.hash_case(H.HF_ETHASH, n, seed=n)
    for block, grid in ((256, 1), (256, 2), (512, 0), (1024, 1), (1024, 0)):
        G.run_and_check(lambda: H.hf_run_solo(c.task, block, grid), [c])


@pytest.mark.parametrize("n,c,h", [(1, 3, 20), (2, 64, 57), (12, 64, 113)])
def test_maxpool_general_path_units_per_wavefront(n, c, h):
    """Fewer units than wavefronts on the chip, some more, and several each."""
    x = (n, c, h, h)
    cs = G.pool_case(x, (3, 3), 1, 1, seed=h)
    for block in (256, 1024):
        G.run_and_check(lambda: H.hf_run_solo(cs.task, block, 0), [cs])


@pytest.mark.parametrize("kind", [H.HF_SHA256D, H.HF_BLAKE2B])
@pytest.mark.parametrize("n", [1, 65, 4097, 65536, 65537, 140_001])
def test_hashes_spread_and_shared_midstate(kind, n):
    """One piece per wavefront (spread over the workgroups) and several, the
    midstate per wavefront (up to 65536 nonces) and per workgroup or interval."""
    c = G.hash_case(kind, n, seed=n, sample=1500)
    for block, grid in ((256, 0), (1024, 0), (512, 3), (1024, 300)):
        G.run_and_check(lambda: H.hf_run_solo(c.task, block, grid), [c])
    m = G.mix_case(5000, 3, seed=n)
    for cfg in ((1, 256, 0), (12, 1024, 64)):  # an interval of one and of several wavefronts
        for pr in (H.make_pair(c.task, m.task), H.make_pair(m.task, c.task)):
            G.run_and_check(lambda: H.hf_run_fused_cfg(pr, H.hf_config(*cfg, 0)), [c, m])
