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
