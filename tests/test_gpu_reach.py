"""Paths that only larger inputs reach: the shared SHA-256 midstate inside batches,
members of the cost model trained in chunks, and fused launches with more
workgroups than the chip holds at once."""
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


@pytest.fixture(scope="module")
def hashes():
    """Nonce counts around the limit above which an interval shares its midstate,
    each with a header of its own, and kinds that use the intervals' LDS."""
    cs = [G.hash_case(H.HF_SHA256D, n, seed=n, sample=300) for n in (65536, 65537, 70_001, 140_001)]
    return [cs[0], cs[2], G.hist_case(300_003, seed=1), cs[1], G.mix_case(4099, 3, seed=2), cs[3],
            G.hash_case(H.HF_SHA256D, 100, seed=9)]


@pytest.mark.parametrize("sched", [(512, 0, 0), (1024, 0, 128), (512, 2, 64), (512, 4, 128), (1024, 8, 64), (256, 1, 64)])
def test_batches_share_midstates_by_interval(hashes, sched):
    """Static members (up to three of a group hash) and worker intervals of one to
    eight wavefronts, several items of each task, eager and replayed."""
    groups = [0, 0, 0, 1, 1, 1, 1]
    block, iw, kb = sched
    s = H.hf_batch_schedule(block, iw, kb, 0)
    even = None if iw else [3, 2, 3, 2, 2, 3, 1] if block == 512 else [5, 5, 6, 4, 4, 6, 2]
    b = H.Batch([c.task for c in hashes], groups, even, block, schedule=s)
    assert b.info()["items"] > 2 * len(hashes)
    for use_graph in (False, True, True, True):
        G.run_and_check(lambda: b.run(use_graph), hashes)
        H.hf_run_solo(hashes[4].task, 256)  # eager work between replays
        torch.cuda.synchronize()
    b.close()


def test_members_in_chunks_train_as_they_do_alone():
    """16 members over 12000 samples exceed the workspace for all at once: chunks of
    14 and two."""
    n, members, d = 12000, 16, H.MLP_FEATURES
    g = inputs.rng(77)
    x = g.standard_normal((n, d)).astype(np.float32)
    y = (np.sin(x[:, 0]) + 0.5 * x[:, 1] * x[:, 2]).astype(np.float32)
    H.hf_mlp_init(d, 60, members=members)
    loss = H.hf_mlp_train(x, y, epochs=2, lr=1e-3)
    both = H.hf_mlp_predict(x[:40]).astype(np.float64)
    first = H.hf_mlp_get_params()
    alone, losses = [], []
    for k in range(members):
        H.hf_mlp_init(d, 60 + k)
        losses.append(H.hf_mlp_train(x, y, epochs=2, lr=1e-3))
        alone.append(H.hf_mlp_predict(x[:40]).astype(np.float64))
        if k == 0:
            assert np.array_equal(H.hf_mlp_get_params(), first)
    # float32 values whose mean is rounded once more
    assert abs(loss - np.mean(losses)) <= 2.0 ** -23 * abs(loss)
    assert np.all(np.abs(both - np.mean(alone, axis=0)) <= 4 * 2.0 ** -24 * np.abs(alone).max(axis=0) + 2.0 ** -22)


@pytest.mark.parametrize("cfg", [(1, 256, 64), (7, 512, 0), (1, 512, 64), (2, 1024, 64)])
def test_fused_streaming_past_the_resident_workgroups(cfg):
    """Upsample (rows and places) and maxpool (rows and general), each with several
    times the units the resident workgroups take, next to kinds that run resident,
    against the solo kernels on a small grid."""
    def up(shape, s, seed):
        x = inputs.cuda_normal(shape, seed)
        o = torch.empty((*shape[:2], shape[2] * s, shape[3] * s), device="cuda")
        return H.task_upsample(x, o, s), [x], [o]

    def pool(shape, k, s, p, seed):
        x = inputs.cuda_normal(shape, seed)
        osh = H.maxpool_out_shape(shape, k, k, s, p)
        o, i = torch.empty(osh, device="cuda"), torch.empty(osh, dtype=torch.int32, device="cuda")
        return H.task_maxpool(x, o, i, k, k, s, p), [x], [o, i]

    def hist(n, seed):
        x = inputs.cuda_zipf_u8(n, seed)
        o = torch.empty(256, dtype=torch.int32, device="cuda")
        return H.task_lds_hist(x, o), [x], [o]

    stream = [up((64, 64, 64, 64), 2, 1), up((40, 64, 33, 65), 3, 2), pool((64, 64, 112, 112), 3, 2, 1, 3),
              pool((64, 64, 111, 111), 2, 2, 0, 4)]
    want = []
    for t, _, outs in stream:
        H.hf_run_solo(t, 256, 64)
        torch.cuda.synchronize()
        want.append([o.clone() for o in outs])
    th, _, oh = hist(5_000_011, 5)
    H.hf_run_solo(th, 256, 64)
    torch.cuda.synchronize()
    wh = oh[0].clone()
    for i, (ta, _, oa) in enumerate(stream):
        j = (i + 1) % len(stream)
        for tb, ob, wb in ((th, oh, [wh]), (stream[j][0], stream[j][2], want[j])):
            for a, b in ((ta, tb), (tb, ta)):
                for o in oa + ob:
                    o.fill_(7)
                H.hf_run_fused_cfg(H.make_pair(a, b), H.hf_config(*cfg, 0))
                torch.cuda.synchronize()
                assert all(torch.equal(o, w) for o, w in zip(oa, want[i])), (i, cfg)
                assert all(torch.equal(o, w) for o, w in zip(ob, wb)), (i, cfg)
