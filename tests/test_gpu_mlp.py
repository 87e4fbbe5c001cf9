"""The learned cost model on the GPU against its fp64 reference, and the tuner
that uses it.

Tolerances: the forward pass within 1e-5 of the magnitude of its terms (the
same network evaluated on |W|, |b| and |x|, which bounds every partial sum);
gradients within 1e-4 relative to the largest gradient of their layer plus
1e-4 relative elementwise (fp32 sums over n = 2000 samples); one Adam step
within 1e-6 absolute on every parameter whose gradient is not tiny; five
steps within 5e-6 (a twentieth of one step's size at lr 1e-3, per step
1e-6) on the parameters whose gradient stays large at every step.  Where a
gradient is near zero, Adam's normalised step turns on its fp32 rounding,
so those parameters are left out of the trajectory check.
"""
import os
import tempfile

import numpy as np
import pytest
import torch

from oracle import mlp as ref
from paper_2007_01277_amd import hfuse as H
from paper_2007_01277_amd import inputs
from paper_2007_01277_amd import learned_tuner as LT

pytestmark = pytest.mark.gpu
D = H.MLP_FEATURES


@pytest.fixture(scope="module", autouse=True)
def _init():
    assert torch.cuda.is_available()
    H.hf_init()


def _data(n, seed):
    g = inputs.rng(seed)
    X = g.standard_normal((n, D)).astype(np.float32)
    y = (np.sin(X[:, 0]) + 0.5 * X[:, 1] * X[:, 2] + 0.1 * g.standard_normal(n)).astype(np.float32)
    return X, y


def _abs_forward(p, X):
    layers = ref.unpack(np.abs(p.astype(np.float64)), X.shape[1])
    h = np.abs(X.astype(np.float64))
    for W, b in layers:
        h = h @ W + b
    return h[:, 0]


def test_forward_matches_reference():
    H.hf_mlp_init(D, 1)
    p = H.hf_mlp_get_params()
    assert p.size == ref.n_params(D)
    X, _ = _data(333, 2)
    got = H.hf_mlp_predict(X).astype(np.float64)
    want, _ = ref.forward(p.astype(np.float64), X)
    assert np.all(np.abs(got - want) <= 1e-5 * _abs_forward(p, X))


def test_gradient_matches_reference():
    H.hf_mlp_init(D, 3)
    p = H.hf_mlp_get_params().astype(np.float64)
    X, y = _data(2000, 4)
    loss, g = H.hf_mlp_grad(X, y)
    rl, rg = ref.grad(p, X, y)
    assert abs(loss - rl) <= 1e-5 * rl
    o = 0
    for a, b in ref.layer_shapes(D):
        for size in (a * b, b):
            gs, rs = g[o:o + size].astype(np.float64), rg[o:o + size]
            assert np.all(np.abs(gs - rs) <= 1e-4 * np.abs(rs) + 1e-4 * np.abs(rs).max()), o
            o += size
    assert o == g.size


def _clear_of_the_kinks(p, n, d, seed):
    """n samples none of whose hidden units lies so near zero that rounding
    could flip its ReLU (for such a unit the gradient is not a function that
    float32 can be compared on)."""
    X = inputs.rng(seed).standard_normal((8 * n + 64, d)).astype(np.float32)
    _, (_, pres) = ref.forward(p, X)
    near = np.min([np.abs(z).min(axis=1) for z in pres[:-1]], axis=0)
    X = np.ascontiguousarray(X[near > 1e-4][:n])
    assert len(X) == n
    return X, np.sin(X[:, 0]).astype(np.float32)


@pytest.mark.parametrize("n,d", [(1, 1), (3, 2), (15, 3), (16, 4), (17, 5), (127, 42), (128, 63), (129, 64), (257, 65),
                                 (300, 200)])
def test_gradient_at_the_edges_of_tiles(n, d):
    """Sample counts around a workgroup's 16 samples and a tile's 128, feature
    counts around a workgroup's four rows: gradient, loss and prediction
    against float64.  A float32 chain of k terms is off by at most k * 2^-24
    of the sum of their magnitudes; four layers and the n samples bound every
    gradient by (d + 192 + n) * 2^-23 of the gradient taken with magnitudes."""
    H.hf_mlp_init(d, 21)
    p = H.hf_mlp_get_params().astype(np.float64)
    X, y = _clear_of_the_kinks(p, n, d, 100 + n)
    loss, g = H.hf_mlp_grad(X, y)
    rl, rg = ref.grad(p, X, y)
    # the same sums with every factor's magnitude (no cancellation)
    layers = ref.unpack(np.abs(p), d)
    acts = [np.abs(X.astype(np.float64))]
    for W, b in layers:
        acts.append(acts[-1] @ W + b)
    dz = (2.0 / n) * (acts[-1][:, 0] + np.abs(y))[:, None]
    mags = []
    for li in reversed(range(len(layers))):
        mags.insert(0, np.concatenate([(acts[li].T @ dz).ravel(), dz.sum(axis=0)]))
        dz = dz @ layers[li][0].T
    eps = (d + 192 + n) * 2.0 ** -23
    assert np.all(np.abs(g.astype(np.float64) - rg) <= eps * np.concatenate(mags))
    big = (acts[-1][:, 0] + np.abs(y)) ** 2
    assert abs(loss - rl) <= eps * big.mean()
    want, _ = ref.forward(p, X)
    assert np.all(np.abs(H.hf_mlp_predict(X) - want) <= eps * acts[-1][:, 0])


def test_members_train_as_they_do_alone():
    """Training side by side gives every member the bits it gets alone."""
    X, y = _data(300, 31)
    H.hf_mlp_init(D, 50, members=3)
    H.hf_mlp_train(X, y, epochs=7, lr=1e-3)
    both = H.hf_mlp_predict(X[:40]).astype(np.float64)
    alone = []
    for k in range(3):
        H.hf_mlp_init(D, 50 + k)
        H.hf_mlp_train(X, y, epochs=7, lr=1e-3)
        alone.append(H.hf_mlp_predict(X[:40]).astype(np.float64))
    # the mean of three float32 predictions, each rounded once more when alone
    assert np.all(np.abs(both - np.mean(alone, axis=0)) <= 4 * 2.0 ** -24 * np.abs(alone).max(axis=0) + 2.0 ** -22)


def test_adam_step_matches_reference():
    H.hf_mlp_init(D, 5)
    H.hf_mlp_adam_reset()
    p = H.hf_mlp_get_params().astype(np.float64)
    X, y = _data(500, 6)
    H.hf_mlp_step(X, y, 1e-3)
    p1 = H.hf_mlp_get_params().astype(np.float64)
    _, rg = ref.grad(p, X, y)
    rp, _, _ = ref.adam_step(p, rg, np.zeros_like(p), np.zeros_like(p), 1, 1e-3)
    big = np.abs(rg) > 1e-4 * np.abs(rg).max()
    assert np.all(np.abs(p1 - rp)[big] <= 1e-6 + 1e-6 * np.abs(rp[big]))
    # no step is longer than lr, up to the float32 rounding of the update
    assert np.all(np.abs(p1 - p) <= 1e-3 * (1 + 1e-5) + 2.0 ** -22 * np.abs(p))


def test_adam_trajectory_follows_reference_for_five_steps():
    H.hf_mlp_init(D, 11)
    H.hf_mlp_adam_reset()
    rp = H.hf_mlp_get_params().astype(np.float64)
    X, y = _data(500, 12)
    m, v = np.zeros_like(rp), np.zeros_like(rp)
    big = np.ones(rp.size, bool)
    for t in range(1, 6):
        H.hf_mlp_step(X, y, 1e-3)
        _, rg = ref.grad(rp, X, y)
        big &= np.abs(rg) > 1e-3 * np.abs(rg).max()
        rp, m, v = ref.adam_step(rp, rg, m, v, t, 1e-3)
    got = H.hf_mlp_get_params().astype(np.float64)
    assert big.sum() > rp.size // 4
    assert np.all(np.abs(got - rp)[big] <= 5e-6 + 1e-6 * np.abs(rp[big]))


def test_training_fits_a_smooth_target_and_roundtrips_through_a_file():
    # the target uses 3 of the 32 inputs; 4000 samples and 600 epochs generalise
    # (the float64 reference reaches a held-out correlation of 0.88 with them)
    X, y = _data(4000, 8)
    H.hf_mlp_init(D, 9)
    loss = H.hf_mlp_train(X, y, epochs=600, lr=2e-3)
    assert loss < 0.1  # standardised MSE: the target's variance is 1
    Xt, yt = _data(500, 10)
    pred = H.hf_mlp_predict(Xt)
    assert np.corrcoef(pred, yt)[0, 1] > 0.8
    with tempfile.TemporaryDirectory() as d:
        path = os.path.join(d, "m.bin")
        H.hf_mlp_save(path)
        H.hf_mlp_init(D, 123)
        H.hf_mlp_load(path)
    assert np.array_equal(H.hf_mlp_predict(Xt), pred)


def test_ensemble_predicts_the_mean_of_its_members():
    # member k of an ensemble starts from the weights a one-network model
    # seeded with seed + k has; untrained, the ensemble's prediction is the
    # mean of those models' predictions (fp32 sums of three terms)
    X, _ = _data(200, 20)
    singles = []
    for k in range(3):
        H.hf_mlp_init(D, 40 + k)
        singles.append(H.hf_mlp_predict(X).astype(np.float64))
    H.hf_mlp_init(D, 40, members=3)
    assert H.hf_mlp_members() == 3
    got = H.hf_mlp_predict(X).astype(np.float64)
    want = np.mean(singles, axis=0)
    assert np.all(np.abs(got - want) <= 1e-6 * (np.abs(want) + np.max(np.abs(singles), axis=0)))


def test_ensemble_trains_and_roundtrips_through_a_file():
    X, y = _data(2000, 21)
    H.hf_mlp_init(D, 7, members=4)
    loss = H.hf_mlp_train(X, y, epochs=300, lr=2e-3)
    assert loss < 0.2
    Xt, yt = _data(300, 22)
    pred = H.hf_mlp_predict(Xt)
    assert np.corrcoef(pred, yt)[0, 1] > 0.8
    with tempfile.TemporaryDirectory() as d:
        path = os.path.join(d, "e.bin")
        H.hf_mlp_save(path)
        H.hf_mlp_init(D, 99)
        H.hf_mlp_load(path)
    assert H.hf_mlp_members() == 4
    assert np.array_equal(H.hf_mlp_predict(Xt), pred)


def test_hf_tune_mlp_profiles_only_topk():
    pairs = LT.draw_pairs(6, seed=6, kmin=18, kmax=22)
    data = LT.collect(pairs, reps=3, seed=6)
    H.hf_mlp_init(D, 0)
    H.hf_mlp_train(data["X"], data["y"] - data["X"][:, LT.SUM_SOLO], epochs=500, lr=1e-3)
    ia, ib = LT.Instance(0, 20, 1), LT.Instance(1, 20, 2)
    pr = H.make_pair(ia.task, ib.task)
    best, st = H.hf_tune(pr, H.HF_TUNE_MLP, 0, 3)
    assert st["n_profiled"] == 3 and st["n_candidates"] == 85
    # the featurisation's own cost: two kernels x three blocks x six launches
    assert st["n_solo_launches"] == 36 and st["solo_ms"] > 0
    assert H.hf_validate_fused(pr, best) == H.HF_OK


def test_hf_tune_mlp_orders_its_launches_on_the_callers_stream():
    """hf_tune(MLP) on a non-blocking stream right after an unsynchronised
    fused launch on that stream: the featurisation's solo launches run on the
    same stream, after it, so both tasks' outputs are right afterwards and
    their (caller-provided) scratch is left zero-filled."""
    from tests import gpu_cases as G
    pairs = LT.draw_pairs(4, seed=16, kmin=16, kmax=18, kinds=LT.DATA_KINDS)
    data = LT.collect(pairs, reps=2, seed=16)
    H.hf_mlp_init(D, 1)
    H.hf_mlp_train(data["X"], data["y"] - data["X"][:, LT.SUM_SOLO], epochs=100, lr=1e-3)
    ca, cb = G.bn_case((16, 64, 28, 28), seed=17), G.hist_case(1 << 22, seed=18)
    scr = [torch.zeros(H.hf_scratch_bytes(c.task) // 4, dtype=torch.int32, device="cuda") for c in (ca, cb)]
    ca.task.scratch, cb.task.scratch = scr[0].data_ptr(), scr[1].data_ptr()
    pr = H.make_pair(ca.task, cb.task)
    side = torch.cuda.Stream()  # created non-blocking by torch
    torch.cuda.synchronize()
    for c in (ca, cb):
        c.reset()
    H.hf_run_fused_cfg(pr, H.hf_config(2, 256, 0, 0), stream=side)
    H.hf_tune(pr, H.HF_TUNE_MLP, 0, 2, stream=side)
    torch.cuda.synchronize()
    ca.check(ca.outputs())
    cb.check(cb.outputs())
    assert all(int(t.abs().sum()) == 0 for t in scr)


def test_sample_store_resumes_an_interrupted_sweep(tmp_path, monkeypatch):
    """Samples are appended per pair as measured; a second sweep over the same
    pairs reads them back and profiles only the pair whose line was cut."""
    pairs = LT.draw_pairs(3, seed=9, kmin=16, kmax=18, kinds=LT.DATA_KINDS)
    st = str(tmp_path / "samples.jsonl")
    a = LT.collect(pairs, reps=2, seed=9, store=st)
    lines = open(st).read().splitlines(True)
    assert len(lines) == 3
    open(st, "w").write("".join(lines[:2]) + lines[2][:40])  # as an interrupted run leaves it
    calls = []
    real = LT.H.hf_profile
    monkeypatch.setattr(LT.H, "hf_profile", lambda *x, **k: calls.append(1) or real(*x, **k))
    b = LT.collect(pairs, reps=2, seed=9, store=st)
    n = len(H.hf_tune_candidates(H.HF_TUNE_EXHAUSTIVE, 0))
    assert len(calls) == n  # only the third pair again
    np.testing.assert_array_equal(a["X"][:2 * n], b["X"][:2 * n])
    np.testing.assert_array_equal(a["y"][:2 * n], b["y"][:2 * n])
    assert len(open(st).read().splitlines()) == 4  # the cut line stays, the new one is appended
