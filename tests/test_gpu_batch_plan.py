"""Batched plans from call to call: other buffers with the same descriptors,
other descriptors, graph replays in between, a captured call, and sets that the
segment chains give back beside sets they serve.  Against the FP64 oracle,
1e-6 * max(|ln L|, 1)."""
import numpy as np
import pytest
import torch

from paper_2003_03508_amd import synth

from test_gpu_parity import binding, ref, assert_close  # noqa: F401

pytestmark = pytest.mark.gpu


def batch(binding, specs, seed, sparse=()):  # noqa: F811
    sets = [synth.make(K, T, seed=seed + i) for i, (K, T) in enumerate(specs)]
    for i in sparse:
        G = sets[i][0].Gamma
        G[0, 1] = 0.0
        G[0] /= G[0].sum()
    return sets, binding.batch_to_device(synth.pack(sets))


def check(out, sets, what):
    got = out.cpu().numpy()
    for i, (prm, obs) in enumerate(sets):
        assert_close(float(got[i]), ref(prm, obs), (what, i, prm.K, obs.T))


SPECS = [(25, 20_000), (40, 5003), (20, 31_000), (9, 2000), (64, 3001), (25, 64), (33, 1), (80, 2500), (3, 700)]


@pytest.mark.parametrize("graph", [True, False])
def test_buffers_and_descriptors_change(binding, graph):  # noqa: F811
    c = binding.Context(0)
    c.batch_graph(graph)
    try:
        a, da = batch(binding, SPECS, 5000)
        b, db = batch(binding, SPECS, 5100)              # same descriptors, other buffers
        s, ds = batch(binding, SPECS[::-1] + [(17, 9000)] * 40, 5200)   # other descriptors, larger tables
        # the first, replayed and changed use of every plan, without waiting in between
        seq = [(a, da), (a, da), (b, db), (b, db), (a, da), (s, ds), (s, ds), (b, db), (a, da), (a, da), (s, ds)]
        outs = [c.loglik_batched(**d) for _, d in seq]
        torch.cuda.synchronize()
        for k, ((sets, _), o) in enumerate(zip(seq, outs)):
            check(o, sets, k)
    finally:
        c.close()


def test_captured_call(binding):  # noqa: F811
    c = binding.Context(0)
    try:
        sets, d = batch(binding, SPECS, 5300)
        out = torch.empty(len(sets), dtype=torch.float64, device="cuda")
        g = torch.cuda.CUDAGraph()
        c.loglik_batched(**d, out=out)
        torch.cuda.synchronize()
        with torch.cuda.graph(g):
            c.loglik_batched(**d, out=out)
        want = out.cpu().numpy()
        for _ in range(3):
            out.zero_()
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert (out.cpu().numpy() == want).all()
        check(out, sets, "replay")
    finally:
        c.close()


@pytest.mark.parametrize("persistent", [True, False])
def test_sets_given_back_beside_served_ones(binding, persistent):  # noqa: F811
    """A sparse transition matrix sends its set to the product path; the
    others of its class (same K) and of other classes stay with the chains."""
    c = binding.Context(0)
    c.set_batch_persistent(persistent)
    try:
        for sparse in ((), (1,), (0, 3), (0, 1, 2, 3, 4)):
            sets, d = batch(binding, [(25, 9000), (25, 8000), (40, 4000), (40, 3000), (18, 5000)], 5400, sparse)
            for rep in range(3):
                check(c.loglik_batched(**d), sets, (sparse, rep))
    finally:
        c.close()


def test_autotune_right_after_a_call(binding):  # noqa: F811
    c = binding.Context(0)
    try:
        sets, d = batch(binding, [(25, 60_000), (40, 30_000), (12, 20_000)], 5500)
        first = c.loglik_batched(**d)
        c.autotune_batched(**d, reps=1)
        check(first, sets, "before")
        check(c.loglik_batched(**d), sets, "after")
        c.set_blocking(0, 1)   # the product path with the tuned lengths
        check(c.loglik_batched(**d), sets, "product")
    finally:
        c.close()


def test_empty_and_short_sets(binding):  # noqa: F811
    c = binding.Context(0)
    try:
        sets, d = batch(binding, [(30, 0), (30, 1), (30, 63), (30, 64), (30, 65), (30, 3000)], 5600)
        for _ in range(2):
            check(c.loglik_batched(**d), sets, "short")
        bad = dict(d)
        bad["xy"] = d["xy"].clone()
        T0 = 1 + 63 + 64 + 65
        fl = d["flag"].clone()
        fl[T0 + 100] = 3
        bad["flag"] = fl
        out = c.loglik_batched(**bad).cpu().numpy()
        assert np.isnan(out[5]) and np.isfinite(out[:5]).all()
    finally:
        c.close()
