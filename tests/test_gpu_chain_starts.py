"""Where the segments of the likelihood's chains start: the part of a flat start
that the warm-up leaves, and segments that are run again.

Two groups of states that mix within themselves at once and exchange slowly: the
chain forgets by 0.76 per step and the warm-up (40 steps, from the diagonal)
leaves 1.4e-5 of the flat start, below the 2^-16 that the check of a single
segment allows.  Without events every segment is off the same way: 2.8e-7 nats
per observation in 64 bits, 1.4e-6 of ln L.  Bound: the blocked FP32
likelihood's 1e-6 |ln L|."""
import numpy as np
import pytest

import oracle
from paper_2003_03508_amd import synth

from test_gpu_chain import product, run, sticky  # noqa: F401
from test_gpu_parity import binding, ctx, ref, assert_close  # noqa: F401

pytestmark = pytest.mark.gpu


def exchange(K, there, back):
    """Two groups of states that mix within themselves at once and exchange slowly."""
    h = K // 2
    G = np.empty((K, K))
    G[:h, :h], G[:h, h:] = (1 - there) / h, there / (K - h)
    G[h:, :h], G[h:, h:] = back / h, (1 - back) / (K - h)
    return G


def two_groups(K, T):
    h = K // 2
    prm, _ = synth.make(K, 10, 1)
    prm.Gamma = exchange(K, 0.02, 0.2)
    prm.p = np.where(np.arange(K) < h, 0.3, 0.01)
    return prm, synth.Observations(flag=np.zeros(T, np.uint8), xy=np.full((T, 2), np.nan))


@pytest.mark.parametrize("K,T", [(20, 20_000), (26, 20_000), (40, 30_000), (64, 20_000), (80, 20_000)])
def test_flat_starts_do_not_add_up(binding, ctx, K, T):  # noqa: F811
    prm, obs = two_groups(K, T)
    assert_close(run(binding, ctx, prm, obs), ref(prm, obs), f"K={K} T={T}")


def served(binding, ctx, product, prm, obs, quiet=False):  # noqa: F811
    """The chains served the call: another rounding than the segment products'
    (a set that is given back returns their bits), near them: FP32 rounding is
    1e-9 of ln L, 1e-8 is allowed; in a quiet record 2e-7 per observation."""
    got, want = run(binding, ctx, prm, obs), run(binding, product, prm, obs)
    assert got != want and abs(got - want) <= (2e-7 * obs.T if quiet else 1e-8 * abs(want)), (got, want)
    return got


@pytest.mark.parametrize("K,T", [(17, 3000), (20, 40_000), (25, 105_000), (33, 9000), (48, 20_000), (64, 7777),
                                 (80, 20_001)])
def test_chains_serve_the_generator_s_records(binding, ctx, product, K, T):  # noqa: F811
    prm, obs = synth.make(K, T, 8800 + K)
    assert_close(served(binding, ctx, product, prm, obs), ref(prm, obs), f"K={K} T={T}")


def starts_off(prm, obs, warm, q):
    """In 64 bits: the segments of q observations whose start, after `warm` steps
    from a flat vector, differs by more than 2^-16 from the forward vector there."""
    e = np.exp(np.asarray(oracle.log_emission(prm.p, prm.mu, prm.Sigma, obs.flag, obs.xy)))

    def walk(v, a, b):
        for t in range(a, b):
            v = (v @ prm.Gamma) * e[t]
            v = v / v.sum()
        return v
    off, v = [], prm.delta
    for b in range(1, obs.T // q):
        v = walk(v, (b - 1) * q, b * q)
        if b * q > warm:
            s = walk(np.full(prm.K, 1.0 / prm.K), b * q - warm, b * q)
            if np.abs(s / v - 1.0).max() > 2.0**-16:
                off.append(b)
    return off


# segments of 32 observations, warm-up 40: a segment inside a walker's sixteen,
# the first of a walker (of the next workgroup, of the same), two of them
@pytest.mark.parametrize("K,T,where", [(20, 1536, (5,)), (20, 1536, (16,)), (20, 1536, (21, 32)), (40, 2048, (9,)),
                                       (40, 2048, (16,)), (40, 2048, (32,)), (80, 2048, (32, 50))])
def test_single_segments_run_again(binding, ctx, product, K, T, where):  # noqa: F811
    """Locations tell the groups apart everywhere but over the warm-up of the
    named segments, which alone start elsewhere and are run again."""
    prm, _ = synth.make(K, 10, 8900 + K)
    prm.Gamma = exchange(K, 0.04, 0.04)
    prm.p[:] = 0.5
    prm.mu[:K // 2, 0], prm.mu[K // 2:, 0] = 0.0, 40.0
    prm.Sigma[:] = (100.0, 0.0, 100.0)
    prm.mu[:, 1] = np.arange(K) * 0.1
    obs = synth.sample_path(np.random.default_rng(8901), prm, T)
    obs.xy[:] = prm.mu[obs.states] + 10.0 * np.random.default_rng(8902).standard_normal((T, 2))
    obs.flag[:] = 1
    for b in where:
        obs.flag[32 * b - 44:32 * b + 4] = 0
    assert starts_off(prm, obs, 40, 32) == list(where)
    assert_close(served(binding, ctx, product, prm, obs), ref(prm, obs), (K, where))


@pytest.mark.parametrize("K,T,stay", [(20, 40_000, 0.96), (40, 9000, 0.96), (80, 5000, 0.96), (25, 500_000, 0.98)])
def test_slow_states_take_the_products(binding, ctx, product, K, T, stay):  # noqa: F811
    prm, obs = sticky(K, T, stay, 43, True)
    got = run(binding, ctx, prm, obs)
    assert got == run(binding, product, prm, obs)
    assert_close(got, ref(prm, obs), (K, T, stay))


@pytest.mark.parametrize("K,T,slow", [(20, 40_000, 3), (25, 500_000, 24), (66, 5000, 65), (80, 20_000, 0)])
def test_one_slow_state_is_served(binding, ctx, product, K, T, slow):  # noqa: F811
    """A background state that is hardly left does not slow the others down."""
    prm, _ = synth.make(K, 10, 5)
    prm.Gamma[slow] = 0.002 * np.random.default_rng(5).dirichlet(np.ones(K))
    prm.Gamma[slow, slow] += 0.998
    prm.p[slow] = 0.001
    obs = synth.sample_path(np.random.default_rng(6), prm, T)
    assert_close(served(binding, ctx, product, prm, obs, quiet=True), ref(prm, obs), (K, T, slow))


@pytest.mark.parametrize("K", [20, 26, 40])
@pytest.mark.parametrize("there,back,p", [(0.004625, 0.087875, (0.15, 0.02)), (0.0035, 0.0665, (0.2, 0.1)),
                                          (0.010125, 0.057375, (0.1, 0.02))])
def test_flat_starts_after_the_last_rerun(binding, ctx, there, back, p, K):  # noqa: F811
    """Groups that exchange so slowly that a segment's start meets the tolerance
    only in the last rerun: 64-bit bias 1.8e-6..3.6e-6 of ln L.  In a batch with a
    long record, whose products cost enough for three reruns."""
    prm, obs = two_groups(K, 8192)
    prm.Gamma = exchange(K, there, back)
    prm.p = np.where(np.arange(K) < K // 2, *p)
    sets = [(prm, obs), synth.make(K, 200_000, 3)]
    out = ctx.loglik_batched(**binding.batch_to_device(synth.pack(sets))).cpu().numpy()
    for i, s in enumerate(sets):
        assert_close(float(out[i]), ref(*s), (K, i))
