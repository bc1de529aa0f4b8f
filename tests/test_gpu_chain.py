"""The segment chains (verified forward vectors) behind the FP32 blocked
likelihood, against the FP64 oracle, and their return to the product path.

Tolerance 1e-6 * max(|ln L|, 1), the blocked FP32 likelihood's bound.  A
segment is accepted when its start is parallel to its neighbour's end within
2^-16 per entry, so even if every one of nb segments were off by that much
ln L would move by nb * 2^-16 nats: below 1e-6 |ln L| for segments of at least
32 observations at 1 nat or more each.

A context whose fold width is set explicitly (to the automatic value) runs the
product path alone: where the chains give a set back, both contexts must
return the same bits."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2003_03508_amd import synth

from test_gpu_parity import binding, ctx, ref, assert_close  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def product(binding):  # noqa: F811
    c = binding.Context(0)
    c.set_blocking(0, 1)
    yield c
    c.close()


def run(binding, c, prm, obs):  # noqa: F811
    return float(c.loglik(**binding.to_device(prm, obs)).item())


# every count of contraction slots, both emission layouts (K <= 32 and above),
# partly filled slots, one to many walkers and workgroups, ragged tails
@pytest.mark.parametrize("K,T", [(17, 1000), (20, 33_333), (21, 4097), (24, 2048), (25, 1023), (25, 65_536 + 1),
                                 (28, 64), (29, 65), (32, 16 * 32 * 4), (33, 16 * 32 * 4 + 1), (36, 127), (37, 5000),
                                 (40, 511), (44, 513), (45, 3000), (48, 12_345), (49, 2000), (56, 100), (60, 4000),
                                 (64, 7777), (65, 64), (69, 3001), (73, 1500), (77, 2222), (80, 20_001),
                                 (1, 4_000_000), (3, 4_000_001), (8, 1_000_001), (13, 1_048_577), (16, 1_000_003)])
def test_matches_oracle(binding, ctx, K, T):  # noqa: F811
    prm, obs = synth.make(K, T, seed=4000 + K)
    assert_close(run(binding, ctx, prm, obs), ref(prm, obs), f"K={K} T={T}")


def test_delta_with_zeros_and_correlated_sigma(binding, ctx):  # noqa: F811
    prm, obs = synth.make(30, 5000, seed=4100)
    prm.delta[:] = 0.0
    prm.delta[7] = 0.25
    prm.delta[29] = 0.5   # not normalised: eq. (2) is linear in delta
    prm.Sigma[:, 1] = 0.4 * np.sqrt(prm.Sigma[:, 0] * prm.Sigma[:, 2])
    assert_close(run(binding, ctx, prm, obs), ref(prm, obs), "delta")


def sticky(K, T, stay, seed, informative):
    """Chains that leave a state with probability 1 - stay; without location
    information they forget by about `stay` per step."""
    rng = np.random.default_rng(seed)
    prm, _ = synth.make(K, 10, seed)
    prm.Gamma = (1.0 - stay) * rng.dirichlet(np.ones(K), size=K)
    prm.Gamma[np.diag_indices(K)] += stay
    prm.Gamma /= prm.Gamma.sum(axis=1, keepdims=True)
    if not informative:
        prm.mu[:] = prm.mu[0]
        prm.Sigma[:] = prm.Sigma[0]
        prm.p[:] = np.linspace(0.3, 0.5, K)
    return prm, synth.sample_path(np.random.default_rng(seed + 1), prm, T)


@pytest.mark.parametrize("informative", [True, False])
@pytest.mark.parametrize("stay", [0.5, 0.9, 0.95, 0.97, 0.98, 0.99, 0.999, 0.99999])
def test_slow_forgetting(binding, ctx, stay, informative):  # noqa: F811
    """From chains that the warm-up covers, over ones that need reruns within
    a walker and across walkers, to ones that are given back."""
    for K, T in ((20, 40_000), (40, 9_001)):
        prm, obs = sticky(K, T, stay, 4200 + K, informative)
        assert_close(run(binding, ctx, prm, obs), ref(prm, obs), f"K={K} stay={stay} informative={informative}")


def test_given_back_chains_return_the_product_path(binding, ctx, product):  # noqa: F811
    """Transition matrices with zero (or negligible) entries are refused before
    the chains run, nearly diagonal ones after them."""
    prm, obs = sticky(20, 30_000, 0.9, 4300, True)
    sparse = synth.HMMParams(**prm.__dict__)
    sparse.Gamma = prm.Gamma.copy()
    sparse.Gamma[3, 5] = 0.0
    tiny = synth.HMMParams(**prm.__dict__)
    tiny.Gamma = prm.Gamma.copy()
    tiny.Gamma[3, 5] = 1e-30
    slow, obs_slow = sticky(20, 30_000, 0.999999, 4301, False)
    for name, p, o in (("zero", sparse, obs), ("tiny", tiny, obs), ("slow", slow, obs_slow)):
        got, want = run(binding, ctx, p, o), run(binding, product, p, o)
        assert got == want, (name, got, want)
        assert_close(got, ref(p, o), name)


def test_identity_transitions(binding, ctx):  # noqa: F811
    K, T = 18, 3000
    prm, _ = synth.make(K, 10, 4400)
    prm.mu[:] = prm.mu.mean(axis=0) + 0.1 * (prm.mu - prm.mu.mean(axis=0))
    obs = synth.sample_path(np.random.default_rng(1), prm, T)
    prm.Gamma = np.eye(K)
    le = oracle.log_emission(prm.p, prm.mu, prm.Sigma, obs.flag, obs.xy).sum(axis=0) + np.log(prm.delta)
    want = le.max() + math.log(np.exp(le - le.max()).sum())
    assert_close(run(binding, ctx, prm, obs), want, "Gamma = I")


@pytest.mark.parametrize("what", ["outlier", "far", "impossible", "flag", "nan", "p"])
def test_extreme_and_invalid_data(binding, ctx, product, what):  # noqa: F811
    """Data far outside every state's ellipse, in the first, an inner and the
    last segment; L = 0; invalid data and parameters; then a good call."""
    prm, obs = synth.make(22, 20_000, seed=4500)
    for t in (0, 11_111, 19_999):
        p = synth.HMMParams(**{k: v.copy() for k, v in prm.__dict__.items()})
        flag, xy = obs.flag.copy(), obs.xy.copy()
        flag[t] = 1
        if what == "outlier":
            xy[t] = (900.0, -700.0)
        elif what == "far":
            xy[t] = (4.0e5, 1.0e5)
        elif what == "impossible":
            flag[:] = 0
            flag[t] = 1
            xy[t] = (10.0, 10.0)
            p.p[:] = 0.0
        elif what == "flag":
            flag[t] = 2
        elif what == "nan":
            xy[t] = (np.nan, 0.0)
        else:
            p.p[3] = 1.5
        o = synth.Observations(flag, xy)
        got = run(binding, ctx, p, o)
        if what in ("flag", "nan", "p"):
            assert math.isnan(got)
        elif what == "impossible":
            assert got == -math.inf
        else:
            assert_close(got, ref(p, o), (what, t))
    assert_close(run(binding, ctx, prm, obs), ref(prm, obs), "after")


@pytest.mark.parametrize("kind", [1, 2])
@pytest.mark.parametrize("K,T", [(18, 3001), (32, 20_000), (33, 9999), (50, 2500), (80, 3000), (5, 1_000_001)])
def test_other_kinds(binding, ctx, kind, K, T):  # noqa: F811
    ks = synth.make_kind(kind, K, T, seed=4600 + K)
    want = oracle.loglik_kind(kind, ks.delta, ks.Gamma, ks.e0, ks.e1, ks.obs)
    d = binding.kind_to_device(ks)

    def call():
        return float(ctx.loglik_kind(kind, d["delta"], d["Gamma"], d["e0"], d["e1"], d["obs"]).item())
    assert_close(call(), want, (kind, K, T))
    bad = d["obs"].clone()
    bad[T // 2] = -1 if kind == 1 else math.inf
    d["obs"] = bad
    assert math.isnan(call())


def test_unaligned_flags_and_graph_capture(binding, ctx):  # noqa: F811
    """Flags at every byte alignment; and a call captured once its scratch
    exists replays with new parameter values."""
    prm, obs = synth.make(25, 5003, seed=4700)
    want = ref(prm, obs)
    d = binding.to_device(prm, obs)
    for k in range(4):
        f = torch.zeros(obs.T + 8, dtype=torch.uint8, device="cuda")
        f[k:k + obs.T] = d["flag"]
        dd = dict(d)
        dd["flag"] = f[k:k + obs.T]
        assert_close(float(ctx.loglik(**dd).item()), want, k)
    out = torch.empty(1, dtype=torch.float64, device="cuda")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ctx.loglik(**d, out=out)
    p2 = synth.HMMParams(prm.delta, prm.Gamma, prm.p * 0.8, prm.mu, prm.Sigma)
    for p in (prm, p2, prm):
        d["p"].copy_(torch.as_tensor(p.p, device="cuda"))
        g.replay()
        torch.cuda.synchronize()
        assert_close(float(out.item()), ref(p, obs), "replay")
        assert float(ctx.loglik(**d).item()) == float(out.item())
