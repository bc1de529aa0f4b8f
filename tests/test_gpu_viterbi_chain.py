"""The Viterbi segment chains (verified score vectors) against the FP64 oracle,
and their return to the max-plus product path.

Tolerances as for the product path: score and the joint log probability along
the returned path within 1e-6 relative of the oracle's maximum; the paths may
differ where both are maxima up to FP32 rounding (T / 1000 states, at least 2).

A context whose fold width is set explicitly runs the product path alone:
where the chains give a call back, both contexts must return the same."""
import math

import numpy as np
import pytest

import oracle
from paper_2003_03508_amd import synth

from test_gpu_chain import product, sticky  # noqa: F401
from test_gpu_parity import binding, ctx  # noqa: F401
from test_gpu_viterbi import _path_score

pytestmark = pytest.mark.gpu


def run(binding, c, prm, obs):  # noqa: F811
    path, first, score = c.viterbi(**binding.to_device(prm, obs))
    return path.cpu().numpy(), int(first.item()), float(score.item())


def check(binding, c, prm, obs, what):  # noqa: F811
    want, wpath, wfirst = oracle.viterbi(prm.delta, prm.Gamma, prm.p, prm.mu, prm.Sigma, obs.flag, obs.xy)
    path, first, score = run(binding, c, prm, obs)
    tol = 1e-6 * max(1.0, abs(want))
    assert abs(score - want) <= tol, (what, score, want)
    assert path.shape == wpath.shape and path.min() >= 0 and path.max() < prm.K
    assert abs(_path_score(prm, obs, first, path) - want) <= tol, what
    assert int((path != wpath).sum()) + int(first != wfirst) <= max(2, obs.T // 1000), what


# every lane layout (four, two, one segment per wavefront, two states per
# lane), K on and off a multiple of four, the shortest records, segment counts
# that do and do not fill the last wavefront, two segment lengths in a record
@pytest.mark.parametrize("K,T", [(1, 1000), (2, 1001), (3, 4097), (4, 1013), (7, 3001), (8, 70_001), (13, 1999),
                                 (16, 1025), (17, 1012), (20, 33_333), (25, 1056), (25, 100_003), (31, 2049), (32, 4000),
                                 (33, 1024), (34, 1111), (44, 6400), (47, 3000), (61, 1777), (64, 20_001), (65, 1024),
                                 (66, 2500), (77, 1301), (80, 9_999)])
def test_matches_oracle(binding, ctx, K, T):  # noqa: F811
    prm, obs = synth.make(K, T, 7000 + K)
    check(binding, ctx, prm, obs, (K, T))


def test_delta_with_zeros_and_missing_runs(binding, ctx):  # noqa: F811
    prm, obs = synth.make(21, 5000, 7100)
    prm.delta[:] = 0.0
    prm.delta[4] = prm.delta[20] = 0.5
    flag = obs.flag.copy()
    flag[:150] = 0        # no locations where the record starts, nor over a
    flag[2000:2400] = 0   # stretch longer than warm-up and lookahead
    flag[-90:] = 0
    check(binding, ctx, prm, synth.Observations(flag=flag, xy=obs.xy), "missing")


@pytest.mark.parametrize("informative", [True, False])
@pytest.mark.parametrize("stay", [0.5, 0.9, 0.95, 0.98, 0.99, 0.999, 0.99999])
def test_slow_forgetting(binding, ctx, product, stay, informative):  # noqa: F811
    """From records that the warm-up and lookahead cover, over ones that need
    segments run again, to ones that are given back."""
    for K, T in ((20, 20_000), (6, 3001), (40, 2001)):
        prm, obs = sticky(K, T, stay, 7200 + K, informative)
        check(binding, ctx, prm, obs, (K, T))
        _, _, want = run(binding, product, prm, obs)
        assert abs(run(binding, ctx, prm, obs)[2] - want) <= 1e-6 * abs(want)


@pytest.mark.parametrize("K", [5, 30, 50, 70])
def test_given_back_is_the_product_path(binding, ctx, product, K):  # noqa: F811
    """Transitions below 2^-56 (here zeros): the product path's own result."""
    prm, obs = synth.make(K, 3000, 7300 + K)
    prm.Gamma[2, 3] = 0.0
    prm.Gamma[4, 0] = 0.0
    prm.Gamma /= prm.Gamma.sum(axis=1, keepdims=True)
    check(binding, ctx, prm, obs, K)
    a, b = run(binding, ctx, prm, obs), run(binding, product, prm, obs)
    assert (a[0] == b[0]).all() and a[1:] == b[1:]


@pytest.mark.parametrize("K", [9, 25, 64, 80])
@pytest.mark.parametrize("t", [0, 31, 1500, 2999])
def test_invalid_observation_anywhere(binding, ctx, K, t):  # noqa: F811
    prm, obs = synth.make(K, 3000, 7400)
    flag, xy = obs.flag.copy(), obs.xy.copy()
    flag[t], xy[t] = 1, (np.nan, 1.0)
    path, first, score = run(binding, ctx, prm, synth.Observations(flag=flag, xy=xy))
    assert math.isnan(score) and first == -1 and (path == -1).all()
    check(binding, ctx, prm, obs, "after invalid data")
