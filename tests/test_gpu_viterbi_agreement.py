"""The Viterbi chains against the max-plus product path (a context with the fold
width set): the same path, and the score within 1e-10.  Both add the score up in
the same FP32 order; what differs is the FP64 sum over segments and the powers of
two taken out of it."""
import numpy as np
import pytest

from paper_2003_03508_amd import synth

from test_gpu_chain import product  # noqa: F401
from test_gpu_parity import binding, ctx  # noqa: F401
from test_gpu_viterbi_chain import check, run

pytestmark = pytest.mark.gpu


def agree(binding, ctx, product, prm, obs, what):  # noqa: F811
    a, b = run(binding, ctx, prm, obs), run(binding, product, prm, obs)
    assert (a[0] == b[0]).all() and a[1] == b[1], what
    assert abs(a[2] - b[2]) <= 1e-10 * abs(b[2]), (what, a[2], b[2])


@pytest.mark.parametrize("K,T", [(3, 5000), (16, 20_011), (25, 100_003), (32, 9001), (48, 7000), (64, 20_001), (80, 5003)])
def test_path_and_score(binding, ctx, product, K, T):  # noqa: F811
    prm, obs = synth.make(K, T, 9100 + K)
    agree(binding, ctx, product, prm, obs, (K, T))


# segments of 32 (T = 1024 and 2048): no location over the warm-up (96 steps) of
# one of them, or over the lookahead (64 steps) past its end, or over both
@pytest.mark.parametrize("K,T", [(7, 1024), (20, 1024), (50, 2048), (80, 2048)])
@pytest.mark.parametrize("before,after", [(104, 4), (4, 72), (104, 72)])
def test_a_segment_without_locations_around_it(binding, ctx, product, K, T, before, after):  # noqa: F811
    prm, obs = synth.make(K, T, 9200 + K)
    prm.p[:] = 0.5   # a missing location says nothing
    obs.flag[:] = 1
    obs.xy[:] = prm.mu[obs.states] + np.sqrt(prm.Sigma[obs.states][:, [0, 2]]) * np.random.default_rng(1).standard_normal((T, 2))
    obs.flag[512 - before:512 + after] = 0
    agree(binding, ctx, product, prm, obs, (K, T, before, after))
    check(binding, ctx, prm, obs, (K, T, before, after))
