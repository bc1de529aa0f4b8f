"""Posterior local passes with several segments per wavefront (K <= 32) and
sums over K rounded up to four, against the FP64 oracle with the tolerances of
the posterior's own tests: segment counts that leave lane groups of the last
wavefront empty, a last segment of one observation, segments shorter than, equal
to and longer than a staged chunk."""
import pytest

import oracle
from paper_2003_03508_amd import synth

from test_gpu_parity import binding, ctx  # noqa: F401
from test_gpu_posterior import _check, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,T,L", [(2, 129, 32), (4, 161, 32), (5, 97, 32), (12, 1, 0), (13, 2049, 64), (16, 641, 40),
                                   (16, 3000, 128), (17, 33, 32), (18, 64, 32), (20, 65, 64), (21, 1985, 31),
                                   (24, 701, 100), (28, 97, 96), (29, 3001, 60), (32, 2177, 64), (36, 129, 64),
                                   (45, 700, 33), (60, 1025, 128)])
def test_lane_groups(binding, ctx, K, T, L):  # noqa: F811
    prm, obs = synth.make(K, T, 9000 + K)
    want = oracle.posterior(prm.delta, prm.Gamma, prm.p, prm.mu, prm.Sigma, obs.flag, obs.xy)
    _check(_run(binding, ctx, prm, obs, L), want, T, (K, T, L))
