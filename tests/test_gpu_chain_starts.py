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

from paper_2003_03508_amd import synth

from test_gpu_chain import run
from test_gpu_parity import binding, ctx, ref, assert_close  # noqa: F401

pytestmark = pytest.mark.gpu


def two_groups(K, T):
    h = K // 2
    prm, _ = synth.make(K, 10, 1)
    G = np.empty((K, K))
    G[:h, :h], G[:h, h:] = 0.98 / h, 0.02 / (K - h)
    G[h:, :h], G[h:, h:] = 0.2 / h, 0.8 / (K - h)
    prm.Gamma = G
    prm.p = np.where(np.arange(K) < h, 0.3, 0.01)
    return prm, synth.Observations(flag=np.zeros(T, np.uint8), xy=np.full((T, 2), np.nan))


@pytest.mark.parametrize("K,T", [(20, 20_000), (26, 20_000), (40, 30_000), (64, 20_000), (80, 20_000)])
def test_flat_starts_do_not_add_up(binding, ctx, K, T):  # noqa: F811
    prm, obs = two_groups(K, T)
    assert_close(run(binding, ctx, prm, obs), ref(prm, obs), f"K={K} T={T}")
