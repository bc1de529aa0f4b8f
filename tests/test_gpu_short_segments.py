"""Short records at K <= 16, whose FP32 segments go down to 8 observations,
against the FP64 oracle (1e-6 * max(|ln L|, 1), the blocked FP32 likelihood's
bound): lengths around one, two and many such segments, one and several fold
levels, and the lengths from which the segments grow."""
import pytest

from paper_2003_03508_amd import synth

from test_gpu_chain import run
from test_gpu_parity import binding, ctx, ref, assert_close  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 3, 13, 16])
@pytest.mark.parametrize("T", [1, 7, 8, 9, 63, 127, 129, 2047, 2049, 32_767, 32_769, 40_001])
def test_short_records(binding, ctx, K, T):  # noqa: F811
    prm, obs = synth.make(K, T, seed=8000 + K)
    assert ctx.plan(K, T)["block_len"] == max(8, -(-T // 4096))
    assert_close(run(binding, ctx, prm, obs), ref(prm, obs), f"K={K} T={T}")
