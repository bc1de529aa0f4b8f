"""One fold launch for up to four products per wavefront (K <= 16), against the
FP64 oracle (1e-6 * max(|ln L|, 1), the blocked FP32 likelihood's bound): counts
of products around one and four per wavefront of the fold's workgroup."""
import pytest

from paper_2003_03508_amd import synth

from test_gpu_chain import run
from test_gpu_parity import binding, ctx, ref, assert_close  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 3, 13, 16])
@pytest.mark.parametrize("T,levels", [(512 * 16, 1), (512 * 16 + 1, 1), (512 * 33, 1), (512 * 64, 1),
                                      (512 * 64 + 1, 2)])
def test_fold_run(binding, ctx, K, T, levels):  # noqa: F811
    prm, obs = synth.make(K, T, seed=8000 + K)
    assert ctx.plan(K, T)["levels"] == levels
    assert_close(run(binding, ctx, prm, obs), ref(prm, obs), f"K={K} T={T}")
