"""Locations are read only where the flag is 1: a record whose last tremor lies
before the end of an xy buffer that stops there.  The buffer is an allocation of
its own (2 MiB: 131,072 pairs), the record goes on behind it.  Against the same
call with a buffer for the whole record, bit for bit."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2003_03508_amd import synth

from test_gpu_parity import binding, ctx  # noqa: F401

pytestmark = pytest.mark.gpu

PAIRS = 1 << 17


@pytest.fixture(scope="module")
def short_xy(binding):  # noqa: F811
    hip = binding.lib()   # finds the runtime it is linked with
    p = ctypes.c_void_p()
    assert hip.hipMalloc(ctypes.byref(p), ctypes.c_size_t(16 * PAIRS)) == 0
    yield hip, p.value
    torch.cuda.synchronize()
    hip.hipFree(p)


@pytest.mark.parametrize("K,T", [(25, PAIRS + 9000), (60, PAIRS + 3001)])
def test_record_longer_than_its_locations(binding, ctx, short_xy, K, T):  # noqa: F811
    hip, xy = short_xy
    prm, obs = synth.make(K, T, 9000 + K)
    obs.flag[PAIRS:] = 0
    obs.flag[PAIRS - 1] = 1
    obs.xy[PAIRS - 1] = prm.mu[0]
    d = binding.to_device(prm, obs)
    torch.cuda.synchronize()
    host = np.ascontiguousarray(obs.xy[:PAIRS])
    assert hip.hipMemcpy(ctypes.c_void_p(xy), ctypes.c_void_p(host.ctypes.data), ctypes.c_size_t(host.nbytes), 1) == 0
    lib, h = binding.lib(), ctx._h
    prm_ptrs = [d[k].data_ptr() for k in ("delta", "Gamma", "p", "mu", "Sigma")]
    f64 = dict(dtype=torch.float64, device="cuda")

    def outputs(xy_ptr):
        ll = torch.zeros(3, **f64)
        lib_out = [ll[i:].data_ptr() for i in range(3)]
        assert lib.hmm_loglik(h, K, *prm_ptrs, T, d["flag"].data_ptr(), xy_ptr, 1, None, lib_out[0]) == 0
        block = torch.as_tensor(prm.packed(), device="cuda")
        one = [np.array([v], t) for v, t in ((K, np.int32), (T, np.int64), (0, np.int64), (0, np.int64))]
        assert lib.hmm_loglik_batched(h, 1, *[a.ctypes.data for a in one[:3]], block.data_ptr(), block.numel(),
                                      one[3].ctypes.data, d["flag"].data_ptr(), xy_ptr, T, 1, None, lib_out[1]) == 0
        gamma = torch.zeros(T, K, dtype=torch.float32, device="cuda")
        stats = torch.zeros(K * K + K + 7 * K, **f64)
        assert lib.hmm_posterior(h, K, *prm_ptrs, T, d["flag"].data_ptr(), xy_ptr, None, gamma.data_ptr(),
                                 stats.data_ptr(), lib_out[2]) == 0
        path = torch.zeros(T, dtype=torch.int32, device="cuda")
        first = torch.zeros(1, dtype=torch.int32, device="cuda")
        score = torch.zeros(1, **f64)
        assert lib.hmm_viterbi(h, K, *prm_ptrs, T, d["flag"].data_ptr(), xy_ptr, None, path.data_ptr(),
                               first.data_ptr(), score.data_ptr()) == 0
        torch.cuda.synchronize()
        return [t.cpu().numpy() for t in (ll, gamma, stats, path, first, score)]

    want = outputs(d["xy"].data_ptr())
    assert np.isfinite(want[0]).all()
    for a, b in zip(outputs(xy), want):
        assert (a == b).all()
