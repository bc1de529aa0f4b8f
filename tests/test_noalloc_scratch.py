"""hmm_loglik_noalloc accepts every K <= 80 at every T < 2^40: its fixed scratch
holds the layout.  On the CPU, against the model of the HIP runtime (the launches
are counted, nothing runs)."""
import ctypes
import os
import subprocess
import sys


from test_batch_plan_lifetime import LIB, model  # noqa: F401


def every_size():
    lib = ctypes.CDLL(LIB)
    f = lib.hmm_loglik_noalloc
    vp = ctypes.c_void_p
    f.argtypes = [ctypes.c_int32] + [vp] * 5 + [ctypes.c_int64] + [vp] * 2 + [ctypes.c_int32] + [vp] * 2
    some = (ctypes.c_double * 16)()
    p = (ctypes.addressof(some) + 15) // 16 * 16
    refused = [(K, T, algo) for K in range(1, 81) for algo in (1, 2, 3)
               for T in [10**6] + [2**k for k in range(31, 40)] + [2**40 - 1]
               if f(K, p, p, p, p, p, T, p, p, algo, None, p) != 0]
    assert not refused, refused


def test_every_size_is_accepted(model):  # noqa: F811
    r = subprocess.run([sys.executable, os.path.abspath(__file__), model], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


if __name__ == "__main__":
    ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)   # ahead of the real runtime
    every_size()
