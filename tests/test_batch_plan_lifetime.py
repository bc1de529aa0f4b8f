"""Lifetimes of batched plans, on the CPU: the library's host code runs against a
model of the HIP runtime (runtime_model.c), which queues the work of every
stream and checks each handle and each piece of memory when it is used and when
it is given back."""
import ctypes
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(ROOT, "paper_2003_03508_amd", "libhmm.so")


class Library:
    """libhmm.so with its runtime calls bound to the model."""

    def __init__(self, model):
        self.m = ctypes.CDLL(model, mode=ctypes.RTLD_GLOBAL)   # ahead of the real runtime
        self.lib = ctypes.CDLL(LIB)
        vp, i32, i64 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64
        self.lib.hmm_loglik_batched.argtypes = [vp, i32, vp, vp, vp, vp, i64, vp, vp, vp, i64, i32, vp, vp]
        self.lib.hmm_autotune_batched.argtypes = [vp, i32, vp, vp, vp, vp, i64, vp, vp, vp, i64, i32, vp, i32, vp]
        self.lib.hmm_ctx_destroy.argtypes = [vp]
        self.lib.hmm_ctx_set_batch_graph.argtypes = [vp, i32]
        for f in ("calls", "syncs", "copies", "launches", "replays", "live"):
            getattr(self.m, "model_" + f).restype = ctypes.c_long
        self.m.model_violations.restype = ctypes.c_long
        self.m.model_violations.argtypes = [ctypes.c_char_p, ctypes.c_size_t]
        self.m.model_fail_at.argtypes = [ctypes.c_long]
        self.h = vp()
        assert self.lib.hmm_ctx_create(ctypes.byref(self.h), 0) == 0

    def count(self, what):
        return getattr(self.m, "model_" + what)()

    def clean(self):
        text = ctypes.create_string_buffer(4096)
        n = self.m.model_violations(text, 4096)
        assert n == 0, text.value.decode()

    def call(self, d, algo=1, stream=None):
        return self.lib.hmm_loglik_batched(self.h, d["n"], *[d[k].ctypes.data for k in ("K", "T", "po", "params")],
                                           d["params"].size, d["oo"].ctypes.data, d["flag"].ctypes.data,
                                           d["xy"].ctypes.data, d["flag"].size, algo, stream, d["out"].ctypes.data)

    def autotune(self, d):
        return self.lib.hmm_autotune_batched(self.h, d["n"], *[d[k].ctypes.data for k in ("K", "T", "po", "params")],
                                             d["params"].size, d["oo"].ctypes.data, d["flag"].ctypes.data,
                                             d["xy"].ctypes.data, d["flag"].size, 1, d["out"].ctypes.data, 1, None)

    def close(self):
        assert self.lib.hmm_ctx_destroy(self.h) == 0
        self.clean()


def aligned(n, dtype):
    a = np.zeros(n + 16, dtype=dtype)
    return a[(-a.ctypes.data // a.itemsize) % (64 // a.itemsize):][:n]


def sets(rng, n, K_lo, K_hi, T_lo, T_hi):
    K = rng.integers(K_lo, K_hi + 1, size=n).astype(np.int32)
    T = rng.integers(T_lo, T_hi + 1, size=n).astype(np.int64)
    blk = K.astype(np.int64) * (K + 7)
    return dict(n=n, K=K, T=T, po=np.concatenate([[0], np.cumsum(blk)[:-1]]).astype(np.int64),
                params=aligned(int(blk.sum()), np.float64), oo=np.concatenate([[0], np.cumsum(T)[:-1]]).astype(np.int64),
                flag=np.zeros(int(T.sum()), np.uint8), xy=aligned(2 * int(T.sum()), np.float64),
                out=aligned(n, np.float64))


def others(d):
    """The same descriptors with other buffers."""
    return dict(d, params=aligned(d["params"].size, np.float64), flag=d["flag"].copy(),
                xy=aligned(d["xy"].size, np.float64), out=aligned(d["n"], np.float64))


def descriptors_change(L):
    """A plan with other descriptors is made after a device synchronisation, of
    memory, events and streams of its own, whatever became of the last one:
    launched once, captured and replayed, or never used to the end."""
    rng = np.random.default_rng(1)
    a, b = (sets(rng, 40, 4, 73, 2000, 65310) for _ in range(2))
    base = L.count("live")
    for graph in (1, 0):
        L.lib.hmm_ctx_set_batch_graph(L.h, graph)
        for uses in (1, 2, 3):
            for d in (a, b):
                before = L.count("syncs")
                for k in range(uses):
                    assert L.call(d) == 0
                    if k == 0:
                        assert L.count("syncs") >= before + (0 if L.first else 1), (graph, uses)
                        L.first = False
                        # memory, pinned tables, their event: nothing left of the plan before
                        assert L.count("live") == base + 3, (graph, uses)
        L.lib.hmm_ctx_set_batch_graph(L.h, graph)   # gives the plan back
        L.first = True
        assert L.count("live") == base
    assert L.count("replays") > 0


def many_changes(L):
    rng = np.random.default_rng(514286259)
    for it in range(25):
        n, K_hi, T_hi = (int(rng.choice(c)) for c in ([1, 2, 6, 32, 40], [8, 20, 40, 73, 80], [4000, 20000, 65310]))
        ds = [sets(rng, n, 4, K_hi, 2000, T_hi) for _ in range(2)]
        ds.append(others(ds[0]))
        for _ in range(12):
            assert L.call(ds[rng.integers(3)], int(rng.choice([0, 1, 1, 1, 2]))) == 0
        if it % 8 == 0:
            assert L.autotune(ds[0]) == 0
        L.clean()


def failed_copy(L):
    """A call whose copy of the new pointers failed leaves no plan that matches
    them: the next call copies again instead of using the old buffers."""
    a = sets(np.random.default_rng(2), 5, 20, 40, 2000, 9000)
    for uses in (1, 3):
        for at in (1, 2, 3):   # waiting for the last copy, the copy, the event after it
            for _ in range(uses):
                assert L.call(a) == 0
            b = others(a)
            L.m.model_fail_at(at)
            assert L.call(b) == -3
            L.m.model_fail_at(0)
            before = L.count("copies")
            assert L.call(b) == 0
            assert L.count("copies") == before + 1, (uses, at)
            assert L.call(b) == 0 and L.count("copies") == before + 1
            L.clean()


def any_call_fails(L):
    """Each runtime call in turn fails: an error comes back, nothing is misused,
    and the call after it works."""
    rng = np.random.default_rng(3)
    a, b = (sets(rng, 6, 4, 73, 2000, 9000) for _ in range(2))
    c = others(b)
    for seq in ((a, b, b, c), (c, a, a, a)):
        for d in seq:   # kernels' attributes are set once
            assert L.call(d) == 0
        for at in range(1, 400):
            start = L.count("calls")
            L.m.model_fail_at(at)
            codes = [L.call(d) for d in seq]
            L.m.model_fail_at(0)
            L.clean()
            assert all(L.call(d) == 0 for d in seq), at
            if L.count("calls") - start < at or not any(codes):
                break
        assert at > 20


CASES = {f.__name__: f for f in (descriptors_change, many_changes, failed_copy, any_call_fails)}


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    if shutil.which("gcc") is None:
        pytest.skip("needs gcc")
    if not os.path.exists(LIB):
        from paper_2003_03508_amd import build
        build.build()
    so = str(tmp_path_factory.mktemp("model") / "runtime_model.so")
    subprocess.run(["gcc", "-O1", "-g", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "runtime_model.c")], check=True)
    return so


@pytest.mark.parametrize("case", sorted(CASES))
def test_plan(model, case):
    # a process of its own: the model takes the place of the HIP runtime
    r = subprocess.run([sys.executable, os.path.abspath(__file__), model, case], capture_output=True, text=True,
                       timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


if __name__ == "__main__":
    lib = Library(sys.argv[1])
    lib.first = True
    CASES[sys.argv[2]](lib)
    lib.close()
