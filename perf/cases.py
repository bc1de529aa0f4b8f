"""The work whose speed this library is measured by: calls of its public entry
points over the range of sizes that users bring, from a short record with a few
states to the longest sequence the 80-state model is run on.

Every case is a dict of plain values.  ``prepare`` draws the inputs with the
package's own generator (``synth``: the tremor HMM of the paper's model section,
or the Poisson / 1-D Gaussian HMMs) and moves them to the GPU; ``run`` makes one
call; ``exact`` evaluates the same quantity in 64 bits with torch alone.
"""
import math

import numpy as np
import torch

from paper_2003_03508_amd import binding, synth


# ---------------------------------------------------------------- the cases
def listed():
    return [
        # a short record with few states: the size a user tries first, and the
        # smallest call of a sampler, where launches and latency count
        {"name": "loglik_k3_t1e4", "op": "loglik", "K": 3, "T": 10_000, "algo": "blocked_f32"},
        # the size of the paper's Shikoku record at its 25 states: one
        # likelihood of a single Markov chain
        {"name": "loglik_k25_t105k", "op": "loglik", "K": 25, "T": 105_000, "algo": "blocked_f32"},
        # the headline workload of bench.py
        {"name": "loglik_k25_t1e6", "op": "loglik", "K": 25, "T": 1_000_000, "algo": "blocked_f32"},
        # the largest model on the longest record
        {"name": "loglik_k80_t4m", "op": "loglik", "K": 80, "T": 4_194_304, "algo": "blocked_f32"},
        # the 16-bit operand option on a ragged length
        {"name": "loglik_k80_bf16", "op": "loglik", "K": 80, "T": 1_000_003, "algo": "blocked_bf16"},
        # another emission family: Poisson counts, ragged length
        {"name": "kind_poisson_k25", "op": "kind", "kind": 1, "K": 25, "T": 999_983},
        # uneven sets in one call: model comparison over K with records of
        # different lengths
        {"name": "batch_mixed_32", "op": "batch", "n": 32, "K_lo": 8, "K_hi": 64, "T_lo": 10_000, "T_hi": 100_000,
         "shared": False},
        # eight Markov chains over one record: the likelihoods of one MCMC
        # iteration of the K = 20 posterior
        {"name": "chains_k20_x8", "op": "batch", "n": 8, "K_lo": 20, "K_hi": 20, "T_lo": 500_000, "T_hi": 500_000,
         "shared": True},
        # the reverse direction: state posteriors and expected counts
        {"name": "posterior_k25", "op": "posterior", "K": 25, "T": 300_007},
        # one EM iteration
        {"name": "em_step_k20", "op": "em", "K": 20, "T": 500_000},
        # classification: the most likely path at the headline size
        {"name": "viterbi_k25_t1e6", "op": "viterbi", "K": 25, "T": 1_000_000},
        # and with a large model on a record of the Shikoku size
        {"name": "viterbi_k64", "op": "viterbi", "K": 64, "T": 105_000},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any K of the range, lengths over their logarithm (mostly odd)."""
    op = rng.choice(["loglik", "loglik", "loglik", "lp", "kind", "batch", "chains", "posterior", "em", "viterbi"])
    if op == "loglik":
        return {"op": "loglik", "K": rng.randint(2, 80), "T": _log_int(rng, 1_000, 3_000_000), "algo": "blocked_f32"}
    if op == "lp":
        return {"op": "loglik", "K": rng.randint(8, 80), "T": _log_int(rng, 10_000, 3_000_000),
                "algo": rng.choice(["blocked_bf16", "blocked_f16"])}
    if op == "kind":
        return {"op": "kind", "kind": rng.choice([1, 2]), "K": rng.randint(2, 80), "T": _log_int(rng, 5_000, 2_000_000)}
    if op == "batch":
        return {"op": "batch", "n": rng.randint(2, 48), "K_lo": 4, "K_hi": rng.randint(8, 80), "T_lo": 2_000,
                "T_hi": _log_int(rng, 4_000, 100_000), "shared": False}
    if op == "chains":
        K = rng.randint(2, 40)
        T = _log_int(rng, 20_000, 500_000)
        return {"op": "batch", "n": rng.randint(1, 32), "K_lo": K, "K_hi": K, "T_lo": T, "T_hi": T, "shared": True}
    K = rng.randint(2, 80)
    T = min(_log_int(rng, 2_000, 1_000_000), 25_000_000 // K)
    if op == "viterbi" and K > 32:
        T = min(T, 200_000)
    return {"op": op, "K": K, "T": T}


# ---------------------------------------------------------------- inputs
def _inputs(case, seed):
    """The host inputs of a case, from the seed alone."""
    op = case["op"]
    if op == "kind":
        return synth.make_kind(case["kind"], case["K"], case["T"], seed)
    if op == "batch":
        rng = np.random.default_rng(seed)
        n = case["n"]
        Ks = rng.integers(case["K_lo"], case["K_hi"] + 1, size=n)
        Ts = rng.integers(case["T_lo"], case["T_hi"] + 1, size=n)
        if not case["shared"]:
            return synth.pack([synth.make(int(K), int(T), int(s))
                               for K, T, s in zip(Ks, Ts, rng.integers(0, 2**62, size=n))])
        # chains: parameter vectors around the generating one, one record
        prm, obs = synth.make(int(Ks[0]), int(Ts[0]), seed)
        sets = []
        for _ in range(n):
            G = prm.Gamma * np.exp(0.05 * rng.standard_normal(prm.Gamma.shape))
            q = synth.HMMParams(prm.delta, G / G.sum(axis=1, keepdims=True),
                                np.clip(prm.p * np.exp(0.02 * rng.standard_normal(prm.K)), 0.01, 0.99),
                                prm.mu + 0.5 * rng.standard_normal(prm.mu.shape),
                                prm.Sigma * np.exp(0.05 * rng.standard_normal((prm.K, 1))))
            sets.append(q)
        blocks = [q.packed() for q in sets]
        return dict(K=np.full(n, prm.K, np.int32), T=np.full(n, obs.T, np.int64),
                    param_off=np.arange(n, dtype=np.int64) * blocks[0].size, params=np.concatenate(blocks),
                    obs_off=np.zeros(n, np.int64), flag=obs.flag, xy=obs.xy)
    return synth.make(case["K"], case["T"], seed)


_ctx = None


def _context():
    """One library context, kept for the process as a user's program keeps it."""
    global _ctx
    if _ctx is None:
        _ctx = binding.Context(0)
    return _ctx


def prepare(case, seed):
    h = _inputs(case, seed)
    st = {"case": case, "ctx": _context()}
    if case["op"] == "kind":
        st["in"] = binding.kind_to_device(h)
    elif case["op"] == "batch":
        st["in"] = binding.batch_to_device(h)
        st["out"] = torch.empty(case["n"], dtype=torch.float64, device="cuda")
    elif case["op"] == "em":
        prm, obs = h
        d = binding.to_device(prm, obs)
        st["in"] = {"params": torch.as_tensor(prm.packed(), device="cuda"), "flag": d["flag"], "xy": d["xy"]}
    else:
        st["in"] = binding.to_device(*h)
    torch.cuda.synchronize()
    return st


# ---------------------------------------------------------------- one pass
def run(st):
    case, ctx, d = st["case"], st["ctx"], st["in"]
    op = case["op"]
    if op == "loglik":
        return ctx.loglik(**d, algo=case["algo"])
    if op == "kind":
        return ctx.loglik_kind(case["kind"], d["delta"], d["Gamma"], d["e0"], d["e1"], d["obs"])
    if op == "batch":
        return ctx.loglik_batched(**d, out=st["out"])
    if op == "posterior":
        return ctx.posterior(**d)
    if op == "em":
        return ctx.em_step(d["params"], case["K"], d["flag"], d["xy"])
    return ctx.viterbi(**d)


def work(case):
    """The forward recursion's arithmetic (one K x K vector-matrix product per
    observation, three with the reverse direction) and the observations read
    once (17 bytes; 4 or 8 for the other kinds), the results written once."""
    op = case["op"]
    if op == "batch":
        n, K = case["n"], 0.5 * (case["K_lo"] + case["K_hi"])
        K2 = (case["K_lo"] ** 2 + case["K_lo"] * case["K_hi"] + case["K_hi"] ** 2) / 3.0
        T = 0.5 * (case["T_lo"] + case["T_hi"])
        return {"bytes": int(17 * T * (1 if case["shared"] else n) + n * 8 * (K2 + 7 * K + 1)),
                "flops": int(2 * n * T * K2)}
    K, T = case["K"], case["T"]
    prm = 8 * K * (K + 7)
    if op == "loglik":
        return {"bytes": 17 * T + prm + 8, "flops": 2 * T * K * K}
    if op == "kind":
        return {"bytes": (4 if case["kind"] == 1 else 8) * T + prm + 8, "flops": 2 * T * K * K}
    if op == "posterior":
        return {"bytes": 17 * T + 4 * T * K + 2 * prm, "flops": 6 * T * K * K}
    if op == "em":
        return {"bytes": 17 * T + 2 * prm, "flops": 6 * T * K * K}
    return {"bytes": 17 * T + 4 * T + prm, "flops": 2 * T * K * K}


# ---------------------------------------------------------------- 64 bits
def _log_e(p, mu, Sigma, flag, xy):
    """ln e_{t,k} of eq. (1): (T, K) FP64."""
    x = torch.nan_to_num(xy)
    sxx, sxy, syy = Sigma[:, 0], Sigma[:, 1], Sigma[:, 2]
    det = sxx * syy - sxy * sxy
    d0 = x[:, 0:1] - mu[None, :, 0]
    d1 = x[:, 1:2] - mu[None, :, 1]
    q = (syy * d0 * d0 - 2.0 * sxy * d0 * d1 + sxx * d1 * d1) / det
    a1 = torch.log(p) - math.log(2.0 * math.pi) - 0.5 * torch.log(det)
    return torch.where(flag[:, None] == 1, a1 - 0.5 * q, torch.log1p(-p)[None, :])


def _log_e_kind(kind, e0, e1, obs):
    y = obs.to(torch.float64)[:, None]
    if kind == 1:
        return y * torch.log(e0) - e0 - torch.lgamma(y + 1.0)
    return -0.5 * torch.log(2.0 * math.pi * e1) - 0.5 * (y - e0) ** 2 / e1


class _Chain:
    """The chain cut into equal segments; steps past the end of the record do nothing."""

    def __init__(self, delta, Gamma, le, segments=2048):
        T, self.K = le.shape
        self.L = max(1, -(-T // segments))
        self.nb = max(1, -(-T // self.L))
        self.T, self.delta, self.G, dev = T, delta, Gamma, le.device
        mx = le.amax(dim=1)
        self.scale = float(mx.sum())
        pad = self.nb * self.L - T
        e = torch.exp(le - mx[:, None])
        if pad:
            e = torch.cat([e, torch.ones((pad, self.K), dtype=e.dtype, device=dev)])
        self.e = e.view(self.nb, self.L, self.K)
        self.tail = pad

    def live(self, s):
        """Segments whose step s lies inside the record (all, or all but the last)."""
        return self.nb if (self.nb - 1) * self.L + s < self.T else self.nb - 1

    def products(self):
        """Per segment: matrix (K, K) with rows scaled to maximum 1, and the rows' logs."""
        N = torch.eye(self.K, dtype=torch.float64, device=self.G.device).repeat(self.nb, 1, 1)
        lr = torch.zeros((self.nb, self.K), dtype=torch.float64, device=self.G.device)
        for s in range(self.L):
            n = self.live(s)
            Y = (N[:n].reshape(-1, self.K) @ self.G).view(n, self.K, self.K) * self.e[:n, s, None, :]
            m = Y.amax(dim=2)
            N[:n] = Y / m[:, :, None]
            lr[:n] += torch.log(m)
        return N.cpu().numpy(), lr.cpu().numpy()

    def forward_messages(self, N, lr):
        """Normalised message before every segment, and ln L."""
        a = self.delta.cpu().numpy().copy()
        ll = math.log(a.sum())
        a /= a.sum()
        out = np.empty((self.nb, self.K))
        for b in range(self.nb):
            out[b] = a
            m = lr[b].max()
            a = (a * np.exp(lr[b] - m)) @ N[b]
            ll += m + math.log(a.sum())
            a /= a.sum()
        return out, ll + self.scale


def _loglik(delta, Gamma, le):
    c = _Chain(delta, Gamma, le)
    return c.forward_messages(*c.products())[1]


def _posterior(delta, Gamma, p, mu, Sigma, flag, xy):
    le = _log_e(p, mu, Sigma, flag, xy)
    c = _Chain(delta, Gamma, le)
    N, lr = c.products()
    a, ll = c.forward_messages(N, lr)
    K, nb, L = c.K, c.nb, c.L
    back = np.empty((nb, K))
    v = np.ones(K)
    for b in range(nb - 1, -1, -1):
        back[b] = v
        lv = lr[b] + np.log(N[b] @ v)
        v = np.exp(lv - lv.max())
    dev = Gamma.device
    al = torch.empty((nb, L + 1, K), dtype=torch.float64, device=dev)
    al[:, 0] = torch.as_tensor(a, device=dev)
    for s in range(L):
        n = c.live(s)
        y = (al[:n, s] @ Gamma) * c.e[:n, s]
        al[:n, s + 1] = y / y.sum(dim=1, keepdim=True)
        al[n:, s + 1] = al[n:, s]
    be = torch.as_tensor(back, device=dev)
    gam = torch.empty((nb, L, K), dtype=torch.float64, device=dev)
    xi = torch.zeros((K, K), dtype=torch.float64, device=dev)
    for s in range(L - 1, -1, -1):
        n = c.live(s)
        g = al[:n, s + 1] * be[:n]
        gam[:n, s] = g / g.sum(dim=1, keepdim=True)
        eb = c.e[:n, s] * be[:n]
        w = eb / ((al[:n, s] @ Gamma) * eb).sum(dim=1, keepdim=True)
        xi += Gamma * (al[:n, s].T @ w)
        nbk = eb @ Gamma.T
        be[:n] = nbk / nbk.amax(dim=1, keepdim=True)
    gamma = gam.reshape(-1, K)[:c.T]
    pre = al[0, 0] * be[0]
    pre = pre / pre.sum()
    f = (flag == 1).to(torch.float64)
    x = torch.nan_to_num(xy)
    cols = [torch.ones_like(f), f, f * x[:, 0], f * x[:, 1], f * x[:, 0] ** 2, f * x[:, 0] * x[:, 1],
            f * x[:, 1] ** 2]
    mom = torch.stack([gamma.T @ w for w in cols], dim=1)
    return gamma, ll, xi, pre, mom


def _viterbi_score(delta, Gamma, le):
    """Max-plus products of segments, then the segments in order."""
    T, K = le.shape
    G = torch.log(Gamma)
    nb = max(1, min(4096, 48_000_000 // K**3, T))
    L = -(-T // nb)
    nb = -(-T // L)
    mx = le.amax(dim=1)
    base = float(mx.sum())
    e = torch.zeros((nb * L, K), dtype=torch.float64, device=le.device)
    e[:T] = le - mx[:, None]
    e = e.view(nb, L, K)
    V = torch.full((nb, K, K), -math.inf, dtype=torch.float64, device=le.device)
    V[:, torch.arange(K), torch.arange(K)] = 0.0
    for s in range(L):
        n = nb if (nb - 1) * L + s < T else nb - 1
        V[:n] = (V[:n, :, :, None] + G[None, None]).amax(dim=2) + e[:n, s, None, :]
    V = V.cpu().numpy()
    d = np.log(delta.cpu().numpy())
    for b in range(nb):
        d = np.max(d[:, None] + V[b], axis=0)
    return float(d.max()) + base


def exact(case, seed):
    """What ``run`` returns, in 64 bits (None for the integer paths)."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    op = case["op"]
    if dev == "cpu" and case.get("T", case.get("T_hi", 0) * case.get("n", 1)) * case.get("K", case.get("K_hi", 0)) ** 2 > 10**8:
        return None
    h = _inputs(case, seed)

    def t(a):
        return torch.as_tensor(np.ascontiguousarray(a), device=dev)

    def one(v):
        return torch.tensor([v], dtype=torch.float64)

    if op == "kind":
        le = _log_e_kind(case["kind"], t(h.e0), t(h.e1), t(h.obs))
        return one(_loglik(t(h.delta), t(h.Gamma), le))
    if op == "batch":
        out = []
        for i in range(case["n"]):
            K, T = int(h["K"][i]), int(h["T"][i])
            b = h["params"][int(h["param_off"][i]):]
            o = int(h["obs_off"][i])
            le = _log_e(t(b[K + K * K:2 * K + K * K]), t(b[2 * K + K * K:4 * K + K * K].reshape(K, 2)),
                        t(b[4 * K + K * K:7 * K + K * K].reshape(K, 3)), t(h["flag"][o:o + T]), t(h["xy"][o:o + T]))
            out.append(_loglik(t(b[:K]), t(b[K:K + K * K].reshape(K, K)), le))
        return torch.tensor(out, dtype=torch.float64)
    prm, obs = h
    delta, Gamma, p, mu, Sigma = (t(a) for a in (prm.delta, prm.Gamma, prm.p, prm.mu, prm.Sigma))
    flag, xy = t(obs.flag), t(obs.xy)
    if op == "loglik":
        return one(_loglik(delta, Gamma, _log_e(p, mu, Sigma, flag, xy)))
    if op == "viterbi":
        return None, None, one(_viterbi_score(delta, Gamma, _log_e(p, mu, Sigma, flag, xy)))
    gamma, ll, xi, pre, mom = _posterior(delta, Gamma, p, mu, Sigma, flag, xy)
    if op == "posterior":
        return {"gamma": gamma, "loglik": one(ll), "xi": xi, "pre": pre, "mom": mom}
    n, n1 = mom[:, 0], mom[:, 1]
    m = mom[:, 2:4] / n1[:, None]
    S = torch.stack([mom[:, 4] / n1 - m[:, 0] ** 2, mom[:, 5] / n1 - m[:, 0] * m[:, 1],
                     mom[:, 6] / n1 - m[:, 1] ** 2], dim=1)
    new = torch.cat([pre, (xi / xi.sum(dim=1, keepdim=True)).reshape(-1), n1 / n, m.reshape(-1), S.reshape(-1)])
    return new, one(ll)
