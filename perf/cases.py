"""The calls of the Elastic Shadow Pricing library whose speed is followed.

Each case is one call sequence that a scheduler makes through
``paper_2608_07971_amd.Solver``, at sizes from the paper's own scale (tens of
jobs) to the largest tables of the benchmark:

  solve     the price loop and the re-selection at the final prices
  granular  one iteration through the separate entry points (select, demand, update)
  epoch     a scheduling epoch: the effective capacity of the pending queue,
            then a warm-started price loop with a stop tolerance
  schedule  the outer rounds (price loop, first-fit packing, co-location checks)
  nearest   the profile fallback: nearest stored profile of each query's job type

Every result of the library is defined bit for bit (binary64 scores in a fixed
order, exact demand sums), so the tolerance is "exact" throughout; ``exact``
recomputes the results with plain torch and Python integers.

Inputs follow the job families of the benchmark's generators: training
families over a grid of GPU counts, compute shares, memory scales, AMP and
micro-batch sizes, a third of inference families in ragged tables.  They are
drawn on the GPU from the seed alone.  Units: "abs" keeps GPUs and gigabytes
(what packing onto GPUs needs), "share" rescales every resource to one unit
per job, where one step size serves all resources and prices settle.
"""
import math
import types

import numpy as np
import torch

import paper_2608_07971_amd as esp

_DEV = "cuda:0"


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------

def _solve(**kw):
    c = {"kind": "solve", "B": 1, "N": 64, "K": 8, "R": 4, "T": 200, "units": "share", "pen": False, "mask": False,
         "trace": False, "tol": 0.0}
    c.update(kw)
    return c


def listed():
    return [
        # the paper's scale, tens of jobs on 64 GPUs: one launch, a chain of short iterations
        _solve(name="solve_tiny", N=64, K=8, R=4, T=200, units="abs"),
        # a department's cluster: 4,096 jobs, still a chain of short iterations over a small table
        _solve(name="solve_small", N=4096, K=32, R=4, T=500, units="abs"),
        # an ordinary data centre: a table of tens of MB, larger than L2 and smaller than the memory-side cache
        _solve(name="solve_mid", N=12000, K=64, R=8, T=200),
        # the benchmark's headline table (604 MB read every iteration)
        _solve(name="solve_large", N=262144, K=64, R=8, T=100),
        # profile families of every size (CSR), the benchmark's ragged table
        _solve(name="solve_ragged", N=1048576, K=0, R=6, T=50),
        # many independent clusters priced at once, running jobs pay to switch and to interfere
        _solve(name="solve_batched", B=64, N=4096, K=64, R=6, T=50, units="abs", pen=True),
        # a caller's own loop over the separate entry points, some configurations ruled out
        {"name": "granular", "kind": "granular", "B": 16, "N": 8192, "K": 32, "R": 6, "mask": True, "pen": False,
         "units": "share"},
        # a scheduling epoch: reserve for the pending queue, then a few warm iterations
        {"name": "epoch", "kind": "epoch", "B": 1, "N": 262144, "NQ": 131072, "K": 0, "KQ": 0, "R": 6, "T": 8,
         "tol": 1e-3},
        # outer rounds on one 512-GPU cluster
        {"name": "schedule_small", "kind": "schedule", "B": 1, "N": 4096, "K": 32, "R": 4, "T": 5, "rounds": 3,
         "gpus": 512},
        # outer rounds on many clusters at once
        {"name": "schedule_batched", "kind": "schedule", "B": 32, "N": 4096, "K": 64, "R": 6, "T": 5, "rounds": 3,
         "gpus": 768},
        # a million unprofiled configurations against a large profile store
        {"name": "nearest_store", "kind": "nearest", "N": 262144, "K": 0, "R": 6, "Q": 1048576, "store": True},
        # a batch of queries against the price loop's own table
        {"name": "nearest_columns", "kind": "nearest", "N": 500, "K": 0, "R": 5, "Q": 20000, "store": False},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_KS = (0, 0, 4, 8, 16, 32, 64, 64, 5, 12, 33, 100, 198)     # 0: ragged families of 1..256


def _mean_k(k):
    return k if k else 12.5


def draw(rng):
    kind = rng.choice(("solve", "solve", "solve", "granular", "epoch", "schedule", "nearest"))
    R = rng.randint(2, 8)
    K = rng.choice(_KS)
    if kind == "solve":
        B = rng.choice((1, 1, 1, 1, 3, 16, _log_int(rng, 2, 256)))
        entries = math.exp(rng.uniform(math.log(300.0), math.log(4.0e6)))
        N = max(8, int(entries / _mean_k(K) / B))
        T = max(3, min(_log_int(rng, 3, 500), int(2.0e9 / (B * N * _mean_k(K)))))
        return _solve(B=B, N=N, K=K, R=R, T=T, units=rng.choice(("abs", "share")), pen=rng.random() < 0.3,
                      mask=rng.random() < 0.3, trace=rng.random() < 0.15, tol=rng.choice((0.0, 0.0, 1e-3)))
    if kind == "granular":
        B = rng.choice((1, 1, 16, _log_int(rng, 2, 100)))
        entries = math.exp(rng.uniform(math.log(1000.0), math.log(4.0e6)))
        return {"kind": "granular", "B": B, "N": max(5, int(entries / _mean_k(K) / B)), "K": K, "R": R,
                "mask": rng.random() < 0.5, "pen": rng.random() < 0.3, "units": rng.choice(("abs", "share"))}
    if kind == "epoch":
        B = rng.choice((1, 1, 4, 20))
        KQ = rng.choice(_KS)
        N = max(16, int(math.exp(rng.uniform(math.log(2000.0), math.log(2.0e6))) / _mean_k(K) / B))
        NQ = max(4, int(math.exp(rng.uniform(math.log(500.0), math.log(2.0e6))) / _mean_k(KQ) / B))
        return {"kind": "epoch", "B": B, "N": N, "NQ": NQ, "K": K, "KQ": KQ, "R": R, "T": rng.randint(3, 8),
                "tol": 1e-3}
    if kind == "schedule":
        B = rng.choice((1, 1, 1, 5, 32))
        K = rng.choice((8, 16, 32, 64, 0, 12))
        N = min(_log_int(rng, 40, 8000), int(3.0e6 / _mean_k(K) / B))
        return {"kind": "schedule", "B": B, "N": N, "K": K, "R": max(R, 3), "T": rng.randint(3, 6),
                "rounds": rng.randint(1, 3), "gpus": _log_int(rng, 16, 2048)}
    K = rng.choice((0, 0, 12, 64, 198))
    return {"kind": "nearest", "N": _log_int(rng, 10, 3.0e6 / _mean_k(K)), "K": K, "R": R,
            "Q": _log_int(rng, 1, 1000000), "store": rng.random() < 0.6}


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

_MS = (1.0, 0.8, 0.6, 0.45)


class _Draws:
    def __init__(self, seed, field):
        self.g = torch.Generator(device=_DEV)
        self.g.manual_seed((int(seed) * 1000003 + field) & 0x7FFFFFFFFFFFFFFF)

    def uniform(self, *shape):
        return torch.rand(*shape, generator=self.g, device=_DEV, dtype=torch.float64)

    def normal(self, *shape):
        return torch.randn(*shape, generator=self.g, device=_DEV, dtype=torch.float64)


def _offsets(r, N, K):
    if K:
        return torch.arange(N + 1, device=_DEV, dtype=torch.int64) * K
    u = r.uniform(N)
    sizes = (1 + torch.floor(torch.log1p(-u) / math.log(0.92)).to(torch.int64)).clamp_(1, 256)
    return torch.cat([torch.zeros(1, device=_DEV, dtype=torch.int64), torch.cumsum(sizes, 0)])


def _families(r, B, N, K, R):
    """Offsets [N+1], utility [B, nnz] and demand [B, nnz, R], float32 on the GPU."""
    off = _offsets(r, N, K)
    nnz = int(off[-1])
    sizes = off[1:] - off[:-1]
    jl = torch.repeat_interleave(torch.arange(N, device=_DEV), sizes)
    kk = torch.arange(nnz, device=_DEV) - off[jl]
    util = torch.empty((B, nnz), dtype=torch.float32, device=_DEV)
    dem = torch.empty((B, nnz, R), dtype=torch.float32, device=_DEV)
    for b in range(B):
        if 0 < K <= 64:
            pt = 4 * ((kk * 64) // K) + 3                     # every micro-batch at its largest
            infer = None
        elif K > 64:
            pt = (kk * 256) // K
            infer = None
        else:
            o = torch.floor(256.0 * r.uniform(N)).to(torch.int64)
            st = 2 * torch.floor(128.0 * r.uniform(N)).to(torch.int64) + 1
            pt = (o[jl] + kk * st[jl]) % 256
            infer = (r.uniform(N) < 1.0 / 3.0)[jl]
        base = torch.exp(0.5 * r.normal(N))[jl]
        mem = (8.0 + 62.0 * r.uniform(N))[jl]
        pcie = (0.05 + 0.45 * r.uniform(N))[jl]
        nvl = (0.05 + 0.55 * r.uniform(N))[jl]
        cpu = torch.floor(2.0 + 7.0 * r.uniform(N))[jl]
        io = (0.01 + 0.19 * r.uniform(N))[jl]
        g = torch.exp2((pt // 64).to(torch.float64)).round()
        ms = torch.tensor(_MS, device=_DEV, dtype=torch.float64)[(pt // 16) % 4]
        s = 0.5 + 0.5 * ((pt // 8) % 2).to(torch.float64)
        a = ((pt // 4) % 2).to(torch.float64)
        mb = torch.exp2((pt % 4).to(torch.float64)).round() / 8.0
        f = 0.6 + 0.4 * r.uniform(nnz)
        u = base * g ** 0.85 * (1.0 - 0.625 * (1.0 - ms)) * s ** 0.7 * (1.0 + 0.3 * a) * mb ** 0.25 * f
        cols = [g, mem * ms * (1.0 - 0.25 * a) * (0.5 + 0.5 * mb) * g ** 0.4, g * s, 16.0 * g, pcie * g * s,
                nvl * g * (1.5 - 0.5 * ms), cpu * g, io * torch.sqrt(g) * (1.0 + 0.3 * a)]
        if infer is not None:
            bs = (pt + 1).to(torch.float64)
            sat = (16.0 + 112.0 * r.uniform(N))[jl]
            w = (4.0 + 16.0 * r.uniform(N))[jl]
            kv = (0.02 + 0.18 * r.uniform(N))[jl]
            u = torch.where(infer, 50.0 * base * bs / (1.0 + bs / sat), u)
            one = torch.ones_like(bs)
            icols = [one, w + kv * bs, (0.2 + 0.8 * bs / 256.0).clamp(max=1.0), 8.0 + 0.05 * bs, pcie * bs / 256.0,
                     nvl * one, 2.0 * one, io * bs / 64.0]
            cols = [torch.where(infer, i, c) for i, c in zip(icols, cols)]
        if R == 6:
            cols = [cols[i] for i in (0, 1, 2, 3, 4, 6)]
        util[b] = u.to(torch.float32)
        for i in range(R):
            dem[b, :, i] = cols[i].to(torch.float32)
    return off, util, dem


def _segment(x, off, how):
    """[B, nnz] -> [B, N] minimum or maximum of each family."""
    B, N = x.shape[0], off.numel() - 1
    K = int(off[1])
    if N * K == x.shape[1] and bool(((off[1:] - off[:-1]) == K).all()):
        v = x.view(B, N, K)
        return v.amin(2) if how == "amin" else v.amax(2)
    jl = torch.repeat_interleave(torch.arange(N, device=x.device), off[1:] - off[:-1]).expand(B, -1)
    start = math.inf if how == "amin" else -math.inf
    out = torch.full((B, N), start, dtype=x.dtype, device=x.device)
    return out.scatter_reduce_(1, jl, x, how)


def _inputs(case, seed):
    """Everything a case's calls read, before the library sees it (GPU tensors and numbers)."""
    kind = case["kind"]
    B, N, R = case.get("B", 1), case["N"], case["R"]
    r = _Draws(seed, 1)
    p = types.SimpleNamespace(B=B, N=N, R=R)
    p.off, p.utility, p.demand = _families(r, B, N, case["K"], R)
    p.nnz = int(p.off[-1])
    p.K = case["K"] or None
    units = case.get("units", "share" if kind == "epoch" else "abs")
    # capacity: between the smallest and the largest total demand of each resource, binding for
    # ordinary prices; outer rounds: the cluster's GPUs (80 GB, 512 GB of host memory, 16 cores each)
    lo = torch.stack([_segment(p.demand[:, :, i], p.off, "amin").double().sum(1) for i in range(R)], 1)
    hi = torch.stack([_segment(p.demand[:, :, i], p.off, "amax").double().sum(1) for i in range(R)], 1)
    cap = lo + (0.3 + 0.3 * r.uniform(B, 1)) * (hi - lo)
    if units == "share":
        p.demand *= (float(N) / cap).to(torch.float32)[:, None, :]
        cap = torch.full_like(cap, float(N))
        p.eta0 = np.full(B, 2.0 / N)
    else:
        p.eta0 = np.array([0.005, 0.01, 0.02])[torch.floor(3.0 * r.uniform(B)).long().clamp_(max=2).cpu().numpy()]
    p.rule = esp.ESP_STEP_INV_SQRT
    p.current = p.switch_cost = p.penalty = p.feasible = None
    if kind == "schedule":
        G = torch.floor(case["gpus"] * (0.75 + 0.25 * r.uniform(B))).clamp_(min=1)
        G[0] = case["gpus"]
        per = torch.tensor([1.0, 80.0, 1.0, 512.0, 1.0, 16.0 if R == 6 else 1.0, 16.0, 1.0], device=_DEV,
                           dtype=torch.float64)[:R]
        cap = G[:, None] * per
        p.gpus = G.to(torch.int32).cpu().numpy()
        share = p.demand[:, :, 2] / p.demand[:, :, 0].clamp(min=1.0)
        p.sensitivity = (0.6 * r.uniform(B, p.nnz)).to(torch.float32)
        p.pressure = (share * (0.5 + 0.5 * r.uniform(B, p.nnz))).to(torch.float32)
        p.tau_base = 1.1 + 0.3 * r.uniform(B, N)
        p.penalty = torch.zeros((B, p.nnz), dtype=torch.float32, device=_DEV)
    p.capacity = cap.cpu().numpy()
    sizes = p.off[1:] - p.off[:-1]
    if case.get("pen"):
        cur = torch.floor(r.uniform(B, N) * sizes).long()
        p.current = torch.where(r.uniform(B, N) < 0.8, cur, -1).to(torch.int32)
        p.switch_cost = np.full(B, 0.05)
        p.penalty = (0.2 * r.uniform(B, p.nnz)).to(torch.float32)
    if case.get("mask"):
        ok = r.uniform(B, p.nnz) >= 0.1
        ok[:, p.off[:-1]] = True                              # every family keeps its first configuration
        p.feasible = ok.to(torch.uint8)
    # prices a warm start carries over (all zero in a cold solve)
    scale = p.utility.double().mean(1, keepdim=True) / p.demand.double().mean(1)
    p.lam0 = (r.uniform(B, R) * 0.3 * scale if kind in ("granular", "epoch") else torch.zeros_like(cap)).contiguous()
    if kind == "epoch":
        q = _Draws(seed, 2)
        p.queue = types.SimpleNamespace(B=B, N=case["NQ"], R=R, K=case["KQ"] or None)
        p.queue.off, p.queue.utility, p.queue.demand = _families(q, B, case["NQ"], case["KQ"], R)
        p.queue.demand *= (float(N) / (lo + 0.5 * (hi - lo))).to(torch.float32)[:, None, :]
        p.queue.feasible = None
        p.pending = (q.uniform(B, case["NQ"]) < 0.5).to(torch.uint8)
    if kind == "nearest":
        q = _Draws(seed, 3)
        Q = case["Q"]
        p.family = torch.floor(N * q.uniform(Q)).long().clamp_(max=N - 1)
        k = torch.minimum(torch.floor(sizes[p.family] * q.uniform(Q)).long(), sizes[p.family] - 1)
        factor = torch.exp(0.25 * q.normal(Q, R))
        factor[q.uniform(Q) < 0.1] = 1.0                      # exact copies of a stored vector
        p.query = (p.demand[0, p.off[p.family] + k].double() * factor).to(torch.float32)[None].contiguous()
        p.family = p.family.to(torch.int32)[None].contiguous()
    return p


def _host(x):
    return None if x is None else x if isinstance(x, np.ndarray) else x.cpu().numpy()


def _instance(p, like=None):
    """The host arrays that esp_create reads."""
    like = like or p
    return types.SimpleNamespace(
        offsets=_host(p.off), utility=_host(p.utility), demand=_host(p.demand), capacity=like.capacity,
        eta0=like.eta0, rule=esp.ESP_STEP_INV_SQRT, feasible=_host(p.feasible), dense_k=p.K,
        current=_host(getattr(p, "current", None)), switch_cost=getattr(p, "switch_cost", None),
        penalty=_host(getattr(p, "penalty", None)))


def prepare(case, seed):
    kind = case["kind"]
    p = _inputs(case, seed)
    s = types.SimpleNamespace(case=case)
    flags = esp.ESP_OPT_PROFILE_STORE if case.get("store") else 0
    s.solver = esp.Solver(_instance(p), _DEV, flags=flags)
    s.lam0, s.lam = p.lam0, p.lam0.clone()
    if kind == "epoch":
        s.queue = esp.Solver(_instance(p.queue, like=p), _DEV)
        s.pending = p.pending
    if kind == "schedule":
        s.model = types.SimpleNamespace(gpus=p.gpus, gpu_memory=80.0, gpu_compute=1.0, r_gpus=0, r_mem=1, r_sm=2,
                                        sensitivity=p.sensitivity, pressure=p.pressure, tau_base=p.tau_base,
                                        beta=0.5, beta_max=0.1, u_target=0.8, kappa=0.5)
    if kind == "nearest":
        s.family, s.query = p.family, p.query
    return s


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def run(state):
    case, s, kind = state.case, state.solver, state.case["kind"]
    if kind == "nearest":
        nearest, estimate = s.nearest_profile(state.family, state.query)
        return {"nearest": nearest, "estimate": estimate}
    state.lam.copy_(state.lam0)
    if kind == "solve":
        return s.solve(state.lam, case["T"], tol=case["tol"], trace=case["trace"])
    if kind == "granular":
        choice = s.score_select(state.lam)
        U = s.reduce_demand(choice)
        s.update_prices(U, 3, state.lam)
        return {"choice": choice, "U": U, "lam": state.lam}
    if kind == "epoch":
        ceff = s.effective_capacity(state.queue, 0.5, state.pending)
        out = s.solve(state.lam, case["T"], tol=case["tol"])
        out["ceff"] = ceff
        return out
    out = s.schedule(state.model, state.lam, case["rounds"], case["T"])
    return {k: out[k] for k in ("choice", "gpu_jobs", "rounds", "violations", "lam")}


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------

_ON_CHIP = 128 << 20     # vector registers of the card: a table below this needs one read per solve


def work(case):
    kind, B, N, R = case["kind"], case.get("B", 1), case["N"], case["R"]
    entries = B * N * _mean_k(case["K"])
    cols = 1 + R + (1 if case.get("pen") or kind == "schedule" else 0)
    table = 4.0 * entries * cols
    per_pass = entries * (2 * R + 1)

    def loop(T):
        reads = T + 1 if table > _ON_CHIP else 1
        return reads * table + 4.0 * B * N, (T + 1) * per_pass

    if kind == "solve":
        byts, flops = loop(case["T"])
    elif kind == "granular":
        byts, flops = table + B * N * (8.0 + 4.0 * R), per_pass
    elif kind == "epoch":
        byts, flops = loop(case["T"])
        q = B * case["NQ"] * _mean_k(case["KQ"])
        byts, flops = byts + 4.0 * q * R + B * case["NQ"], flops + q * R
    elif kind == "schedule":
        byts, flops = loop(case["T"])
        byts, flops = case["rounds"] * (byts + 20.0 * B * N), case["rounds"] * flops
    else:
        byts = case["Q"] * (12.0 + 4.0 * R + 4.0 * (1 + R) * _mean_k(case["K"]))
        byts = min(byts, table + case["Q"] * (12.0 + 4.0 * R))
        flops = case["Q"] * _mean_k(case["K"]) * 3.0 * R
    return {"bytes": byts, "flops": flops}


def tolerance(case):
    # binary64 results in a fixed order of operations and exact sums: every bit is defined
    return "exact"


# ---------------------------------------------------------------------------
# The same results from plain torch and Python integers
# ---------------------------------------------------------------------------

def _exact_sum(x):
    """Correctly rounded sum of the float32 values of each row of x [rows, n]: the values as
    integer multiples of the row's lowest bit, in 40-bit halves."""
    out = []
    for row in x.double():
        low = int(torch.frexp(row[row > 0]).exponent.min()) - 24 if bool((row > 0).any()) else 0
        v = row * 2.0 ** -low
        hi = torch.floor(v * 2.0 ** -40)
        total = (int(hi.to(torch.int64).sum()) << 40) + int((v - hi * 2.0 ** 40).to(torch.int64).sum())
        out.append(math.ldexp(float(total), low) if total < 1 << 53 else float(total * 2 ** low) if low >= 0
                   else total / (1 << -low))
    return np.array(out)


class _Market:
    """Select, demand and price loop of one problem in binary64."""

    def __init__(self, p):
        self.p = p
        self.u = p.utility.double()
        if p.feasible is not None:
            self.u = torch.where(p.feasible.bool(), self.u, -math.inf)
        self.pen = None if p.penalty is None else p.penalty.double()
        sizes = p.off[1:] - p.off[:-1]
        self.jl = torch.repeat_interleave(torch.arange(p.N, device=_DEV), sizes)
        self.k = torch.arange(p.nnz, device=_DEV) - p.off[self.jl]
        self.idx = torch.arange(p.nnz, device=_DEV)
        self.move = None
        if p.current is not None:
            cur = p.current.long()[:, self.jl]
            self.move = (cur >= 0) & (cur != self.k)

    def select(self, lam):
        lam = torch.as_tensor(lam, device=_DEV)
        rent = self.p.demand[:, :, 0].double() * lam[:, 0:1]
        for i in range(1, self.p.R):
            rent = rent + self.p.demand[:, :, i].double() * lam[:, i:i + 1]
        s = self.u - rent
        if self.move is not None:
            s = torch.where(self.move, s - torch.as_tensor(self.p.switch_cost, device=_DEV)[:, None], s)
        if self.pen is not None:
            s = s - self.pen
        best = _segment(s, self.p.off, "amax")[:, self.jl]
        first = torch.where(s == best, self.idx, self.p.nnz)
        return _segment(first.double(), self.p.off, "amin").long() - self.p.off[:-1]

    def demand(self, choice):
        e = (choice.long() + self.p.off[:-1])[:, :, None].expand(-1, -1, self.p.R)
        d = torch.gather(self.p.demand, 1, e)                 # [B, N, R]
        B, N, R = d.shape
        return _exact_sum(d.permute(0, 2, 1).reshape(B * R, N)).reshape(B, R)

    def step(self, lam, U, cap, t):
        eta = self.p.eta0 / np.sqrt(float(t))
        x = lam + eta[:, None] * (U - cap)
        return np.where(x > 0.0, x, 0.0)

    def solve(self, lam, T, cap, tol, trace=False):
        lam, B = lam.copy(), self.p.B
        live, done = np.ones(B, bool), np.zeros(B, np.int32)
        tl, tu = np.full((max(T, 1), B, self.p.R), np.nan), np.full((max(T, 1), B, self.p.R), np.nan)
        for t in range(1, T + 1):
            if not live.any():
                break
            U = self.demand(self.select(lam))
            new = self.step(lam, U, cap, t)
            ok = (np.abs(new - lam) <= tol * np.maximum(lam, 1.0)).all(1) & (tol > 0.0)
            tl[t - 1, live], tu[t - 1, live] = new[live], U[live]
            lam[live] = new[live]
            done[live] = t
            live &= ~ok
        choice = self.select(lam)
        out = {"iters_done": done, "choice": choice.to(torch.int32), "U": self.demand(choice), "lam": lam}
        if trace:
            out["tr_lam"], out["tr_U"] = tl, tu
        return out


def _pack(p, b, choice):
    """First fit of one cluster: jobs of each GPU [G][4]."""
    G, e = int(p.gpus[b]), p.off[:-1] + choice.long()
    d = p.demand[b, e, :3].double().cpu().numpy()
    mem, sm, cnt = np.full(G, 80.0), np.full(G, 1.0), np.zeros(G, np.int64)
    occ = np.full((G, 4), -1, np.int64)
    failed = []
    for j in range(p.N):
        g = d[j, 0]
        if not (1.0 <= g <= 8.0 and g == math.floor(g)):
            continue
        nm, ns = d[j, 1] / g, d[j, 2] / g
        if any(g >= f[0] and nm >= f[1] and ns >= f[2] for f in failed):
            continue                                          # room only shrinks
        at = np.flatnonzero((cnt < 4) & (mem >= nm) & (sm >= ns))[:int(g)]
        if at.size < g:
            failed = [f for f in failed if not (f[0] >= g and f[1] >= nm and f[2] >= ns)] + [(g, nm, ns)]
            continue
        mem[at] -= nm
        sm[at] -= ns
        occ[at, cnt[at]] = j
        cnt[at] += 1
    return occ


def _check(p, b, choice, occ):
    """Violating pairs and each job's largest excess slowdown."""
    e = (p.off[:-1] + choice.long())
    sa, pr = p.sensitivity[b, e].double().cpu().numpy(), p.pressure[b, e].double().cpu().numpy()
    G = occ.shape[0]
    add = min(0.5 * (float((occ[:, 0] >= 0).sum()) / float(G) / 0.8 - 1.0), 0.1)
    tau = p.tau_base[b].cpu().numpy() + add
    inc, bad = np.zeros(p.N), 0
    for x in range(4):
        for y in range(x + 1, 4):
            at = occ[:, y] >= 0
            jx, jy = occ[at, x], occ[at, y]
            ox = (1.0 + sa[jx] * pr[jy]) - tau[jx]
            oy = (1.0 + sa[jy] * pr[jx]) - tau[jy]
            np.maximum.at(inc, jx, ox)
            np.maximum.at(inc, jy, oy)
            bad += int(((ox > 0.0) | (oy > 0.0)).sum())
    return bad, inc


def _schedule(p, case):
    B, N, gmax = p.B, p.N, int(p.gpus.max())
    lam = p.lam0.cpu().numpy().copy()
    choice = np.zeros((B, N), np.int32)
    jobs = np.full((B, gmax, 4), -1, np.int32)
    rounds, violations = np.zeros(B, np.int32), np.zeros(B, np.int32)
    live = np.ones(B, bool)
    p.penalty = torch.zeros_like(p.penalty)
    for m in range(1, case["rounds"] + 1):
        out = _Market(p).solve(lam, case["T"], p.capacity, 0.0)
        for b in np.flatnonzero(live):
            c = out["choice"][b]
            lam[b], choice[b] = out["lam"][b], c.cpu().numpy()
            occ = _pack(p, b, c)
            violations[b], inc = _check(p, b, c, occ)
            jobs[b, :] = -1
            jobs[b, :occ.shape[0]] = occ
            rounds[b] = m
            e = (p.off[:-1] + c.long())
            more = torch.as_tensor(inc, device=_DEV)
            raised = (p.penalty[b, e].double() + 0.5 * more).to(torch.float32)
            p.penalty[b, e] = torch.where(more > 0.0, raised, p.penalty[b, e])
            live[b] = violations[b] > 0
        if not live.any():
            break
    return {"choice": choice, "gpu_jobs": jobs, "rounds": rounds, "violations": violations, "lam": lam}


def _nearest(p):
    Q = p.family.shape[1]
    nearest = torch.empty(Q, dtype=torch.int32, device=_DEV)
    step = 1 << 16
    for q0 in range(0, Q, step):
        f = p.family[0, q0:q0 + step].long()
        v = p.query[0, q0:q0 + step].double()
        size = p.off[f + 1] - p.off[f]
        k = torch.arange(int(size.max()), device=_DEV)
        e = p.off[f][:, None] + torch.minimum(k[None, :], size[:, None] - 1)
        d = p.demand[0, e].double()                           # [q, k, R]
        x = v[:, None, 0] - d[:, :, 0]
        acc = x * x
        for i in range(1, p.R):
            x = v[:, None, i] - d[:, :, i]
            acc = acc + x * x
        acc = torch.where(k[None, :] < size[:, None], acc, math.inf)
        first = torch.where(acc == acc.amin(1, keepdim=True), k[None, :], 1 << 30)
        nearest[q0:q0 + step] = first.amin(1).to(torch.int32)
    est = p.utility[0, p.off[p.family[0].long()] + nearest.long()]
    return {"nearest": nearest[None], "estimate": est[None]}


def exact(case, seed):
    kind, p = case["kind"], _inputs(case, seed)
    if kind == "nearest":
        return _nearest(p)
    if kind == "schedule":
        return _schedule(p, case)
    lam = p.lam0.cpu().numpy()
    m = _Market(p)
    if kind == "solve":
        return m.solve(lam, case["T"], p.capacity, case["tol"], case["trace"])
    if kind == "granular":
        choice = m.select(lam)
        U = m.demand(choice)
        return {"choice": choice.to(torch.int32), "U": U, "lam": m.step(lam, U, p.capacity, 3)}
    q = p.queue
    least = torch.stack([_segment(q.demand[:, :, i], q.off, "amin") for i in range(p.R)], 1)     # [B, R, NQ]
    least = torch.where(p.pending.bool()[:, None, :], least, 0.0).reshape(p.B * p.R, q.N)
    ceff = p.capacity - 0.5 * _exact_sum(least).reshape(p.B, p.R)
    out = m.solve(lam, case["T"], ceff, case["tol"])
    out["ceff"] = ceff
    return out
