"""Performance cases of the GEM commit pipeline: the calls that programs make,
through the binding of the C ABI (``paper_1805_08469_amd.gem``), each at the
size and with the options it is used with.

A case is a dict of plain values.  ``kind`` says which calls a pass makes:

  run      gem_sim_run of T commits, then theta and the rows of the workers that
           committed last are read
  record   the same with the histograms of the scale factors recorded and read
  segment  gem_sim_run with one scale factor per segment (norms)
  batch    gem_commit_batch of K queued updates, then the same reads
  loop     a worker loop: gem_generate and gem_commit for each of T commits

A pass continues where the last one stopped (the clock runs on); a new state
starts at theta = 0, as the workloads do.  Every value is the same bits
however the commits are scheduled on the GPU, so the tolerance is "exact".
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_1805_08469_amd import gem as G

MU, EPS = 0.9, 1e-16


def _case(name, kind, P, n, T, K, law=G.GEM_LAW_EXP, p0=0.0, p1=0.0, sigma=0.02, lr=0.01,
          bf16=False, proxy="local", rule="gem", kappa=1.0, pull="post", nseg=0):
    c = dict(kind=kind, P=P, n=n, T=T, K=K, law=law, p0=p0, p1=p1, sigma=sigma, lr=lr, bf16=bf16,
             proxy=proxy, rule=rule, kappa=kappa, pull=pull, nseg=nseg)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The tiny workload: a toy model, commits asked for one at a time; launches and
        # latencies are all there is to it.
        _case("tiny-run", "run", 4096, 4, 2000, 1, sigma=0.1),
        # The small workload: a small CNN's parameters, one commit per pass; the whole
        # state fits the Infinity Cache.
        _case("small-run", "run", 1_200_000, 20, 1000, 1, G.GEM_LAW_EXP_UNIFORM_MEAN, 0.8, 1.2,
              sigma=0.05, lr=0.005),
        # ResNet-18's parameters with 50 workers, passes of 8.
        _case("resnet18-run", "run", 11_700_000, 50, 400, 8, sigma=0.05),
        # The headline workload: 25M parameters, 100 workers of unequal speed, passes of 32
        # (a fifth of its 5000 commits).
        _case("headline-run", "run", 25_000_000, 100, 1000, 32, G.GEM_LAW_EXP_LOGNORMAL_MEAN, 0.0,
              0.5),
        # The same with one moment shared by all workers.
        _case("shared-moment-run", "run", 25_000_000, 100, 1000, 32, G.GEM_LAW_EXP_LOGNORMAL_MEAN,
              0.0, 0.5, proxy="global"),
        # The large workload: 124M parameters, heavy-tailed workers that send bfloat16
        # updates; a short run (64 workers, so that three such states fit one card).
        _case("large-bf16-run", "run", 124_000_000, 64, 160, 16, G.GEM_LAW_PARETO, 1.5, 1.0 / 3.0,
              bf16=True),
        # A rule set by its modes instead of the defaults: the higher-energy proxy
        # (kappa = 2), an odd size.
        _case("kappa-run", "run", 3_141_593, 30, 500, 16, sigma=0.05, kappa=2.0),
        # The scale factors followed over a run: one histogram per commit.
        _case("recorded-run", "record", 11_700_000, 50, 320, 32, sigma=0.05),
        # The master's own work on real updates: a batch of 32 queued float32 updates.
        _case("batch-f32", "batch", 25_000_000, 100, 32, 32, G.GEM_LAW_EXP_LOGNORMAL_MEAN, 0.0,
              0.5),
        # A short batch of bfloat16 updates, odd size.
        _case("batch-bf16", "batch", 11_689_513, 50, 8, 8, bf16=True),
        # Workers served one by one: each generates its update at its snapshot and commits it.
        _case("worker-loop", "loop", 1_200_000, 20, 40, 1, sigma=0.05, lr=0.005),
        # One scale factor per tensor of a model, from norms: 62 segments.
        _case("tensor-norms", "segment", 11_700_000, 50, 100, 1, sigma=0.05, nseg=62),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


MOST = 1.9e10        # element-commits of a drawn case; the largest listed ones have 2.5e10
MOST_ROWS = 3.2e9    # elements of its snapshot (and of its moment) rows


def draw(rng: random.Random):
    kind = rng.choice(["run"] * 5 + ["record", "segment", "batch", "batch", "loop"])
    P = int(_log(rng, 3000, 60e6 if kind == "run" else 25e6)) | (1 if rng.random() < 0.7 else 0)
    n = int(_log(rng, 2, min(100, max(3, MOST_ROWS / P)) + 1))
    law, p0, p1 = rng.choice([(G.GEM_LAW_EXP, 0.0, 0.0), (G.GEM_LAW_EXP_UNIFORM_MEAN, 0.8, 1.2),
                              (G.GEM_LAW_EXP_LOGNORMAL_MEAN, 0.0, 0.5),
                              (G.GEM_LAW_PARETO, 1.5, 1.0 / 3.0)])
    kw = dict(law=law, p0=p0, p1=p1, sigma=rng.choice([0.02, 0.05, 0.1]),
              lr=rng.choice([0.005, 0.01]), bf16=rng.random() < 0.3)
    if kind in ("run", "record"):
        T = int(min(_log(rng, 100, 2000), MOST / P))
        K = rng.choice([1, 8, 16, 32]) if kind == "run" else rng.choice([8, 32])
        if kind == "run":
            kw.update(rng.choice([{}, {}, {}, {"proxy": "global"}, {"kappa": 2.0},
                                  {"rule": "adaptive"}, {"pull": "pre"}]))
        return _case("", kind, P, n, max(T, 16), K, **kw)
    if kind == "segment":
        T = int(max(8, min(_log(rng, 20, 200), 2e9 / P)))
        nseg = rng.choice([1, 1, 62, 161])
        return _case("", kind, P, n, T, 1, nseg=nseg, **kw)
    if kind == "batch":
        K = rng.choice([2, 4, 8, 16, 32])
        if rng.random() < 0.3:
            kw["proxy"] = "global"
        return _case("", kind, P, n, K, K, **kw)
    T = int(_log(rng, 10, 100))
    return _case("", kind, P, n, T, 1, **kw)


# ---- inputs --------------------------------------------------------------------
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _problem(case, seed):
    """Curvatures h ~ LogUniform[1e-4, 1] and minimiser theta* ~ N(0, 1), on the device."""
    g = _generator(1000003 * seed + 1)
    P = case["P"]
    h = torch.rand(P, device="cuda", generator=g).mul_(-math.log(1e-4)).add_(math.log(1e-4)).exp_()
    ts = torch.randn(P, device="cuda", generator=g)
    return h, ts


def _updates(case, seed):
    """K queued updates of a batch, of the size a step of the workloads has."""
    g = _generator(1000003 * seed + 2)
    dt = torch.bfloat16 if case["bf16"] else torch.float32
    return [torch.randn(case["P"], device="cuda", generator=g).mul_(1e-3).to(dt)
            for _ in range(case["K"])]


def _schedule(case, seed):
    pull = G.GEM_PULL_PRE_COMMIT if case["pull"] == "pre" else G.GEM_PULL_POST_COMMIT
    return G.gem_schedule_make(case["n"], case["T"], case["law"], case["p0"], case["p1"],
                               seed=seed, pull_mode=pull)[0]


def _read_workers(case, worker):
    """The workers that committed last: four, in a worker loop two, of a batch one."""
    most = {"loop": 2, "batch": 1}.get(case["kind"], 4)
    seen = []
    for w in worker[::-1].tolist():
        if w not in seen:
            seen.append(w)
        if len(seen) == most:
            break
    return seen


def _offsets(case):
    """Tensors that grow along the model, as a CNN's do."""
    P, k = case["P"], case["nseg"]
    off = [0]
    for j in range(1, k):
        off.append(max(off[-1] + 1, int(P * (j / k) ** 2)))
    return np.array(off + [P], dtype=np.int64)


def prepare(case, seed):
    hp = G.gem_hyperparams_default()
    hp.kappa = case["kappa"]
    hp.rule = G.GEM_RULE_ADAPTIVE if case["rule"] == "adaptive" else G.GEM_RULE_GEM
    hp.pull_mode = G.GEM_PULL_PRE_COMMIT if case["pull"] == "pre" else G.GEM_PULL_POST_COMMIT
    hp.proxy_mode = G.GEM_PROXY_GLOBAL if case["proxy"] == "global" else G.GEM_PROXY_LOCAL
    hp.pi_scope = G.GEM_PI_SEGMENT if case["kind"] == "segment" else G.GEM_PI_ELEMENT
    P = case["P"]
    g = G.Gem(P, case["n"], hp, stream=torch.cuda.current_stream().cuda_stream)
    worker = _schedule(case, seed)
    read = _read_workers(case, worker)
    s = {"case": case, "gem": g, "worker": worker, "read": read,
         "theta": torch.empty(P, device="cuda"),
         "S": torch.empty(len(read), P, device="cuda"),
         "M": torch.empty(1 if case["proxy"] == "global" else len(read), P, device="cuda")}
    if case["kind"] == "batch":
        s["updates"] = _updates(case, seed)
        s["ptrs"] = [u.data_ptr() for u in s["updates"]]
    else:
        h, ts = _problem(case, seed)
        g.set_quadratic(h.cpu().numpy(), ts.cpu().numpy(), case["lr"], case["sigma"], seed,
                        bf16=case["bf16"])
    if case["kind"] == "segment":
        g.set_segments(_offsets(case))
    if case["kind"] == "loop":
        s["update"] = torch.empty(P, device="cuda",
                                  dtype=torch.bfloat16 if case["bf16"] else torch.float32)
    return s


def _ok(rc):
    if rc != G.GEM_OK:
        raise G.GemError(rc, "perf case")


def run(state):
    case, g = state["case"], state["gem"]
    worker, kind, L = state["worker"], case["kind"], G.lib()
    dt = G.GEM_BF16 if case["bf16"] else G.GEM_F32
    out = {}
    if kind in ("run", "segment"):
        g.sim_run(worker, None, case["K"])
    elif kind == "record":
        G.gem_pi_hist_start(g.h, case["T"])
        g.sim_run(worker, None, case["K"])
        out["pi_hist"] = G.gem_pi_hist_read(g.h, case["T"]).astype(np.int64)
    elif kind == "batch":
        g.commit_batch(state["ptrs"], dt, worker)
    else:
        ptr = state["update"].data_ptr()
        for w in worker.tolist():
            _ok(G.gem_generate(g.h, w, ptr, dt))
            if case["bf16"]:
                g.commit_batch([ptr], dt, [w])
            else:
                g.commit(ptr, w)
    # theta, and the rows of the workers that committed last, into device tensors
    S, M = state["S"], state["M"]
    _ok(L.gem_read_theta(g.h, state["theta"].data_ptr(), 1))
    for k, w in enumerate(state["read"]):
        _ok(L.gem_read_state(g.h, w, G.GEM_SNAPSHOT, S[k].data_ptr(), 1))
        if case["proxy"] != "global":
            _ok(L.gem_read_state(g.h, w, G.GEM_MOMENT, M[k].data_ptr(), 1))
    if case["proxy"] == "global":      # one moment, stored as worker 0's
        _ok(L.gem_read_state(g.h, 0, G.GEM_MOMENT, M.data_ptr(), 1))
    out.update(theta=state["theta"], S=S, M=M)
    return out


# ---- what a pass cannot do without ------------------------------------------------
def work(case):
    P, T, n = case["P"], case["T"], case["n"]
    D = len(set(_schedule(case, 1).tolist()))
    given = case["kind"] == "batch"
    generated = not given
    if case["kind"] == "segment":
        # a commit's factor needs the whole vector first, so every commit reads theta, the
        # snapshot, the moment, h and theta*, and writes the pull and the moment
        bytes_ = 28.0 * P * T
    elif case["kind"] == "loop":
        # one commit at a time: snapshot, h, theta* read and the update written, then the
        # update, theta, the snapshot and the moment read, theta, the pull and the moment written
        d = 2 if case["bf16"] else 4
        bytes_ = (12.0 + d + d + 24.0) * P * T
    else:
        # theta and each committing worker's rows read and written once
        rows = 8.0 + 8.0 * D if case["proxy"] == "global" else 16.0 * D
        bytes_ = P * (8.0 + rows)
        if generated:
            bytes_ += 8.0 * P                                   # h, theta*
        if given:
            bytes_ += (2.0 if case["bf16"] else 4.0) * P * T    # the updates
    # operations of an element-commit: the GEM step (with its division) about 20, the noise (a
    # quarter of a Philox4x32-10 block, half a Box-Muller pair) and the update about 40 more
    return {"bytes": bytes_, "flops": (60.0 if generated else 20.0) * P * T}


def tolerance(case):
    return "exact"


# ---- the same in 64 bits, in plain torch ------------------------------------------
def _philox(q, t, seed):
    """Philox4x32-10 words of the counters (q mod 2^32, q >> 32, t, 0), as int64 tensors."""
    m32 = 0xFFFFFFFF
    c0, c1 = q & m32, q >> 32
    c2, c3 = torch.full_like(q, t & m32), torch.zeros_like(q)
    k0, k1 = seed & m32, (seed >> 32) & m32

    def mul(a, x):                      # the 64-bit product's words, without overflow
        lo, hi = x & 0xFFFF, x >> 16
        p0, p1 = lo * a, hi * a         # each below 2^48
        s = (p1 & 0xFFFF) * 65536 + p0
        return (p1 >> 16) + (s >> 32), s & m32

    for _ in range(10):
        ha, la = mul(0xD2511F53, c0)
        hb, lb = mul(0xCD9E8D57, c2)
        c0, c1, c2, c3 = hb ^ c1 ^ k0, lb, ha ^ c3 ^ k1, la
        k0, k1 = (k0 + 0x9E3779B9) & m32, (k1 + 0xBB67AE85) & m32
    return c0, c1, c2, c3


def _normals(i0, count, t, seed):
    q = torch.arange(i0 // 4, (i0 + count + 3) // 4, dtype=torch.int64, device="cuda")
    w = _philox(q, t, seed)
    z = torch.empty(q.numel(), 4, dtype=torch.float64, device="cuda")
    for k in (0, 2):
        r = (((w[k] >> 8) + 1).double() * 2.0 ** -24).log_().mul_(-2.0).sqrt_()
        phi = (w[k + 1] >> 8).double().mul_(2.0 * math.pi * 2.0 ** -24)
        z[:, k] = r * phi.cos()
        z[:, k + 1] = r * phi.sin()
    return z.view(-1)[:count]


def _f32(x):
    return float(np.float32(x))


def _bf16(d):
    return d.float().bfloat16().double()


def exact(case, seed):
    P, T, n = case["P"], case["T"], case["n"]
    if P * T > 2.6e10:
        return None
    worker = _schedule(case, seed).tolist()
    shared, pre = case["proxy"] == "global", case["pull"] == "pre"
    given = case["kind"] == "batch"
    upd = _updates(case, seed) if given else None
    h_all, ts_all = (None, None) if given else _problem(case, seed)
    off = _offsets(case).tolist() if case["kind"] == "segment" else None
    mu, eps, kappa = _f32(MU), _f32(EPS), _f32(case["kappa"])
    lr, sigma = _f32(case["lr"]), _f32(case["sigma"])
    read = _read_workers(case, np.array(worker))
    read_m = [0] if shared else read
    rows = sorted(set(worker))
    out = {k: torch.empty(r, P, dtype=torch.float64, device="cuda")
           for k, r in (("theta", 1), ("S", len(read)), ("M", len(read_m)))}
    # the commits are elementwise: a part of the vector at a time (segments need all of it)
    part = P if off else max(4, min(P, int(1.5e9 / len(rows))) // 4 * 4)
    zero = torch.zeros((), dtype=torch.float64, device="cuda")
    for i0 in range(0, P, part):
        m = min(part, P - i0)
        th = torch.zeros(m, dtype=torch.float64, device="cuda")
        S = {w: torch.zeros_like(th) for w in rows}
        M = {w: torch.zeros_like(th) for w in ([0] if shared else rows)}
        if not given:
            h, ts = h_all[i0:i0 + m].double(), ts_all[i0:i0 + m].double()
        pulled = dict.fromkeys(rows, 0)
        for t, w in enumerate(worker):
            s = S[w]
            if given:
                d = upd[t][i0:i0 + m].double()
            else:
                d = _normals(i0, m, t, seed).mul_(sigma).add_((s - ts).mul_(h)).mul_(-lr)
                d = _bf16(d) if case["bf16"] else d
            key = 0 if shared else w
            mom = M[key].mul_(mu).add_(d)
            if case["rule"] == "adaptive":
                new = th + d / (t - pulled[w] + 1)
            elif off:
                new = th.clone()
                for a, b in zip(off[:-1], off[1:]):
                    pi = (kappa * mom[a:b].norm() - (th[a:b] - s[a:b]).norm()) / (d[a:b].norm() + eps)
                    new[a:b] += torch.maximum(pi, zero) * d[a:b]
            else:
                pi = mom.abs().mul_(kappa).sub_((th - s).abs_()).div_(d.abs().add_(eps))
                new = th + pi.clamp_(min=0.0).mul_(d)
            S[w] = th if pre else new
            pulled[w] = t if pre else t + 1
            th = new
        out["theta"][0, i0:i0 + m] = th
        for k, w in enumerate(read):
            out["S"][k, i0:i0 + m] = S[w]
        for k, w in enumerate(read_m):
            out["M"][k, i0:i0 + m] = M[w]
    out["theta"] = out["theta"][0]
    if case["kind"] == "record":
        out["pi_hist"] = None
    return out
