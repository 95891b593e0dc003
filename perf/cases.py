"""The work that programs have this package do, as cases that can be timed and
compared: single decisions of a batch of tuners, decisions inside a
simulation, whole simulation runs, and the export of the learned models.

A case is a dict of plain values:

    kind     "step"    one decision, Tuner.step, on contexts and rewards that a
                       program has measured (a live controller's call)
             "sim"     one decision and the simulator's response, Tuner.step
                       and GpuEnv.step (the loop that a study writes itself)
             "run"     run_closed_loop from a fresh tuner to the last reward
             "export"  Tuner.export, the models as theta and A^-1
    B, K, d  instances, frequency arms, context features
    play     arms that no pruning rule has removed yet, per instance (0: all)
    prune    pruning rules in force (bit 1: confidence bounds; 2, 4, 8: the
             reward rules), exploit: the switch to greedy exploitation is on,
             refine: the windowed action space is on
    scores   1: the call also returns every arm's bounds
    sched    1: the exploration weight decays with the decisions made
    T, fused decisions of a run, and whether it takes the fused simulator step

A tuner that is not fresh holds models as they are in the middle of a run:
every factor upper triangular with a positive diagonal, between its prior 1 and
what some tens of updates leave, and weights near the mean reward of -0.9.
Pruning by confidence bounds comes every 50th decision in the runs; single
decisions are those in between, so their sets of arms stay as they are.
"""
import math

import torch

from agft_workloads import ENV, get_workload
from paper_2508_01744_amd import GpuEnv, Tuner, env_config, run_closed_loop

RING = 16          # contexts and rewards that a repeated decision goes round
SIM_T = 64         # windows of arrivals that a repeated simulation step goes round
NEVER = 1 << 30


def _case(name, kind, B, K, d, **kw):
    c = dict(name=name, kind=kind, B=B, K=K, d=d, play=0, prune=0, exploit=0, refine=0, scores=0, sched=0, T=0,
             fused=0)
    c.update(kw)
    return c


def listed():
    return [
        # one controller with a coarse grid: a call is one launch's latency
        _case("one_tuner", "sim", 1, 16, 8),
        # a rack of controllers, no pruning: each step reads every model, which stay in the last-level cache
        _case("sim_4096x64_d8", "sim", 4096, 64, 8),
        # the largest batch between two pruning steps, a few arms removed: HBM's rate
        _case("step_65536x128_d16", "step", 65536, 128, 16, play=122, prune=1),
        # all pruning rules, which read every arm's reward count and sum at each step
        _case("rules_16384x128_d16", "step", 16384, 128, 16, play=116, prune=15),
        # most instances past their switch to exploitation, the rest exploring
        _case("greedy_65536x128_d16", "step", 65536, 128, 16, prune=1, exploit=1),
        # the refined action space: 21 arms in play around each instance's anchor
        _case("window_65536x128_d16", "step", 65536, 128, 16, prune=1, refine=1),
        # wide contexts, the first steps of a run: every arm in play
        _case("step_1024x256_d32", "step", 1024, 256, 32, prune=1, sched=1),
        # the same late in a run: three arms left
        _case("late_1024x256_d32", "step", 1024, 256, 32, play=3, prune=1, sched=1),
        # an inspected decision of a ragged batch: the bounds of every arm come back
        _case("scores_1000x129_d16", "step", 1000, 129, 16, play=100, prune=1, scores=1),
        # the first decisions of a large simulation, tuner set-up included
        _case("run_65536x128_d16", "run", 65536, 128, 16, prune=1, T=20),
        # a small simulation past its first pruning step through the fused step
        _case("run_1024x256_d32", "run", 1024, 256, 32, prune=1, sched=1, T=60, fused=1),
        # what a program reads the learned models with
        _case("export_4096x128_d16", "export", 4096, 128, 16),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "sim", "run", "export"])
    d = rng.choice([8, 16, 16, 32])
    K = _log_uniform(rng, 8, 400)
    c = dict(kind=kind, d=d, K=K, play=0, prune=0, exploit=0, refine=0, scores=0, sched=rng.choice([0, 0, 1]), T=0,
             fused=0)
    model = 4 * (d + d * (d + 1) // 2)
    most = 4e9   # bytes of models
    if kind == "step":
        c["prune"] = rng.choice([0, 1, 1, 15])
        c["exploit"], c["refine"] = rng.choice([(0, 0), (0, 0), (1, 0), (0, 1), (1, 1)])
        c["scores"] = rng.choice([0, 0, 1])
        c["play"] = max(1, int(K * rng.choice([1.0, 0.95, 0.5, 0.1])))
    elif kind == "sim":
        most = 1e9
    elif kind == "run":
        c["T"] = rng.randint(10, 70)
        c["fused"] = rng.choice([0, 1])
        c["prune"] = rng.choice([0, 1])
        most = 5e10 / c["T"]
    else:
        most = 4e9 / (4 * (d * d + d)) * model
    hi = max(2, min(65536, int(most / (K * model))))
    c["B"] = min(hi, _log_uniform(rng, 1, hi) | rng.choice([0, 1]))
    if kind == "run":
        c["B"] = min(c["B"], 4096)   # near-ties of a run are few where its decisions are
    return c


# ---- inputs ----

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 13)


def _uniform(g, shape, lo, hi):
    return torch.rand(shape, generator=g, device="cuda") * (hi - lo) + lo


def _positions(B, K, d, chunks):
    """For every float of an instance's records, [blocks, NB * chunks * 4]: the
    arm it belongs to and the element of that arm, theta_i as i and S_ij as
    d + d*i + j, -1 for padding (the layout that agft.h documents)."""
    G, NB, M = d // 2, 64 // d, (d // 2) * (d // 4)
    tf = (chunks - M) * 4 // G
    size = NB * chunks * 4
    slot, elem = [0] * size, [-1] * size
    for r in range(NB):
        for j in range(G):
            for e in range(d + 3):
                at = (r * M + (e // 4) * G + j) * 4 + e % 4 if e < d else (NB * M * 4 + r * (chunks - M) * 4 + tf * j + e - d)
                slot[at] = r
                elem[at] = (d + d * e + j if e <= j else d + d * (d - e) + d - 1 - j if e <= d else 2 * j + e - d - 1)
    KB = (K + NB - 1) // NB
    arm = torch.arange(KB)[:, None] * NB + torch.tensor(slot)[None, :]
    el = torch.tensor(elem)[None, :].expand(KB, size).clone()
    el[arm >= K] = -1
    return arm.cuda(), el.cuda()


def _fill_models(view, B, K, d, g):
    arms = view["arms"]
    flat = arms.view(B, arms.shape[1], -1)
    _, el = _positions(B, K, d, arms.shape[2] // (64 // d))
    i, j = (el - d) // d, (el - d) % d
    theta = (el >= 0) & (el < d)
    factor = el >= d
    diag = factor & (i == j)
    mean = torch.where(diag, 0.5, torch.where(theta & (el == 0), -0.9, 0.0)).float()
    dev = torch.where(diag, 0.15, torch.where(factor, 0.05, torch.where(theta, 0.08, 0.0))).float()
    least = torch.where(diag, 0.1, -math.inf).float()
    flat.normal_(generator=g)
    flat.mul_(dev).add_(mean)
    torch.maximum(flat, least, out=flat)
    return arms


def _models(view, B, K, d, dtype, rows=slice(None)):
    """theta [b, K, d] and S [b, K, d, d] from the records."""
    arms = view["arms"]
    arm, el = _positions(B, K, d, arms.shape[2] // (64 // d))
    at = torch.zeros(K, d + d * d, dtype=torch.long, device="cuda")
    ok = el >= 0
    at[arm[ok], el[ok]] = torch.arange(el.numel(), device="cuda").view(el.shape)[ok]
    has = torch.zeros(K, d + d * d, dtype=torch.bool, device="cuda")
    has[arm[ok], el[ok]] = True
    flat = arms[rows].reshape(-1, arm.numel())
    can = flat[:, at.view(-1)].to(dtype).view(-1, K, d + d * d) * has
    return can[..., :d].contiguous(), can[..., d:].reshape(-1, K, d, d)


def _records(theta, S, shape):
    """Records of the given [.., KB, NB * chunks, 4] shape from theta and S."""
    b, K, d = theta.shape
    arm, el = _positions(b, K, d, shape[2] // (64 // d))
    can = torch.cat([theta, S.reshape(b, K, d * d)], dim=2).view(b, -1)
    ok = el >= 0
    out = torch.zeros(b, el.numel(), dtype=theta.dtype, device=theta.device)
    out[:, ok.view(-1)] = can[:, (arm * (d + d * d) + el)[ok]]
    return out.view(b, *shape[1:])


def _contexts(g, n, B, d):
    x = torch.randn(n, B, d, generator=g, device="cuda").clamp_(-3, 3)
    x[..., 0] = 1.0
    return x


def _rewards(g, n, B):
    return torch.randn(n, B, generator=g, device="cuda") * 0.15 - 0.9


def _mid_run(case, seed):
    """A tuner in the middle of its run, a decision awaiting its reward."""
    B, K, d = case["B"], case["K"], case["d"]
    g = _gen(seed)
    opt = {}
    if case["prune"] & 14:
        # the reward rules look at every arm and find none to remove
        opt["heuristics"] = dict(ext_rounds=60, ext_min_n=3, ext_thr=-1.9, hist_after=0, hist_min_n=2, hist_kappa=12.0,
                                 hist_min_arms=3, cascade_k=3 * K // 8)
    if case["exploit"]:
        # no instance switches by itself: its mode stays what it is
        opt["exploit"] = dict(ph_delta=0.05, ph_lambda=5.0, ph_window=NEVER, ph_min_rounds=0)
    if case["refine"]:
        opt["refine"] = dict(refine_period=50, refine_stride=10, refine_half=10, refine_mature=100, refine_min_n=4)
    tuner = Tuner(B, K, d, alpha0=0.5, alpha_sched=case["sched"], prune_rule=case["prune"], prune_period=NEVER,
                  device="cuda", **opt)
    ctx = _contexts(g, RING, B, d)
    reward = _rewards(g, RING, B)
    tuner.step(ctx[0], None)   # (what it decides is written over below)
    v = tuner.view()
    _fill_models(v, B, K, d, g)
    k = torch.arange(K, device="cuda")
    key = torch.rand(B, K, generator=g, device="cuda")
    if case["refine"]:
        half = 10
        c = torch.randint(0, K, (B,), generator=g, device="cuda")
        lo, hi = (c - half).clamp(min=0), (c + half).clamp(max=K - 1)
        v["window"].copy_(torch.stack([lo, hi, torch.ones_like(lo)], 1))
        space = (k >= lo[:, None]) & (k <= hi[:, None])
        key = torch.where(space, key, key + 1.0)
    else:
        space = torch.ones(B, K, dtype=torch.bool, device="cuda")
    order = key.argsort(dim=1)
    play = case["play"] or K
    keep = torch.zeros(B, K, dtype=torch.bool, device="cuda")
    keep.scatter_(1, order[:, :play], True)
    KW = v["mask"].shape[1]
    bits = torch.zeros(B, KW * 32, dtype=torch.int64, device="cuda")
    bits[:, :K] = keep
    words = (bits.view(B, KW, 32) << torch.arange(32, device="cuda")).sum(2)
    v["mask"].copy_(torch.where(words >= 1 << 31, words - (1 << 32), words))
    live = keep & space
    v["kact"].copy_(live.sum(1))
    v["aprev"].copy_(order[:, 0])
    v["xprev"].copy_(_contexts(g, 1, B, d)[0])
    if case["prune"] & 14 or case["refine"]:
        n = torch.randint(2, 20, (B, K), generator=g, device="cuda")
        mean = torch.randn(B, K, generator=g, device="cuda") * 0.05 - 0.9
        v["stats"][..., 0].copy_(n)
        v["stats"][..., 1].copy_((n * mean).float().view(torch.int32))
    if case["exploit"]:
        v["mode"].copy_(torch.where(torch.rand(B, generator=g, device="cuda") < 0.8, 100, -1))
        for a in range(0, B, 4096):
            v["theta"][a:a + 4096].copy_(_theta(v, B, K, d, slice(a, a + 4096)))
    return tuner, v, live, ctx, reward


def _theta(view, B, K, d, rows):
    arms = view["arms"]
    arm, el = _positions(B, K, d, arms.shape[2] // (64 // d))
    at = torch.zeros(K, d, dtype=torch.long, device="cuda")
    ok = (el >= 0) & (el < d)
    at[arm[ok], el[ok]] = torch.arange(el.numel(), device="cuda").view(el.shape)[ok]
    return arms[rows].reshape(-1, arm.numel())[:, at.view(-1)].view(-1, K, d)


def _draws(g, T, B):
    """Arrivals and latency noise of windows 0..T: loads from light to heavy, with bursts."""
    rate = _uniform(g, (1, B), 0.5, 20.0) * _uniform(g, (T + 1, B), 0.5, 1.5)
    arrivals = torch.poisson(rate, generator=g).to(torch.int32)
    return arrivals, torch.randn(T + 1, B, generator=g, device="cuda") * ENV["noise_sd"]


def _workload(case, T):
    return get_workload(4, B=case["B"], K=case["K"], d=case["d"], T=T, prune=case["prune"], alpha_sched=case["sched"],
                        drift=0.3 if case["sched"] else 0.0)


def prepare(case, seed):
    B = case["B"]
    if case["kind"] == "run":
        arrivals, noise = _draws(_gen(seed), case["T"], B)
        return dict(case=case, wl=_workload(case, case["T"]), arrivals=arrivals, noise=noise)
    tuner, view, live, ctx, reward = _mid_run(case, seed)
    st = dict(case=case, tuner=tuner, view=view, i=0, live=live, action=torch.empty(B, dtype=torch.int32, device="cuda"))
    if case["kind"] == "step":
        st["ctx"], st["reward"] = list(ctx.unbind(0)), list(reward.unbind(0))
        st["scores"] = torch.empty(B, 2, case["K"], device="cuda") if case["scores"] else None
    elif case["kind"] == "sim":
        arrivals, noise = _draws(_gen(seed + 1), SIM_T, B)
        st["env"] = env = GpuEnv(env_config(_workload(case, SIM_T), ENV), arrivals, noise)
        env.reset()
        env.reward.copy_(reward[0])
    return st


def run(st):
    kind = st["case"]["kind"]
    if kind == "run":
        out = run_closed_loop(st["wl"], ENV, st["arrivals"], st["noise"], fused=bool(st["case"]["fused"]))
        env, tuner = out["env"], out["tuner"]
        v = tuner.view()
        return dict(action=out["last_action"], reward=env.reward, ctx=env.ctx, arms=v["arms"], mask=v["mask"])
    tuner = st["tuner"]
    if kind == "export":
        theta, ainv = tuner.export(theta=True, ainv=True)
        return dict(theta=theta, ainv=ainv)
    i = st["i"]
    st["i"] = i + 1
    v = st["view"]
    out = dict(action=st["action"], arms=v["arms"])
    if kind == "sim":
        env = st["env"]
        tuner.step(env.ctx, env.reward, st["action"])
        out["reward"], out["ctx"] = env.step(i % SIM_T, st["action"])
        return out
    tuner.step(st["ctx"][i % RING], st["reward"][i % RING], st["action"], st["scores"])
    out["mask"] = v["mask"]
    if st["scores"] is not None:
        out["scores"] = st["scores"]
    if v["theta"] is not None:
        out["theta"] = v["theta"]
    return out


# ---- what a pass cannot do without ----

def _in_play(case):
    n = case["play"] or case["K"]
    return min(n, 21) if case["refine"] else n


def _step_work(case):
    """Bytes and operations of one decision: every model in play read once (theta
    alone by an exploiting instance), one written back, and each instance's words."""
    B, K, d = case["B"], case["K"], case["d"]
    model = d + d * (d + 1) // 2
    n = _in_play(case)
    explore = 0.2 if case["exploit"] else 1.0
    per = 4 * model * (explore * (n - 1) + 2) + (1 - explore) * 4 * d * (n - 1) + 4 * (3 * d + 7) + 4 * ((K + 31) // 32)
    if case["prune"] & 14:
        per += 8 * K
    if case["exploit"]:
        per += 72 + 4 * d
    if case["scores"]:
        per += 8 * K
    ops = 2 * model * (explore * n + 3) + (1 - explore) * 2 * d * n
    return B * per, B * ops


def work(case):
    B, K, d = case["B"], case["K"], case["d"]
    model = d + d * (d + 1) // 2
    env = B * (4 * (2 * 31 + 3 + 3) + 4 * d)   # the simulator's state read and written, its draws, the next context
    if case["kind"] == "export":
        return dict(bytes=4.0 * B * K * (model + d + d * d), flops=float(B * K * d * d * d) / 1.5)
    b, f = _step_work(case)
    if case["kind"] == "step":
        return dict(bytes=float(b), flops=float(f))
    if case["kind"] == "sim":
        return dict(bytes=float(b + env), flops=float(f))
    T = case["T"]   # and the models are written once before the first decision, the last reward folded in after the last
    return dict(bytes=float(T * (b + env) + 4 * model * B * K + 8 * model * B), flops=float(T * f))


def tolerance(case):
    # 32-bit sums in another order; a near-tie may take the other arm of a few instances
    return {"rel": 1e-5, "max": 1e-2, "differ": 1e-3}


# ---- the same in 64 bits ----

def _update(theta, S, x, r):
    """One reward folded into theta [n, d] and S [n, d, d] with S S^T = A^-1, A += x x^T."""
    f = (S * x[:, :, None]).sum(1)
    al = 1.0 + (f * f).cumsum(1)
    prev = al - f * f
    run_ = S * f[:, None, :]
    g = run_.cumsum(2)
    theta = theta + g[:, :, -1] / al[:, -1:] * (r - (theta * x).sum(1))[:, None]
    S = (prev / al).sqrt()[:, None, :] * S - (f / (prev * al).sqrt())[:, None, :] * (g - run_)
    return theta, S


def _bounds(theta, S, x, alpha, live, greedy):
    m = (theta * x[:, None, :]).sum(2)
    w = ((S * x[:, None, :, None]).sum(2) ** 2).sum(2).sqrt() * alpha
    if greedy is not None:
        w = torch.where(greedy[:, None], torch.zeros_like(w), w)
    low = torch.full_like(m, -math.inf)
    return torch.where(live, m + w, low), torch.where(live, m - w, low)


def _first_largest(u):
    k = torch.arange(u.shape[1], device=u.device)
    return torch.where(u == u.max(1, keepdim=True).values, k, u.shape[1]).min(1).values


class _Env64:
    """The simulated serving nodes (agft_sim.h's closed form) in 64 bits."""

    def __init__(self, case, T, arrivals, noise):
        self.K, self.d, self.T = case["K"], case["d"], T
        self.drift = 0.3 if case["sched"] else 0.0
        self.n, self.eta = arrivals.double(), noise.double()
        B = self.n.shape[1]
        one = torch.ones(B, dtype=torch.float64, device="cuda")
        self.q, self.cap, self.f = 0.0 * one, ENV["svc_init"] * one, ENV["f_init"] * one
        z, rho = self._window(0, 1.0)
        self.z, self.rho = [z] * 4, [rho] * 3

    def _window(self, w, scale):
        e, n, f = ENV, self.n[w], self.f
        b, c = e["b"] * scale, e["c"] * scale
        lat = (e["l0"] * (e["a"] + b * n / f) + self.eta[w]).clamp(min=e["lat_min"])
        ref = e["l0"] * (e["a"] + b * n)
        rho = -((e["P0"] + c * f ** 3) * lat * lat) / ((e["P0"] + c) * ref * ref)
        self.q = (self.q + n - self.cap).clamp(0, e["q_cap"])
        raw = [n, torch.log1p(self.q), (self.q + n).clamp(max=e["run_cap"]), torch.log(lat * (1 + self.q / self.cap)),
               lat / e["tpot_div"], (n / self.cap).clamp(max=1.0), f]
        mu, sd = (torch.tensor(e[k], dtype=torch.float64, device="cuda") for k in ("mu", "sd"))
        return (torch.stack(raw, 1) - mu) / sd, rho

    def context(self):
        one = torch.ones_like(self.f)[:, None]
        if self.d == 8:
            return torch.cat([one, self.z[0]], 1)
        if self.d == 16:
            return torch.cat([one, self.z[0], self.z[1], self.rho[0][:, None]], 1)
        return torch.cat([one, *self.z, *[r[:, None] for r in self.rho]], 1)

    def step(self, t, a):
        e, n = ENV, max(1, self.K - 1)
        self.f = (e["f_lo"] + (e["f_hi"] - e["f_lo"]) * a / n) if self.K > 1 else torch.full_like(self.f, e["f_hi"])
        span = e["svc_hi"] - e["svc_lo"]
        cap = e["svc_lo"] + torch.div(2 * span * a + n, 2 * n, rounding_mode="floor")
        self.cap = (cap if self.K > 1 else torch.full_like(a, e["svc_hi"])).double()
        z, rho = self._window(t + 1, 1.0 + self.drift * (t / (self.T - 1) if self.T > 1 else 0.0))
        self.z, self.rho = [z] + self.z[:3], [rho] + self.rho[:2]
        return rho


def _exact_run(case, arrivals, noise, shape):
    """run_closed_loop's results for some of the instances."""
    K, d, T = case["K"], case["d"], case["T"]
    b = arrivals.shape[1]
    env = _Env64(case, T, arrivals, noise)
    theta = torch.zeros(b, K, d, dtype=torch.float64, device="cuda")
    S = torch.eye(d, dtype=torch.float64, device="cuda").repeat(b, K, 1, 1)
    live = torch.ones(b, K, dtype=torch.bool, device="cuda")
    row = torch.arange(b, device="cuda")
    alpha0 = get_workload(4).alpha0
    for t in range(T):
        x = env.context()
        u, low = _bounds(theta, S, x, alpha0 / math.sqrt(t + 1.0) if case["sched"] else alpha0, live, None)
        if case["prune"] & 1 and t > 0 and t % 50 == 0:
            live = live & (u >= low.max(1, keepdim=True).values)
            u = torch.where(live, u, -math.inf)
        a = _first_largest(u)
        rho = env.step(t, a)
        theta[row, a], S[row, a] = _update(theta[row, a], S[row, a], x, rho)
    return env.rho[0], env.context(), _records(theta, S, shape)


def exact(case, seed):
    B, K, d = case["B"], case["K"], case["d"]
    st = prepare(case, seed)
    f64 = torch.float64
    part = max(1, min(B, int(2e8 // (K * d * d))))
    parts = [slice(a, min(B, a + part)) for a in range(0, B, part)]
    if case["kind"] == "run":
        shape = Tuner.from_workload(st["wl"], B=1, device="cuda").view()["arms"].shape
        out = [_exact_run(case, st["arrivals"][:, p], st["noise"][:, p], shape) for p in parts]
        reward, ctx, arms = (torch.cat(v) for v in zip(*out))
        return dict(action=None, reward=reward, ctx=ctx, arms=arms, mask=None)
    v = st["view"]
    if case["kind"] == "export":
        out = []
        for p in parts:
            theta, S = _models(v, B, K, d, f64, p)
            out.append((theta, torch.matmul(S, S.transpose(2, 3).contiguous())))
        theta, ainv = (torch.cat(t) for t in zip(*out))
        return dict(theta=theta, ainv=ainv)
    sim = case["kind"] == "sim"
    env = _Env64(case, SIM_T, st["env"].arrivals, st["env"].noise) if sim else None
    reward = (st["env"].reward if sim else st["reward"][0]).to(f64)
    x = env.context() if sim else st["ctx"][0].to(f64)
    greedy = v["mode"] >= 0 if case["exploit"] else None
    alpha = 0.5 / math.sqrt(2.0) if case["sched"] else 0.5
    arms, copies, scores, action = [], [], [], []
    for p in parts:
        theta, S = _models(v, B, K, d, f64, p)
        row, a = torch.arange(theta.shape[0], device="cuda"), v["aprev"][p].long()
        theta[row, a], S[row, a] = _update(theta[row, a], S[row, a], v["xprev"][p].to(f64), reward[p])
        arms.append(_records(theta, S, v["arms"].shape))
        if case["exploit"]:
            copies.append(theta)
        if case["scores"] or sim:
            u, low = _bounds(theta, S, x[p], alpha, st["live"][p], None if greedy is None else greedy[p])
            if case["scores"]:
                scores.append(torch.stack([u, low], 1))
            action.append(_first_largest(u))
    out = dict(action=None, arms=torch.cat(arms))
    if sim:
        out["reward"] = env.step(0, torch.cat(action))
        out["ctx"] = env.context()
        return out
    out["mask"] = None
    if case["scores"]:
        out["scores"] = torch.cat(scores)
    if case["exploit"]:
        out["theta"] = torch.cat(copies)
    return out
