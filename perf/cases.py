"""What is timed: the calls a user of this library makes, over the range of sizes they make them at.

A case is one of the parts of a PQL program, driven through LearnerSession (the package's public
plumbing around the C entry points):

  critic     pql_critic_update with its Polyak step (Algorithm 3, the V-learner's step)
  policy     pql_actor_update with the copy into the lagged policy (Algorithm 2, the P-learner's step)
  act        pql_actor_act on all environments (Algorithm 1, the Actor's step)
  replay     pql_replay_push of one Actor step, then pql_sample_nstep of one batch
  iteration  one whole Actor iteration at the paper's default ratios: one Actor step and push, eight
             critic updates on freshly sampled batches, four policy updates

Parameters, Adam moments and step numbers are those of a run in progress (a target that lags the
critics, moments of the size gradients have), observations are of unit scale as a simulator's
standardised ones are.  `exact` computes the same results with plain torch in double precision.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2307_12983_amd.session import LearnerSession
from paper_2307_12983_amd.workloads import Workload

F32 = lambda x: float(np.float32(x))  # noqa: E731  (hyper-parameters cross the C interface as floats)
LR, GAMMA, TAU, BETA1, BETA2, EPS = F32(5e-4), F32(0.99), F32(0.05), F32(0.9), F32(0.999), F32(1e-8)
V_MIN, V_MAX, NORM_EPS = -10.0, 10.0, F32(1e-5)
CRITIC_STEPS, POLICY_STEPS = 1000, 500          # Adam steps done when a case begins
DEVICE = "cuda:0"


def _case(kind, obs, act, hidden, batch, envs, rows=0, name=None, **kw):
    c = dict(kind=kind, obs=obs, act=act, hidden=hidden, batch=batch, envs=envs, rows=rows, nstep=3, atoms=0,
             sac=False, clip=0.0, obs_norm=False, folded=True, sigma_min=0.05, sigma_max=0.8)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest program: 64 environments, batch 256, all of Table B.1's defaults (gradient clipping,
        # observation standardisation); bound by launches and latency
        _case("iteration", 8, 2, "64,64", 256, 64, 64, "tiny_iteration", clip=0.5, obs_norm=True),
        # the default workload as a program runs it
        _case("iteration", 60, 8, "256,256", 8192, 4096, 244, "ant_iteration", sigma_min=0.2, sigma_max=0.2),
        # its parts
        _case("critic", 60, 8, "256,256", 8192, 4096, name="ant_critic"),
        _case("policy", 60, 8, "256,256", 8192, 4096, name="ant_policy"),
        _case("act", 60, 8, "256,256", 8192, 4096, name="ant_act"),
        # distributional critics (PQL-D) with the paper's gradient clipping
        _case("critic", 60, 8, "256,256", 8192, 4096, name="ant_dist_critic", atoms=51, clip=0.5),
        # a wider network, ordinary batch
        _case("critic", 108, 21, "512,256,128", 8192, 16384, name="humanoid_critic", folded=False),
        # many environments in one Actor step
        _case("act", 108, 21, "512,256,128", 8192, 16384, name="humanoid_act", obs_norm=True),
        # a dexterous hand: odd observation size, wide layers, doubled batch
        _case("policy", 211, 20, "512,512,256", 16384, 16384, name="shadow_policy"),
        # the largest update
        _case("critic", 211, 20, "1024,512,256", 32768, 32768, name="scale_critic", nstep=5),
        # the largest replay traffic: 14 GB ring, one row in, one batch out
        _case("replay", 211, 20, "1024,512,256", 32768, 32768, 244, "scale_replay", nstep=5),
        # a network of one's own with widths that fit no tile, the stochastic policy and separate calls
        _case("policy", 45, 11, "200,100", 3001, 1000, name="ragged_sac_policy", sac=True, folded=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    top = work(_case("critic", 211, 20, "1024,512,256", 32768, 32768))
    while True:
        kind = rng.choice(["critic", "critic", "policy", "policy", "act", "replay", "iteration"])
        o, a = _log(rng, 6, 240), _log(rng, 2, 24)
        depth = rng.choice([2, 2, 3, 3, 1, 4])
        step = rng.choice([64, 32, 32, 1])
        first = _log(rng, 32, 1024)
        hidden = [max(step, first // step * step)]
        for _ in range(depth - 1):
            hidden.append(max(step, hidden[-1] // rng.choice([1, 1, 2]) // step * step, 24))
        batch, envs = _log(rng, 64, 32768), _log(rng, 32, 32768)
        if rng.random() < 0.5:
            batch = max(64, batch // 64 * 64)
        variant = rng.choice(["plain", "plain", "plain", "sac", "dist"])
        c = _case(kind, o, a, ",".join(str(h) for h in hidden), batch, envs,
                  rng.randrange(8, 245) if kind in ("replay", "iteration") else 0, nstep=rng.choice([1, 3, 3, 5]),
                  atoms=rng.choice([51, 51, 21]) if variant == "dist" else 0, sac=variant == "sac",
                  clip=rng.choice([0.0, 0.0, 0.5]), obs_norm=rng.random() < 0.3 and kind in ("act", "replay", "iteration"),
                  folded=rng.random() < 0.7, sigma_min=rng.choice([0.05, 0.2]), sigma_max=rng.choice([0.2, 0.8]))
        w = work(c)
        if w["flops"] <= top["flops"] and c["rows"] * envs * (2 * o + a + 2) * 4 <= 15e9:
            return c


# ---- shapes -----------------------------------------------------------------------------------
def _layers(n_in, hidden, n_out):
    sizes = [n_in] + [int(h) for h in hidden.split(",")] + [n_out]
    return list(zip(sizes[:-1], sizes[1:]))


def _actor(c):
    return _layers(c["obs"], c["hidden"], 2 * c["act"] if c["sac"] else c["act"])


def _critic(c):
    return _layers(c["obs"] + c["act"], c["hidden"], c["atoms"] if c["atoms"] >= 2 else 1)


def _count(dims):
    return sum(i * o + o for i, o in dims)


def work(case):
    """Multiply-adds on weight matrices (two operations each) and every array read or written once."""
    c = case
    pa, pc = sum(i * o for i, o in _actor(c)), sum(i * o for i, o in _critic(c))
    na, nc = _count(_actor(c)), 2 * _count(_critic(c))
    pa1, pc1 = (d[0][0] * d[0][1] for d in (_actor(c), _critic(c)))
    act_cols = c["act"] * _critic(c)[0][1]
    B, N, o, a, n = c["batch"], c["envs"], c["obs"], c["act"], c["nstep"]
    step = {
        "critic": (B * (2 * pa + 8 * pc + 2 * (2 * pc + 2 * (pc - pc1))),
                   4.0 * (B * (2 * o + a + 2) + na + nc * 9)),          # theta, m, v, Q' in and out, g out
        "policy": (B * (2 * pa + 4 * pc + 4 * (pc - pc1 + act_cols) + 2 * pa + 2 * (pa - pa1)),
                   4.0 * (B * o + nc + na * 8)),
        "act": (2 * pa * N, 4.0 * (N * (o + a) + na)),
        "push": (0, 4.0 * 2 * N * (2 * o + a + 2)),
        "sample": (0, 4.0 * B * (2 * (2 * o + a) + 2 * n + 4)),
    }
    times = {"critic": {"critic": 1}, "policy": {"policy": 1}, "act": {"act": 1}, "replay": {"push": 1, "sample": 1},
             "iteration": {"act": 1, "push": 1, "sample": 8, "critic": 8, "policy": 4}}[c["kind"]]
    return {"bytes": float(sum(k * step[s][1] for s, k in times.items())),
            "flops": float(sum(k * step[s][0] for s, k in times.items()))}


def tolerance(case):
    """Single precision throughout.  Gradients and losses are 32-bit sums over the batch behind a chain of
    32-bit layers; the largest single entries are held by `max`."""
    if case["kind"] == "replay":
        return {"rel": 2e-6, "max": 1e-5}
    if case["kind"] == "act":
        return {"rel": 1e-5, "max": 2e-4}
    if case["kind"] == "iteration":
        return {"rel": 1e-3, "max": 0.5}
    return {"rel": 2e-5, "max": 2e-3}


# ---- inputs -----------------------------------------------------------------------------------
def _gen(seed, part):
    g = torch.Generator(device=DEVICE)
    g.manual_seed((int(seed) * 8 + part) % (1 << 62))
    return g


def _params(dims, g):
    parts = []
    for i, o in dims:
        parts.append((torch.rand(i * o + o, generator=g, device=DEVICE) * 2 - 1) / math.sqrt(i))
    return torch.cat(parts)


def _networks(c, seed):
    """Parameters and moments of a run in progress, drawn from the seed."""
    g = _gen(seed, 0)
    d = {"actor": _params(_actor(c), g), "critic": torch.cat([_params(_critic(c), g), _params(_critic(c), g)])}
    lag = lambda t: t + 0.02 * t.abs().mean() * torch.randn(t.numel(), generator=g, device=DEVICE)  # noqa: E731
    d["actor_lag"], d["critic_target"] = lag(d["actor"]), lag(d["critic"])
    for p, t in (("a", d["actor"]), ("c", d["critic"])):
        size = 1e-3 * torch.exp(torch.randn(t.numel(), generator=g, device=DEVICE))
        d[p + "_v"] = size * size
        d[p + "_m"] = 0.3 * size * torch.randn(t.numel(), generator=g, device=DEVICE)
    if c["sac"]:
        d["temperature"] = torch.tensor([math.log(0.2), 1e-3, 1e-5, 0.0], device=DEVICE)
    return d


def _batch(c, seed):
    g = _gen(seed, 1)
    B, o, a = c["batch"], c["obs"], c["act"]
    r = lambda *s: torch.randn(*s, generator=g, device=DEVICE)  # noqa: E731
    u = lambda *s: torch.rand(*s, generator=g, device=DEVICE)  # noqa: E731
    alive = (u(B) >= 0.01 * c["nstep"]).float()
    return {"obs": r(B, o), "act": u(B, a) * 2 - 1, "ret": r(B) * math.sqrt(c["nstep"]), "next_obs": r(B, o),
            "boot": alive * F32(GAMMA ** c["nstep"])}


def _row(c, g):
    N, o, a = c["envs"], c["obs"], c["act"]
    obs = torch.randn(N, o, generator=g, device=DEVICE)
    if c["obs_norm"]:
        obs = obs * 3 + 1                                   # a simulator's own units
    act = torch.rand(N, a, generator=g, device=DEVICE) * 2 - 1
    rew = torch.randn(N, generator=g, device=DEVICE)
    done = (torch.rand(N, generator=g, device=DEVICE) < 0.01).float()
    nxt = obs + 0.1 * torch.randn(N, o, generator=g, device=DEVICE)
    return {"obs": obs, "act": act, "rew": rew, "next_obs": nxt, "done": done}


def _rng_seed(seed):
    return (0x5EED0000 + int(seed) * 0x9E3779B1) % (1 << 63)


def prepare(case, seed):
    c = case
    w = Workload("case", c["obs"], c["act"], c["envs"], c["envs"] * max(c["rows"], c["nstep"]), c["batch"], c["nstep"],
                 tuple(int(h) for h in c["hidden"].split(",")), 0.01, lr=LR, gamma=GAMMA, tau=TAU,
                 sigma_min=F32(c["sigma_min"]), sigma_max=F32(c["sigma_max"]), beta1=BETA1, beta2=BETA2, eps=EPS,
                 max_grad_norm=c["clip"], obs_norm=c["obs_norm"], obs_norm_eps=NORM_EPS, num_atoms=c["atoms"],
                 v_min=V_MIN, v_max=V_MAX, sac=c["sac"])
    s = LearnerSession(w, device=DEVICE, seed=_rng_seed(seed))
    for k, v in _networks(c, seed).items():
        getattr(s, k).copy_(v)
    if c["folded"]:
        s.fold_followups()
    state = {"case": c, "s": s, "env": []}
    if c["kind"] in ("critic", "policy"):
        for k, v in _batch(c, seed).items():
            getattr(s.batch, k)[:c["batch"]].copy_(v)
    else:
        g = _gen(seed, 2)
        # the ring as a run in progress has it: every row written (an Actor alone needs only the statistics)
        for _ in range(c["rows"] if c["rows"] else (1 if c["obs_norm"] else 0)):
            s.push(_row(c, g))
        state["env"] = [_row(c, _gen(seed, 3))]
    at = s.ctx.get_state()
    at[5], at[6] = CRITIC_STEPS, POLICY_STEPS
    s.ctx.set_state(at)
    return state


# ---- the pass that is timed -------------------------------------------------------------------
def _critic_outputs(s):
    return {"critic": s.critic, "target": s.critic_target, "m": s.c_m, "v": s.c_v, "grads": s.c_g, "loss": s.critic_out}


def _policy_outputs(s):
    out = {"actor": s.actor, "lagged": s.actor_lag, "m": s.a_m, "v": s.a_v, "grads": s.a_g, "loss": s.actor_out}
    if s.temperature is not None:
        out["temperature"] = s.temperature
    return out


def run(state):
    c, s = state["case"], state["s"]
    B = c["batch"]
    if c["kind"] == "critic":
        s.critic_update(B)
        s.soft_update_targets()
        return _critic_outputs(s)
    if c["kind"] == "policy":
        s.actor_update(s.batch.obs, B)
        s.sync_lagged_policy()
        return _policy_outputs(s)
    row = state["env"][0]
    if c["kind"] == "act":
        return {"act": s.act(row["obs"])}
    if c["kind"] == "replay":
        s.push(row)
        s.sample(B)
        return {k: getattr(s.batch, k)[:B] for k in ("idx", "obs", "act", "ret", "next_obs", "boot")}
    act = s.act(row["obs"])
    s.ctx.pql_replay_push(s.storage, row["obs"], act, row["rew"], row["next_obs"], row["done"])
    for k in range(8):
        s.sample(B)
        s.critic_update(B)
        s.soft_update_targets()
        if k % 2:
            s.actor_update(s.batch.obs, B)
            s.sync_lagged_policy()
    return {"act": act, "v_learner": _critic_outputs(s), "p_learner": _policy_outputs(s)}


# ---- the same in double precision -----------------------------------------------------------------
def _philox(seed, stream, call, count):
    """Words 0 and 1 of Philox-4x32-10 (Salmon et al., SC'11) for elements 0..count-1."""
    low, s32 = np.uint64(0xFFFFFFFF), np.uint64(32)
    x = [np.arange(count, dtype=np.uint64)] + [np.full(count, v, np.uint64) for v in (stream, call & 0xFFFFFFFF, call >> 32)]
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32
    for _ in range(10):
        p, q = np.uint64(0xD2511F53) * x[0], np.uint64(0xCD9E8D57) * x[2]
        x = [(q >> s32) ^ x[1] ^ np.uint64(k0), q & low, (p >> s32) ^ x[3] ^ np.uint64(k1), p & low]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return x[0], x[1]


def _normal(seed, stream, call, rows, cols):
    w0, w1 = _philox(seed, stream, call, rows * cols)
    u = [((w >> np.uint64(8)).astype(np.float64) + 0.5) * 2.0 ** -24 for w in (w0, w1)]
    return torch.from_numpy((np.sqrt(-2 * np.log(u[0])) * np.cos(2 * np.pi * u[1])).reshape(rows, cols)).to(DEVICE)


def _mlp(params, dims, x):
    at = 0
    for k, (i, o) in enumerate(dims):
        x = x @ params[at:at + i * o].reshape(i, o) + params[at + i * o:at + i * o + o]
        at += i * o + o
        if k < len(dims) - 1:
            x = torch.where(x > 0, x, torch.expm1(torch.clamp(x, max=0.0)))
    return x


def _sac_sample(c, params, obs, eps):
    out = _mlp(params, _actor(c), obs)
    mu, raw = out[:, :c["act"]], out[:, c["act"]:]
    ls = torch.clamp(raw, -5.0, 2.0)
    u = mu + torch.exp(ls) * eps
    det = 2.0 * (math.log(2.0) - u - torch.nn.functional.softplus(-2.0 * u))
    return torch.tanh(u), (-0.5 * eps * eps - ls - 0.5 * math.log(2.0 * math.pi) - det).sum(1)


def _atoms(c):
    return torch.linspace(V_MIN, V_MAX, c["atoms"], dtype=torch.float64, device=DEVICE)


def _adam(c, theta, g, m, v, t):
    norm = float(g.norm())
    if c["clip"] > 0 and norm > F32(c["clip"]):
        g = g * (F32(c["clip"]) / norm)
    m, v = BETA1 * m + (1 - BETA1) * g, BETA2 * v + (1 - BETA2) * g * g
    theta = theta - LR * (m / (1 - BETA1 ** t)) / (torch.sqrt(v / (1 - BETA2 ** t)) + EPS)
    return theta, m, v, g, (norm if c["clip"] > 0 else 0.0)


def _exact_critic(c, seed):
    d = {k: v.double() for k, v in _networks(c, seed).items()}
    b = {k: v.double() for k, v in _batch(c, seed).items()}
    B, n = c["batch"], d["critic"].numel() // 2
    q = lambda p, i, s, a: _mlp(p[i * n:(i + 1) * n], _critic(c), torch.cat([s, a], 1))  # noqa: E731
    entropy = 0.0
    if c["sac"]:
        a2, logp = _sac_sample(c, d["actor_lag"], b["next_obs"], _normal(_rng_seed(seed), 4, CRITIC_STEPS, B, c["act"]))
        entropy = torch.exp(d["temperature"][0]) * logp
    else:
        a2 = torch.tanh(_mlp(d["actor_lag"], _actor(c), b["next_obs"]))
    t = [q(d["critic_target"], i, b["next_obs"], a2) for i in (0, 1)]
    theta = d["critic"].clone().requires_grad_()
    out = [q(theta, i, b["obs"], b["act"]) for i in (0, 1)]
    if c["atoms"] >= 2:
        z = _atoms(c)
        p = [torch.softmax(x, 1) for x in t]
        p = torch.where((p[0] @ z <= p[1] @ z)[:, None], p[0], p[1])
        tz = torch.clamp(b["ret"][:, None] + b["boot"][:, None] * z, V_MIN, V_MAX)
        target = torch.zeros_like(p)
        for j in range(c["atoms"]):
            target += p[:, j:j + 1] * torch.clamp(1 - (tz[:, j:j + 1] - z).abs() / (z[1] - z[0]), 0, 1)
        losses = [-(target * torch.log_softmax(x, 1)).sum(1).mean() for x in out]
    else:
        y = b["ret"] + b["boot"] * (torch.minimum(t[0][:, 0], t[1][:, 0]) - entropy)
        losses = [((x[:, 0] - y) ** 2).mean() for x in out]
    g, = torch.autograd.grad(losses[0] + losses[1], theta)
    theta, m, v, g, norm = _adam(c, d["critic"], g, d["c_m"], d["c_v"], CRITIC_STEPS + 1)
    loss = torch.tensor([float(losses[0]), float(losses[1]), norm], dtype=torch.float64)
    return {"critic": theta, "target": TAU * theta + (1 - TAU) * d["critic_target"], "m": m, "v": v, "grads": g,
            "loss": loss}


def _exact_policy(c, seed):
    d = {k: v.double() for k, v in _networks(c, seed).items()}
    obs = _batch(c, seed)["obs"].double()
    B, n = c["batch"], d["critic"].numel() // 2
    theta = d["actor"].clone().requires_grad_()
    logp = None
    if c["sac"]:
        act, logp = _sac_sample(c, theta, obs, _normal(_rng_seed(seed), 5, POLICY_STEPS, B, c["act"]))
    else:
        act = torch.tanh(_mlp(theta, _actor(c), obs))
    q = [_mlp(d["critic"][i * n:(i + 1) * n], _critic(c), torch.cat([obs, act], 1)) for i in (0, 1)]
    q = [torch.softmax(x, 1) @ _atoms(c) if c["atoms"] >= 2 else x[:, 0] for x in q]
    J = -torch.minimum(q[0], q[1]).mean()
    loss = [float(J), 0.0, 0.0, 0.0]
    if c["sac"]:
        alpha, mean = torch.exp(d["temperature"][0]), logp.mean()
        g, = torch.autograd.grad(J + alpha * mean, theta)
        loss[2], loss[3] = float(alpha * mean), float(mean)
    else:
        g, = torch.autograd.grad(J, theta)
    theta, m, v, g, loss[1] = _adam(c, d["actor"], g, d["a_m"], d["a_v"], POLICY_STEPS + 1)
    out = {"actor": theta, "lagged": theta, "m": m, "v": v, "grads": g, "loss": torch.tensor(loss, dtype=torch.float64)}
    if c["sac"]:
        t = d["temperature"]
        gt = (-torch.exp(t[0]) * (loss[3] - c["act"])).reshape(1)
        x, tm, tv, _, _ = _adam(dict(c, clip=0.0), t[:1], gt, t[1:2], t[2:3], POLICY_STEPS + 1)
        out["temperature"] = torch.cat([x, tm, tv, t[3:]])
    return out


def _exact_act(c, seed):
    g, row = _gen(seed, 2), _row(c, _gen(seed, 3))
    obs = row["obs"].double()
    if c["obs_norm"]:
        seen = _row(c, g)["obs"].double()
        obs = (obs - seen.mean(0)) / torch.sqrt(seen.var(0, unbiased=False) + NORM_EPS)
    theta, N = _networks(c, seed)["actor"].double(), c["envs"]
    eps = _normal(_rng_seed(seed), 2, 0, N, c["act"])
    if c["sac"]:
        return {"act": _sac_sample(c, theta, obs, eps)[0]}
    lo, hi = F32(c["sigma_min"]), F32(c["sigma_max"])
    sigma = lo + torch.arange(N, dtype=torch.float64, device=DEVICE) / max(N - 1, 1) * (hi - lo)
    return {"act": torch.clamp(torch.tanh(_mlp(theta, _actor(c), obs)) + sigma[:, None] * eps, -1.0, 1.0)}


def _exact_replay(c, seed):
    g, N, T, n, B = _gen(seed, 2), c["envs"], max(c["rows"], c["nstep"]), c["nstep"], c["batch"]
    rows = [_row(c, g) for _ in range(c["rows"])]
    seen = [r["obs"] for r in rows]
    rows.append(_row(c, _gen(seed, 3)))
    seen.append(rows[-1]["obs"])
    mean = sum(x.double().sum(0) for x in seen) / (len(seen) * N)
    var = sum(((x.double() - mean) ** 2).sum(0) for x in seen) / (len(seen) * N)
    first, kept = max(0, len(rows) - T), min(len(rows), T)          # chronological row of the oldest one kept
    V = (kept - n + 1) * N
    w0, w1 = _philox(_rng_seed(seed), 1, 0, B)
    p = np.array([(((int(h) << 32) | int(l)) * V) >> 64 for h, l in zip(w1, w0)], dtype=np.int64)
    j, e = torch.from_numpy(p // N + first).to(DEVICE), torch.from_numpy(p % N).to(DEVICE)

    def take(field, j):
        out = torch.zeros((B,) + tuple(rows[0][field].shape[1:]), dtype=torch.float64, device=DEVICE)
        for k in range(len(rows)):
            at = (j == k).nonzero()[:, 0]
            if at.numel():
                out[at] = rows[k][field][e[at]].double()
        return out

    ret = torch.zeros(B, dtype=torch.float64, device=DEVICE)
    alive = torch.ones_like(ret)
    for k in range(n):
        ret += GAMMA ** k * take("rew", j + k) * alive
        alive = alive * (1 - take("done", j + k))
    norm = lambda x: (x - mean) / torch.sqrt(var + NORM_EPS) if c["obs_norm"] else x  # noqa: E731
    return {"idx": None, "obs": norm(take("obs", j)), "act": take("act", j), "ret": ret,
            "next_obs": norm(take("next_obs", j + n - 1)), "boot": GAMMA ** n * alive}


def exact(case, seed):
    kind = {"critic": _exact_critic, "policy": _exact_policy, "act": _exact_act, "replay": _exact_replay}.get(case["kind"])
    return kind(case, seed) if kind else None          # an iteration is thousands of roundings deep
