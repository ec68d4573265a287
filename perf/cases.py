"""The work a learner program has this framework do, as measurable cases.

Two kinds of case, each through the public binding (paper_2312_06126_amd.Spz):

* "update": a learner's interval between two publications of its weights: optionally new
  transitions pushed, `steps` whole update steps enqueued in one call, then the losses of
  those steps and the weights of the actor and both critics read back;
* "act": actions of the current policy for a set of sampler observations, from host arrays
  (`act`) or from device memory (`act_noalloc`).

Sizes: the five update workloads of synth/workloads.py (small, walker, humanoid, ant and
large networks), the large one's per-GPU share of eight-way data parallelism, ragged
networks such as the tests use, and generic sizes between them.

`exact` is the same computation in 64 bits with plain torch (autograd) and numpy, without
this repository's code: Philox4x32-10 (Salmon et al., SC'11) for the initial weights, the
replay indices and the noise, then SAC or TD3 as published.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2312_06126_amd import Spz

GAMMA, TAU, LR, BETA1, BETA2, EPS = 0.99, 0.005, 3e-4, 0.9, 0.999, 1e-8
LOG_STD = (-20.0, 2.0)
SMOOTH, SMOOTH_CLIP, DELAY = 0.2, 0.5, 2
P_DONE = 0.01
ACT_COUNTER = 7
BASE_ROWS = 65536   # distinct transitions made per state; a larger ring holds copies of them


def _update(name, algo, prec, obs, act, hidden, batch, steps, rows, **kw):
    c = dict(name=name, kind="update", algo=algo, prec=prec, obs=obs, act=act, hidden=hidden, batch=batch,
             steps=steps, rows=rows, zeros=0, learn_alpha=True, streams=1, graphs=False, sequential=False, push=0)
    c.update(kw)
    return c


def _act(name, algo, prec, obs, act, hidden, n, **kw):
    c = dict(name=name, kind="act", algo=algo, prec=prec, obs=obs, act=act, hidden=hidden, n=n, device=True,
             stochastic=algo == "sac")
    c.update(kw)
    return c


def listed():
    return [
        # The smallest learner: a classic-control SAC, launch-bound, replayed from graphs.
        _update("sac_small", "sac", "fp32", 8, 2, "64-64", 256, 32, 10000, learn_alpha=False, graphs=True),
        # A ragged SAC with the default options (eager, two streams) in the published order
        # of updates: widths, batch and dimensions that are no multiple of anything.
        _update("sac_ragged_seq", "sac", "fp32", 27, 8, "200-120", 1000, 16, 50001, streams=2, sequential=True),
        # Walker-shaped SAC: float32, two 256-wide layers, an ordinary large batch.
        _update("sac_walker", "sac", "fp32", 17, 6, "256-256", 8192, 16, 262144, graphs=True),
        # Humanoid-shaped SAC with bfloat16 products, and the whole learner interval: new
        # experience pushed without waiting, updates, weights published.
        _update("sac_humanoid_cycle", "sac", "bf16", 376, 17, "256-256", 16384, 16, 262144, zeros=10, graphs=True,
                push=4096),
        # Ant-shaped TD3 in float32, 400-300 (ragged in tiles), delayed actor updates.
        _update("td3_ant", "td3", "fp32", 111, 8, "400-300", 32768, 8, 262144, graphs=True),
        # TD3 with bfloat16 products, default two streams, a batch between the others.
        _update("td3_bf16", "td3", "bf16", 45, 7, "256-256", 4096, 16, 262144, streams=2),
        # The large network at its per-GPU share of an eight-way data-parallel batch.
        _update("sac_large_16k", "sac", "bf16", 376, 17, "1024-1024-1024", 16384, 8, 262144, zeros=10),
        # The large network at its full batch: the benchmark's workload.
        _update("sac_large", "sac", "bf16", 376, 17, "1024-1024-1024", 131072, 8, 524288, zeros=10),
        # Actions for a handful of samplers in a serving loop: latency and launches.
        _act("act_few", "sac", "bf16", 376, 17, "256-256", 16),
        # The test process: mean actions from host observations, float32.
        _act("act_host", "sac", "fp32", 17, 6, "256-256", 1000, device=False, stochastic=False),
        # Actions for a large set of samplers through the large actor.
        _act("act_many", "sac", "bf16", 376, 17, "1024-1024-1024", 12288),
    ]


# Widths of hidden layers in use: powers of two, and the 400-300 and odd sizes of published
# and ragged configurations.
HIDDEN = {
    "small": ["32-32", "64-64", "100-50", "128-128", "64", "96-96-96"],
    "middle": ["256-256", "200-120", "256-128", "400-300", "192-192-192", "256-256-256", "320-320"],
    "large": ["512-512", "512-512-512", "768-768", "1024-1024", "1024-1024-1024", "640-640-640"],
}


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    while True:
        size = rng.choice(["small", "middle", "middle", "large"])
        prec = "bf16" if size == "large" else rng.choice(["fp32", "bf16"])
        algo = rng.choice(["sac", "sac", "td3"])
        obs, act = _log_int(rng, 3, 400), _log_int(rng, 1, 24)
        hidden = rng.choice(HIDDEN[size])
        if rng.random() < 0.25:
            c = _act("", algo, prec, obs, act, hidden, _log_int(rng, 1, 12288), device=rng.random() < 0.6)
            if c["stochastic"]:
                c["stochastic"] = rng.random() < 0.5
            del c["name"]
            return c
        batch = _log_int(rng, *{"small": (64, 8192), "middle": (512, 65536), "large": (2048, 131072)}[size])
        if rng.random() < 0.5:
            batch = max(64, batch // 256 * 256)
        steps = rng.choice([8, 16]) if batch < 32768 else rng.choice([4, 8])
        c = _update("", algo, prec, obs, act, hidden, batch, steps, rng.choice([10000, 50001, 131072, 262144]),
                    zeros=rng.choice([0, 10]), learn_alpha=rng.random() < 0.7, streams=rng.choice([1, 2]),
                    graphs=rng.random() < 0.5, sequential=rng.random() < 0.25,
                    push=rng.choice([0, 0, 0, 512, 4096]))
        del c["name"]
        largest = listed()[7]
        # float32 products run at about a sixteenth of the bfloat16 rate
        if work(c)["flops"] * (16 if prec == "fp32" else 1) <= work(largest)["flops"]:
            return c


# ------------------------------------------------------------------------------ the framework
def _widths(case):
    return [int(x) for x in case["hidden"].split("-")]


def _hparams(case):
    sac = case["algo"] == "sac"
    return dict(algo=case["algo"], gemm_prec=case["prec"], capacity=case.get("rows", 4096), gamma=GAMMA, tau=TAU,
                lr_actor=LR, lr_critic=LR, lr_alpha=LR, beta1=BETA1, beta2=BETA2, eps=EPS,
                alpha_init=_alpha0(case), learn_alpha=sac and case.get("learn_alpha", True),
                target_entropy=-float(case["act"]), log_std_min=LOG_STD[0], log_std_max=LOG_STD[1],
                policy_noise=SMOOTH, noise_clip=SMOOTH_CLIP, policy_delay=DELAY,
                ordering="sequential" if case.get("sequential") else "snapshot", graphs=case.get("graphs", False))


def _alpha0(case):
    if case["algo"] == "td3":
        return 0.0
    return 1.0 if case.get("learn_alpha", True) else 0.2


def _transitions(case, n, seed):
    """n float32 transitions (obs, act, rew, done, next_obs) on the GPU: normal observations and
    rewards, uniform actions, rare episode ends; humanoid-shaped observations have constant
    zero columns."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    o, a = case["obs"], case["act"]
    obs = torch.randn(n, o, device="cuda", generator=g)
    nobs = torch.randn(n, o, device="cuda", generator=g)
    act = torch.rand(n, a, device="cuda", generator=g) * 2 - 1
    rew = torch.randn(n, device="cuda", generator=g)
    done = (torch.rand(n, device="cuda", generator=g) < P_DONE).float()
    if case.get("zeros"):
        obs[:, ::case["zeros"]] = 0
        nobs[:, ::case["zeros"]] = 0
    return obs, act, rew, done, nobs


def _ring(case, seed):
    return _transitions(case, min(case["rows"], BASE_ROWS), 2 * seed)


def _host(arrays):
    return [x.cpu().numpy() for x in arrays]


def prepare(case, seed):
    spz = Spz(case["obs"], case["act"], _widths(case), case.get("batch", 4096), _hparams(case), seed=seed,
              n_streams=case.get("streams", 2))
    state = {"case": dict(case), "spz": spz}
    if case["kind"] == "act":
        obs = _observations(case, seed)
        state["obs"] = obs if case["device"] else obs.cpu().numpy()
        state["act"] = torch.empty(case["n"], case["act"], device="cuda") if case["device"] else None
        return state
    rows = _host(_ring(case, seed))
    n = rows[2].shape[0]
    for r0 in range(0, case["rows"], n):
        spz.buffer_push(*[x[:min(n, case["rows"] - r0)] for x in rows])
    state["push"] = _host(_transitions(case, case["push"], 2 * seed + 1)) if case["push"] else None
    return state


def _observations(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(case["n"], case["obs"], device="cuda", generator=g)


def run(state):
    case, spz = state["case"], state["spz"]
    if case["kind"] == "act":
        if not case["device"]:
            return spz.act(state["obs"], case["stochastic"], ACT_COUNTER)
        stream = torch.cuda.current_stream()
        spz.act_noalloc(state["obs"].data_ptr(), case["n"], state["act"].data_ptr(), case["stochastic"], ACT_COUNTER,
                        stream)
        return state["act"]
    if state["push"] is not None:
        spz.buffer_push_async(*state["push"])
    spz.update(case["steps"], torch.cuda.current_stream())
    losses = spz.read_losses(spz.step() - case["steps"] + 1, case["steps"])
    return {"first": losses[0], "later": losses[1:], "actor": spz.read_params("actor"),
            "critic1": spz.read_params("critic1"), "critic2": spz.read_params("critic2")}


# ------------------------------------------------------------------------------ what a pass cannot do without
def _nets(case):
    h = _widths(case)
    out = (2 if case["algo"] == "sac" else 1) * case["act"]
    return [case["obs"]] + h + [out], [case["obs"] + case["act"]] + h + [1]


def _macs(dims):
    return sum(i * o for i, o in zip(dims, dims[1:]))


def _count(dims):
    return sum((i + 1) * o for i, o in zip(dims, dims[1:]))


def work(case):
    da, dc = _nets(case)
    e = 2 if case["prec"] == "bf16" else 4
    if case["kind"] == "act":
        return {"bytes": case["n"] * (case["obs"] + case["act"]) * 4 + _count(da) * e,
                "flops": 2 * case["n"] * _macs(da)}
    fa, fc = _macs(da), _macs(dc)
    a1, c1 = da[0] * da[1], dc[0] * dc[1]   # first layers: no input gradient, but for the action's columns
    actor_passes = 1.0 if case["algo"] == "sac" else 1.0 / DELAY
    # target action and target critics; critics forward and backward
    macs = fa + 2 * fc + 2 * fc + 2 * (2 * fc - c1)
    # the actor's forward and backward, the critics on its action, the gradient through the
    # critic that attains the minimum (TD3: through critic 1)
    macs += actor_passes * (3 * fa - a1 + (2 if case["algo"] == "sac" else 1) * fc
                            + fc - c1 + case["act"] * dc[1])
    params = _count(da) + 2 * _count(dc)
    rows = case["batch"] * ((2 * case["obs"] + case["act"]) * e + 8)
    pushed = case["push"] * (2 * case["obs"] + case["act"] + 2) * (4 + e)
    # parameters, targets and both Adam moments read and written once, the weights read back
    return {"bytes": case["steps"] * rows + pushed + (2 * 4 + 1) * 4 * params,
            "flops": 2.0 * case["batch"] * case["steps"] * macs}


def tolerance(case):
    """About four times the largest distance from `exact` measured over the listed and drawn cases.

    Actions: 4e-3 (bfloat16), 3e-7 (float32). Weights after a few steps: up to 5e-3
    (bfloat16), 9e-5 (float32). A single weight may be off by much more than that: Adam's
    first steps have the size lr whatever the gradient, so an element whose gradient is within
    rounding of zero can go the other way, 2 lr a step (6e-4 against weights of rms 0.02 to
    0.2); "max" allows that for every step of two passes.
    """
    if case["kind"] == "act":
        return {"rel": 1.5e-2, "max": 0.2} if case["prec"] == "bf16" else {"rel": 1.2e-6, "max": 2e-5}
    return {"rel": 2e-2 if case["prec"] == "bf16" else 4e-4, "max": 0.9}


# ------------------------------------------------------------------------------ 64-bit values
_MASK = np.uint64(0xFFFFFFFF)


def _philox(seed, n, step, purpose, tensor=0):
    """The first n words of Philox4x32-10 at counters (i, step, purpose, tensor), key = seed."""
    u = np.uint64
    c0 = np.arange((n + 3) // 4, dtype=u)
    c1, c2, c3 = (np.full_like(c0, x) for x in (step, purpose, tensor))
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32
    for _ in range(10):
        p0, p1 = u(0xD2511F53) * c0, u(0xCD9E8D57) * c2
        c0, c1, c2, c3 = ((p1 >> u(32)) ^ c1 ^ u(k0), p1 & _MASK, (p0 >> u(32)) ^ c3 ^ u(k1), p0 & _MASK)
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return np.stack([c0, c1, c2, c3], axis=1).reshape(-1)[:n]


def _normals(seed, rows, cols, step, purpose):
    n = rows * cols
    w = (_philox(seed, (n + 3) // 4 * 4, step, purpose) >> np.uint64(8)).astype(np.float64).reshape(-1, 2, 2)
    w = torch.from_numpy(w).cuda()
    rad = torch.sqrt(-2.0 * torch.log((w[..., 0] + 1.0) * 2.0 ** -24))
    ang = 2.0 * math.pi * 2.0 ** -24 * w[..., 1]
    return torch.stack([rad * torch.cos(ang), rad * torch.sin(ang)], dim=-1).reshape(-1)[:n].reshape(rows, cols)


def _init(seed, net, dims):
    layers = []
    for i, (fan_in, out) in enumerate(zip(dims, dims[1:])):
        k = float(np.float32(1.0 / math.sqrt(fan_in)))
        pair = []
        for b, shape in enumerate([(out, fan_in), (out,)]):
            w = _philox(seed, math.prod(shape), 0, 0, net * 16 + 2 * i + b) >> np.uint64(8)
            v = ((2.0 * (w.astype(np.float64) * 2.0 ** -24) - 1.0) * k).astype(np.float32)
            pair.append(torch.from_numpy(v.reshape(shape)).cuda().double())
        layers.append(pair)
    return layers


def _mlp(layers, x):
    for i, (w, b) in enumerate(layers):
        x = torch.addmm(b, x, w.t())
        if i + 1 < len(layers):
            x = torch.relu(x)
    return x


def _policy(layers, s, eps, a):
    z = _mlp(layers, s)
    mu, ls = z[:, :a], torch.clamp(z[:, a:], *LOG_STD)
    u = mu + torch.exp(ls) * eps
    logp = (-0.5 * eps * eps - ls - 0.5 * math.log(2 * math.pi)
            - 2.0 * (math.log(2.0) - u - torch.nn.functional.softplus(-2.0 * u))).sum(1)
    return torch.tanh(u), logp


class _Adam:
    def __init__(self, params):
        self.p, self.t = params, 0
        self.m = [torch.zeros_like(x) for x in params]
        self.v = [torch.zeros_like(x) for x in params]

    def step(self, grads):
        self.t += 1
        for p, m, v, g in zip(self.p, self.m, self.v, grads):
            m.mul_(BETA1).add_(g, alpha=1 - BETA1)
            v.mul_(BETA2).addcmul_(g, g, value=1 - BETA2)
            p.sub_(LR * (m / (1 - BETA1 ** self.t)) / (torch.sqrt(v / (1 - BETA2 ** self.t)) + EPS))


def _flat(layers):
    return [x for pair in layers for x in pair]


def _grads(loss, params):
    return torch.autograd.grad(loss, params)


def _learner(case, seed):
    """The update steps in float64: the loss records and the flat weights of actor and critics."""
    da, dc = _nets(case)
    sac, a, batch = case["algo"] == "sac", case["act"], case["batch"]
    actor = _init(seed, 0, da)
    critics = [_init(seed, 1 + k, dc) for k in range(2)]
    tcritics = [[[x.clone() for x in pair] for pair in net] for net in critics]
    tactor = [[x.clone() for x in pair] for pair in actor]
    log_alpha = torch.full((1,), math.log(_alpha0(case)) if sac else 0.0, dtype=torch.float64, device="cuda")
    learn_alpha = sac and case["learn_alpha"]
    opt_a, opt_c, opt_al = _Adam(_flat(actor)), _Adam(_flat(critics[0]) + _flat(critics[1])), _Adam([log_alpha])
    base = [x.double() for x in _ring(case, seed)]
    pushed = [x.double() for x in _transitions(case, case["push"], 2 * seed + 1)] if case["push"] else None
    n0, size = base[2].shape[0], case["rows"]
    records = []
    for t in range(1, case["steps"] + 1):
        idx = (_philox(seed, batch, t, 1) * np.uint64(size)) >> np.uint64(32)
        idx = torch.from_numpy(idx.astype(np.int64)).cuda()
        rows = [x[idx % n0] for x in base]
        if pushed is not None:   # the full ring's oldest rows were overwritten
            new = (idx < case["push"]).nonzero()[:, 0]
            for x, p in zip(rows, pushed):
                x[new] = p[idx[new]]
        s, act, r, d, s2 = rows
        alpha = math.exp(float(log_alpha)) if sac else 0.0
        eps2 = _normals(seed, batch, a, t, 2)
        with torch.no_grad():
            if sac:
                a2, logp2 = _policy(actor, s2, eps2, a)
            else:
                noise = torch.clamp(SMOOTH * eps2, -SMOOTH_CLIP, SMOOTH_CLIP)
                a2, logp2 = torch.clamp(torch.tanh(_mlp(tactor, s2)) + noise, -1.0, 1.0), 0.0
            x2 = torch.cat([s2, a2], 1)
            qt = [_mlp(net, x2)[:, 0] for net in tcritics]
            y = r + GAMMA * (1 - d) * (torch.minimum(*qt) - alpha * logp2)
            x = torch.cat([s, act], 1)
        lq, q1, gc = 0.0, None, []
        for net in critics:
            for p in _flat(net):
                p.requires_grad_(True)
            q = _mlp(net, x)[:, 0]
            loss = ((q - y) ** 2).mean()
            gc += _grads(loss, _flat(net))
            lq += float(loss)
            q1 = float(q.mean()) if q1 is None else q1
            for p in _flat(net):
                p.requires_grad_(False)
        if case["sequential"]:
            opt_c.step(gc)
        rec = [lq, 0.0, 0.0, alpha, 0.0, q1, 0.0, 0.0]
        actor_step = sac or t % DELAY == 0
        if actor_step:
            for p in _flat(actor):
                p.requires_grad_(True)
            if sac:
                ap, logp = _policy(actor, s, _normals(seed, batch, a, t, 3), a)
                qp = [_mlp(net, torch.cat([s, ap], 1))[:, 0] for net in critics]
                loss = (alpha * logp - torch.where(qp[0] <= qp[1], qp[0], qp[1])).mean()
                mean_logp = float(logp.mean())
                rec[2], rec[4] = -float(log_alpha) * (mean_logp - a), mean_logp
            else:
                loss = -_mlp(critics[0], torch.cat([s, torch.tanh(_mlp(actor, s))], 1))[:, 0].mean()
            ga = _grads(loss, _flat(actor))
            rec[1], rec[7] = float(loss), 1.0
            for p in _flat(actor):
                p.requires_grad_(False)
        if not case["sequential"]:
            opt_c.step(gc)
        if actor_step:
            opt_a.step(ga)
            if learn_alpha:
                opt_al.step([torch.full_like(log_alpha, -(mean_logp - a))])
            pairs = list(zip(tcritics, critics)) + ([] if sac else [(tactor, actor)])
            for tgt, net in pairs:
                for tp, p in zip(_flat(tgt), _flat(net)):
                    tp.mul_(1 - TAU).add_(p, alpha=TAU)
        records.append(rec)
    weights = [torch.cat([x.reshape(-1) for x in _flat(net)]).cpu().numpy() for net in [actor] + critics]
    return np.array(records), weights


def exact(case, seed):
    if case["kind"] == "act":
        actor = _init(seed, 0, _nets(case)[0])
        obs = _observations(case, seed).double()
        if not case["stochastic"]:
            out = torch.tanh(_mlp(actor, obs)[:, :case["act"]])
        else:
            out = _policy(actor, obs, _normals(seed, case["n"], case["act"], ACT_COUNTER, 4), case["act"])[0]
        return out if case["device"] else out.cpu().numpy()
    records, weights = _learner(case, seed)
    out = {"first": records[0], "later": records[1:], "actor": weights[0], "critic1": weights[1],
           "critic2": weights[2]}
    # A ReLU whose input is within float32 rounding of zero may be open in one computation and
    # closed in the other. Over about a million units and more some are, a few at a time, and
    # what they do to Adam's steps (1e-7 without them, 1e-5 to 1e-4 with) says nothing about
    # precision: such float32 runs have a 64-bit value only before their first weight step.
    # (In bfloat16 thousands of units differ, and the distance is a steady one.)
    if case["prec"] == "fp32" and case["batch"] * case["steps"] * sum(_widths(case)) > 4e6:
        out.update({k: None for k in out if k != "first"})
    return out
