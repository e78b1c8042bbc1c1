"""The calls that the library's speed is measured on, and the ranges they stand for.

Each case is one call of a public entry point on inputs a training program has in GPU memory:
row-major rollout buffers from a handful of environments to tens of thousands, time-major
buffers, long token rows, the action-axis form of Retrace, masked and whitened GAE, and traces of
feature vectors. Outputs are allocated by the call, as the binding does by default; a workspace
is made once in ``prepare`` where the call documents one, as a training loop keeps it.

Sizes are those of ``workloads.CONFIGS`` and of ``bench.py --extra``, or plain odd ones.
"""
import math

import torch

import paper_2608_17641_amd as rl

GAMMA, LAM = 0.99, 0.95
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
LINE = 128  # bytes of a cache line: the smallest piece a sparse read brings in

# estimator -> ([N, T] data inputs beside the continuation, outputs, whether it bootstraps)
ESTIMATORS = {
    "gae": (("r", "v"), 2, True),
    "vtrace": (("r", "v", "log_rho"), 2, True),
    "retrace": (("r", "q", "eq", "log_rho"), 2, True),
    "td_lambda": (("r", "v"), 1, True),
    "discounted": (("r",), 1, True),
    "elig_trace": (("x",), 1, False),
    "episodic_prefix": (("x",), 1, False),
}


def listed():
    return [
        # the classic on-policy setting: a few environments, a short rollout (latency only)
        dict(name="gae_8x128_f32", kind="rows", est="gae", N=8, T=128, dtype="f32",
             p_term=0.01, p_trunc=0.0),
        # thousands of simulated environments, short rollouts, forward direction
        dict(name="elig_4096x32_f32", kind="rows", est="elig_trace", N=4096, T=32, dtype="f32",
             p_term=0.02, p_trunc=0.01),
        # the benchmark's headline: thousands of environments, 256 steps, truncations
        dict(name="gae_4096x256_f32", kind="rows", est="gae", N=4096, T=256, dtype="f32",
             p_term=0.02, p_trunc=0.01),
        # token-level returns of a language-model batch: few rows, each long, flag at the end
        dict(name="td_rlhf_64x4096_f32", kind="rlhf", est="td_lambda", N=64, T=4096, dtype="f32"),
        # the same rollout as the headline in the [T, N] buffers that most PPO code keeps
        dict(name="gae_tm_256x4096_f32", kind="time_major", est="gae", N=4096, T=256, dtype="f32",
             p_term=0.02, p_trunc=0.01),
        # an off-policy learner's time-major batch in bfloat16, a round decimal environment count
        dict(name="vtrace_tm_100x10000_bf16", kind="time_major", est="vtrace", N=10000, T=100,
             dtype="bf16", p_term=0.005, p_trunc=0.005),
        # episodes cut at an odd step count: no row starts on a vector but one in four
        dict(name="vtrace_4096x2001_f32", kind="rows", est="vtrace", N=4096, T=2001, dtype="f32",
             p_term=0.02, p_trunc=0.01),
        # replay segments in bfloat16, the estimator with the most inputs
        dict(name="retrace_16384x512_bf16", kind="rows", est="retrace", N=16384, T=512,
             dtype="bf16", p_term=0.005, p_trunc=0.005),
        # the largest rollout of the bfloat16 sweep
        dict(name="gae_65536x2048_bf16", kind="rows", est="gae", N=65536, T=2048, dtype="bf16",
             p_term=0.005, p_trunc=0.005),
        # Q-values and policies over an 18-action discrete space
        dict(name="retrace_full_4096x256x18_f32", kind="retrace_full", N=4096, T=256, A=18,
             dtype="f32", p_term=0.02, p_trunc=0.01),
        # multi-turn tool-use rows: observation tokens skipped, advantages whitened
        dict(name="masked_norm_1024x2048_f32", kind="masked", N=1024, T=2048, dtype="f32",
             normalize=True),
        # eligibility traces of a linear value function's 256 features
        dict(name="elig_vec_64x1024x256_f32", kind="vec", N=64, T=1024, F=256, dtype="f32",
             p_term=0.02, p_trunc=0.01),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _rows(rng, T, most):
    """Environments beside T steps: up to `most` steps in all."""
    return max(1, min(65536, _log_int(rng, max(8, min(1024, most // T)), max(16, most // T))))


def draw(rng):
    kind = rng.choice(["rows", "rows", "rows", "rlhf", "time_major", "time_major", "strided_rows",
                       "retrace_full", "masked", "vec"])
    dtype = rng.choice(["f32", "f32", "bf16"])
    flags = dict(p_term=rng.choice([0.005, 0.02]), p_trunc=rng.choice([0.0, 0.005, 0.01]))
    if kind == "rows" or kind == "strided_rows" or kind == "time_major":
        T = _log_int(rng, 16, 4096)
        names = list(ESTIMATORS) if kind == "rows" else ["gae", "vtrace", "td_lambda", "elig_trace"]
        case = dict(kind=kind, est=rng.choice(names), N=_rows(rng, T, 1 << 25), T=T, dtype=dtype, **flags)
        if kind == "strided_rows":  # the first T steps of wider rows
            case["ld"] = T + rng.choice([1, 4, 8, 64])
        return case
    if kind == "rlhf":
        return dict(kind=kind, est=rng.choice(["gae", "td_lambda"]), N=_log_int(rng, 4, 512),
                    T=_log_int(rng, 512, 32768), dtype=dtype)
    if kind == "retrace_full":
        T, A = _log_int(rng, 32, 1024), _log_int(rng, 2, 64)
        return dict(kind=kind, N=_rows(rng, T, (1 << 26) // A), T=T, A=A, dtype=dtype, **flags)
    if kind == "masked":
        return dict(kind=kind, N=_log_int(rng, 16, 2048), T=_log_int(rng, 256, 8192), dtype=dtype,
                    normalize=rng.random() < 0.5)
    F = rng.choice([1, 3, 8, 16, 33, 64, 100, 256])
    T = _log_int(rng, 16, 1024)
    return dict(kind="vec", N=max(1, min(4096, _log_int(rng, 8, (1 << 25) // (T * F) + 9))), T=T, F=F,
                dtype=dtype, **flags)


# ---------------------------------------------------------------- inputs

def _normal(g, shape, dtype, scale=1.0):
    return (scale * torch.randn(shape, device="cuda", generator=g)).to(dtype)


def _flag(g, shape, p):
    return (torch.rand(shape, device="cuda", generator=g) < p).to(torch.uint8)


def _stored(case, t):
    """An [N, T] tensor in the layout the case keeps its buffers in."""
    if case["kind"] == "time_major":
        return t.t().contiguous().t()
    if case["kind"] == "strided_rows":
        wide = torch.zeros((t.shape[0], case["ld"]), dtype=t.dtype, device=t.device)
        wide[:, :t.shape[1]] = t
        return wide[:, :t.shape[1]]
    return t


def _multiturn_mask(g, N, T):
    """Alternating runs of observation (mean 96) and action (mean 48) tokens, observation first."""
    runs = 2 * (T // 72) + 32
    u = torch.rand((N, runs), device="cuda", generator=g).clamp_(min=1e-7)
    mean = torch.tensor([96.0, 48.0], device="cuda").repeat(runs // 2)
    ends = torch.cumsum(1 + torch.floor(torch.log(u) / torch.log1p(-1.0 / mean)), dim=1)
    steps = torch.arange(T, device="cuda", dtype=torch.float32).expand(N, T).contiguous()
    return (torch.searchsorted(ends, steps, right=True) % 2).to(torch.uint8)


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    dt, kind, N, T = DTYPES[case["dtype"]], case["kind"], case["N"], case["T"]
    s = dict(case=case, ws=None)
    p_term, p_trunc = case.get("p_term", 0.0), case.get("p_trunc", 0.0)
    if kind == "vec":
        s.update(x=_normal(g, (N, T, case["F"]), dt), term=_flag(g, (N, T), p_term),
                 trunc=_flag(g, (N, T), p_trunc) if p_trunc else None,
                 ws=rl.make_workspace_columns(N * case["F"], T, "cuda"))
        return s
    if kind in ("rlhf", "masked"):
        # a per-token penalty, a score on the row's last token, which ends the episode
        r = 0.01 * torch.randn((N, T), device="cuda", generator=g)
        term = torch.zeros((N, T), dtype=torch.uint8, device="cuda")
        term[:, -1] = 1
        if kind == "masked":
            s["mask"] = _multiturn_mask(g, N, T)
            r *= s["mask"]
            if case["normalize"]:
                s["ws"] = torch.zeros(max(64, rl.rlcs_workspace_size_masked(N, T)), dtype=torch.uint8,
                                      device="cuda")
        elif T > 4096:
            s["ws"] = rl.make_workspace(N, T, "cuda")
        r[:, -1] += torch.randn((N,), device="cuda", generator=g)
        s.update(r=r.to(dt), v=_normal(g, (N, T), dt), term=term, trunc=None, bv=None, boot=None)
        return s
    s["boot"] = _normal(g, (N,), dt)
    s["term"] = _stored(case, _flag(g, (N, T), p_term))
    s["trunc"] = _stored(case, _flag(g, (N, T), p_trunc)) if p_trunc else None
    s["bv"] = _stored(case, _normal(g, (N, T), dt)) if p_trunc else None
    if kind == "retrace_full":
        A = case["A"]
        s["r"] = _normal(g, (N, T), dt)
        s["q"] = _normal(g, (N, T, A), dt)
        s["pi"] = torch.softmax(torch.randn((N, T, A), device="cuda", generator=g), dim=-1).to(dt)
        behaviour = torch.softmax(torch.randn((N, T, A), device="cuda", generator=g), dim=-1)
        u = torch.rand((N, T, 1), device="cuda", generator=g)
        taken = (behaviour.cumsum(-1) < u).sum(-1, keepdim=True).clamp_(max=A - 1)
        s["mu"] = behaviour.gather(-1, taken)[..., 0].clamp_(min=1e-6).to(dt)
        s["actions"] = taken[..., 0].to(torch.int32)
        return s
    names = ESTIMATORS[case["est"]][0]
    for name in names:
        # log-ratios of two policies' log-probabilities, each N(0, 0.5)
        s[name] = _stored(case, _normal(g, (N, T), dt, math.sqrt(0.5) if name == "log_rho" else 1.0))
    if kind == "time_major":
        s["ws"] = rl.make_workspace_columns(N, T, "cuda")
    return s


# ---------------------------------------------------------------- the call

def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "vec":
        return rl.rlcs_elig_trace_vec(s["x"], s["term"], s["trunc"], gamma=GAMMA, lam=LAM, ws=s["ws"])
    if kind == "retrace_full":
        return rl.rlcs_retrace_full(s["r"], s["q"], s["pi"], s["actions"], s["mu"], s["term"], s["trunc"],
                                    s["bv"], s["boot"], gamma=GAMMA, lam=LAM)
    if kind == "masked":
        return rl.rlcs_gae_masked(s["r"], s["v"], s["mask"], s["term"], gamma=1.0, lam=LAM,
                                  normalize=c["normalize"], ws=s["ws"])
    gamma = 1.0 if kind == "rlhf" else GAMMA
    strided = kind in ("time_major", "strided_rows")
    est = c["est"]
    if est == "gae":
        f = rl.rlcs_gae_strided if strided else rl.rlcs_gae
        return f(s["r"], s["v"], s["term"], s["trunc"], s["bv"], s["boot"], gamma=gamma, lam=LAM, ws=s["ws"])
    if est == "vtrace":
        f = rl.rlcs_vtrace_strided if strided else rl.rlcs_vtrace
        return f(s["r"], s["v"], s["log_rho"], s["term"], s["trunc"], s["bv"], s["boot"], gamma=gamma, ws=s["ws"])
    if est == "retrace":
        return rl.rlcs_retrace(s["r"], s["q"], s["eq"], s["log_rho"], s["term"], s["trunc"], s["bv"], s["boot"],
                               gamma=gamma, lam=LAM, ws=s["ws"])
    if est == "td_lambda":
        f = rl.rlcs_td_lambda_strided if strided else rl.rlcs_td_lambda
        return f(s["r"], s["v"], s["term"], s["trunc"], s["bv"], s["boot"], gamma=gamma, lam=LAM, ws=s["ws"])
    if est == "discounted":
        return rl.rlcs_discounted(s["r"], s["term"], s["trunc"], s["bv"], s["boot"], gamma=gamma, ws=s["ws"])
    if est == "elig_trace":
        f = rl.rlcs_elig_trace_strided if strided else rl.rlcs_elig_trace
        return f(s["x"], s["term"], s["trunc"], gamma=gamma, lam=LAM, ws=s["ws"])
    return rl.rlcs_episodic_prefix(s["x"], s["term"], s["trunc"], ws=s["ws"])


# ---------------------------------------------------------------- what a pass cannot do without

def work(case):
    es = 4 if case["dtype"] == "f32" else 2
    steps, kind = case["N"] * case["T"], case["kind"]
    p_trunc = case.get("p_trunc", 0.0)
    flags = 2 if p_trunc else 1
    if kind == "vec":
        return {"bytes": steps * (case["F"] * (es + 4) + flags), "flops": 2.0 * steps * case["F"]}
    if kind == "masked":
        return {"bytes": steps * (2 * es + 2 + 8), "flops": 8.0 * steps}
    # continuations: the lines of 128 bytes that hold a truncated step
    cont = es * (1.0 - (1.0 - p_trunc) ** (LINE // es))
    if kind == "retrace_full":
        return {"bytes": steps * (2 * es * case["A"] + 2 * es + 4 + flags + cont + 8) + case["N"] * es,
                "flops": steps * (2.0 * case["A"] + 8)}
    names, outs, boots = ESTIMATORS[case["est"]]
    boot = case["N"] * es if boots and kind != "rlhf" else 0
    return {"bytes": steps * (len(names) * es + flags + (cont if boots else 0) + 4 * outs) + boot,
            "flops": 8.0 * steps}


def tolerance(case):
    # All arithmetic and every output is float32 whatever the inputs' type: measured against 64
    # bits 5e-8 to 7e-7 (2-norm).
    return {"rel": 3e-6, "max": 5e-5}


# ---------------------------------------------------------------- the same in 64 bits

def _f32(x):
    """A parameter as the C interface takes it."""
    return float(torch.tensor(x, dtype=torch.float32))


def _wide(t):
    """[N, ...] input as contiguous float64 with time first: [T, N]."""
    return None if t is None else t.t().to(torch.float64).contiguous()


def _backward(alpha, beta):
    """A_t = alpha_t + beta_t A_{t+1}, in place of alpha; A past the end is 0."""
    for t in range(alpha.shape[0] - 2, -1, -1):
        alpha[t].addcmul_(beta[t], alpha[t + 1])
    return alpha


def _successor(nxt, boot, term, trunc, bv):
    """The value after each step: the next one's, the bootstrap at the window's edge, the
    continuation after a truncation, 0 after a termination."""
    edge = boot.to(torch.float64)[None] if boot is not None else torch.zeros_like(nxt[:1])
    s = torch.cat([nxt[1:], edge])
    if trunc is not None:
        s = torch.where(trunc, bv, s)
    return s.masked_fill_(term, 0.0)


def exact(case, seed):
    if case["T"] > 65536:
        return None
    s = prepare(case, seed)
    kind, lam = case["kind"], _f32(LAM)
    gamma = 1.0 if kind in ("rlhf", "masked") else _f32(GAMMA)
    if kind == "vec":
        x = s["x"].to(torch.float64)
        done = s["term"] != 0
        if s["trunc"] is not None:
            done = done | (s["trunc"] != 0)
        keep = gamma * lam * (~done).to(torch.float64)[..., None]
        for t in range(1, case["T"]):
            x[:, t] += keep[:, t - 1] * x[:, t - 1]
        return x
    term = s["term"].t() != 0
    trunc = None if s["trunc"] is None else s["trunc"].t() != 0
    done = term if trunc is None else term | trunc
    out = lambda a: a.t()  # noqa: E731
    if kind == "masked":
        r, v, mask = _wide(s["r"]), _wide(s["v"]), s["mask"].t() != 0
        adv = torch.empty_like(r)
        a, w = torch.zeros_like(r[0]), torch.zeros_like(r[0])
        for t in range(case["T"] - 1, -1, -1):
            a, w = a.masked_fill(done[t], 0.0), w.masked_fill(done[t], 0.0)
            new = r[t] + gamma * w - v[t] + gamma * lam * a
            a, w = torch.where(mask[t], new, a), torch.where(mask[t], v[t], w)
            adv[t] = a
        ret = adv + v
        if case["normalize"]:
            part = adv[mask]
            mean = part.mean() if part.numel() else 0.0
            var = part.var() if part.numel() > 1 else torch.zeros((), dtype=torch.float64, device=adv.device)
            adv = (adv - mean) / torch.sqrt(var + _f32(1e-8))
        return out(adv), out(ret)
    bv, boot = _wide(s["bv"]), s["boot"] if "boot" in s else None
    keep = (~done).to(torch.float64)
    if kind == "retrace_full":
        q, pi = s["q"].to(torch.float64), s["pi"].to(torch.float64)
        at = s["actions"].long()[..., None]
        r, eq, qa = _wide(s["r"]), (q * pi).sum(-1).t().contiguous(), q.gather(-1, at)[..., 0].t().contiguous()
        c = lam * torch.clamp(pi.gather(-1, at)[..., 0].t() / _wide(s["mu"]), max=1.0)
        alpha = r + gamma * _successor(eq, boot, term, trunc, bv) - qa
        delta = _backward(alpha, gamma * keep * torch.cat([c[1:], torch.zeros_like(c[:1])]))
        return out(delta), out(qa + delta)
    est = case["est"]
    if est in ("elig_trace", "episodic_prefix"):
        x, decay = _wide(s["x"]), gamma * lam if est == "elig_trace" else 1.0
        for t in range(1, case["T"]):
            x[t] += decay * keep[t - 1] * x[t - 1]
        return out(x)
    r = _wide(s["r"])
    if est == "discounted":
        last = torch.zeros_like(r)
        return out(_backward(r + gamma * _successor(last, boot, term, trunc, bv), gamma * keep))
    if est == "retrace":
        q, eq = _wide(s["q"]), _wide(s["eq"])
        c = lam * torch.clamp(torch.exp(_wide(s["log_rho"])), max=1.0)
        alpha = r + gamma * _successor(eq, boot, term, trunc, bv) - q
        delta = _backward(alpha, gamma * keep * torch.cat([c[1:], torch.zeros_like(c[:1])]))
        return out(delta), out(q + delta)
    v = _wide(s["v"])
    succ = _successor(v, boot, term, trunc, bv)
    if est == "gae":
        adv = _backward(r + gamma * succ - v, gamma * lam * keep)
        return out(adv), out(adv + v)
    if est == "td_lambda":
        # full discount on continuations and on the window's edge
        full = torch.zeros_like(done) if trunc is None else trunc.clone()
        full[-1] = True
        alpha = r + torch.where(full, gamma, gamma * (1.0 - lam)) * succ
        return out(_backward(alpha, gamma * lam * keep))
    rho = torch.clamp(torch.exp(_wide(s["log_rho"])), max=1.0)
    vs = v + _backward(rho * (r + gamma * succ - v), gamma * rho * keep)
    pg = rho * (r + gamma * _successor(vs, boot, term, trunc, bv) - v)
    return out(vs), out(pg)
