"""The framework's work as its users have it done, one case per use.

A case names a path (``kind``), the networks it runs (``net``), their
arithmetic (``compute``) and the sizes.  ``listed`` holds the cases that are
followed one by one; ``draw`` gives others of the same ranges.  Networks are
random with the benchmark's shapes and scales: time and rounding depend on
the shapes, not on trained values.

``exact`` evaluates the same definitions in binary64 with plain torch.
"""
import math

import numpy as np
import torch

import paper_2606_19729_amd as V

# d_s, discrete actions (0: continuous), d_a, d_w, d_o, d_wz, hidden layers of the samplers, of the likelihood
NETS = {
    "small": (4, 5, 0, 4, 2, 2, [64, 64], [64, 64]),
    "continuous": (4, 0, 4, 4, 2, 2, [64, 64], [64, 64]),
    "realistic": (16, 0, 4, 16, 32, 32, [256] * 3, [256] * 3),
    "wide": (4, 5, 0, 4, 2, 2, [1024] * 2, [1024] * 2),
    "target_finding": (45, 6, 0, 45, 36, 36, [1024] * 4, [256] * 3),
}
# denoisers of the teacher samplers: d_x, d_c, discrete actions, d_a, hidden layers
DENOISERS = {
    "transition": (4, 4, 5, 0, [1024] * 5),
    "distilled_shape": (4, 4, 5, 0, [1024] * 4),
    "observation": (32, 16, 0, 4, [512] * 5),
    "latent": (64, 44, 6, 0, [512] * 5),
}
STREAM_PLAN, STREAM_OBSERVE, STREAM_UPDATE, STREAM_BRANCH = 3, 4, 5, 6


def listed():
    return [
        # one decision of a small planner: a call that is all launch latency
        dict(name="plan_small_f32", kind="plan", net="small", compute="f32", K=32, N=128, H=10, weighted=False),
        # the belief update that follows every executed action, at the benchmark's belief size
        dict(name="update_realistic_f32", kind="update", net="realistic", compute="f32", N=4096),
        # the headline workload: every candidate x every particle x the horizon
        dict(name="plan_realistic_f32", kind="plan", net="realistic", compute="f32", K=1024, N=4096, H=20,
             weighted=False),
        # forward simulation with states and observations kept, in bfloat16, at sizes that fill no tile evenly
        dict(name="simulate_realistic_bf16", kind="simulate", net="realistic", compute="bf16", K=500, N=2000, H=20),
        # the paper's target-finding task through its four-layer samplers, weighted belief
        dict(name="plan_target_finding_bf16", kind="plan", net="target_finding", compute="bf16", K=100, N=1000, H=20,
             weighted=True),
        # uneven planning instances of a multi-agent program, planned and updated in one captured graph
        dict(name="batch_small_bf16", kind="batch", net="small", compute="bf16", n=12, n_lo=256, n_hi=8192, h_lo=5,
             h_hi=30, k_lo=64, k_hi=1024),
        # one grouped widening step of the tree search: thousands of action nodes with uneven successor counts
        dict(name="widen_realistic_bf16", kind="widen", net="realistic", compute="bf16", M=4096, group=1024),
        # one training step's gradient of the distillation loss
        dict(name="distill_small_f32", kind="distill", net="small", compute="f32", B=65536, H=20),
        # one training step's gradient of the likelihood network, large batch in bfloat16
        dict(name="contrast_realistic_bf16", kind="contrast", net="realistic", compute="bf16", B=4096),
        # the same in binary32 on a batch that is no multiple of a tile
        dict(name="contrast_realistic_f32", kind="contrast", net="realistic", compute="f32", B=1000),
        # sampling the transition teacher for a distillation data set
        dict(name="teacher_transition_bf16", kind="teacher", net="transition", compute="bf16", N=20000, steps=50),
        # reweighting and resampling a very large belief whose log-likelihoods are at hand
        dict(name="reweight_large", kind="reweight", net="", compute="f32", N=1 << 24, rows=16, weighted=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["plan", "plan", "plan", "update", "update", "simulate", "batch", "widen", "distill", "return",
                       "contrast", "contrast", "teacher", "reweight"])
    while True:
        c = dict(kind=kind)
        if kind == "plan":
            c["net"] = rng.choice(["small", "continuous", "realistic", "wide", "target_finding"])
            c["compute"] = "bf16" if c["net"] in ("wide", "target_finding") else rng.choice(["f32", "bf16"])
            c.update(K=_log(rng, 8, 1024), N=_log(rng, 64, 8192), H=rng.randint(5, 30),
                     weighted=rng.random() < 0.5)
        elif kind == "update":
            c["net"] = rng.choice(["small", "realistic", "wide", "target_finding"])
            c["compute"] = "bf16" if c["net"] in ("wide", "target_finding") else rng.choice(["f32", "bf16"])
            c["N"] = _log(rng, 64, 65536)
        elif kind == "simulate":
            c["net"] = rng.choice(["small", "realistic"])
            c["compute"] = rng.choice(["f32", "bf16"])
            c.update(K=_log(rng, 8, 512), N=_log(rng, 64, 4096), H=rng.randint(5, 30))
        elif kind == "batch":
            c.update(net="small", compute=rng.choice(["f32", "bf16"]), n=rng.randint(2, 12), n_lo=256,
                     n_hi=_log(rng, 512, 8192), h_lo=5, h_hi=rng.randint(8, 30), k_lo=64, k_hi=_log(rng, 128, 1024))
        elif kind == "widen":
            c.update(net=rng.choice(["small", "realistic"]), compute=rng.choice(["f32", "bf16"]),
                     M=_log(rng, 64, 4096), group=_log(rng, 64, 1024))
        elif kind == "distill":
            c.update(net="small", compute="f32", B=_log(rng, 1024, 65536), H=rng.randint(5, 25))
        elif kind == "return":
            c.update(net="continuous", compute="f32", B=64 * _log(rng, 16, 1024), H=rng.randint(5, 25))
        elif kind == "contrast":
            c["net"] = rng.choice(["small", "realistic", "realistic"])
            c["compute"] = "f32" if c["net"] == "small" else rng.choice(["f32", "bf16"])
            c["B"] = _log(rng, 64, 4096)
        elif kind == "teacher":
            c["net"] = rng.choice(sorted(DENOISERS))
            c.update(compute="bf16", N=_log(rng, 256, 32768), steps=1 if c["net"] == "distilled_shape"
                     else rng.randint(10, 50))
        else:
            c.update(net="", compute="f32", N=_log(rng, 1024, 1 << 24), rows=rng.choice([4, 16, 45]),
                     weighted=rng.random() < 0.5)
        w = work(c)
        if w["flops"] <= 2.3e13 and w["bytes"] <= 8e9:
            return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
class Desc:
    """Shapes and parameters of the networks, as paper_2606_19729_amd.Model takes them."""


def _mlp(rng, dims, gain=1.0, bias=None):
    out = []
    for j, (n_in, n_out) in enumerate(zip(dims[:-1], dims[1:])):
        sd = math.sqrt((gain if j < len(dims) - 2 else 1.0) / n_in)
        out.append((rng.standard_normal((n_out, n_in), dtype=np.float32) * np.float32(sd),
                    rng.standard_normal(n_out, dtype=np.float32) * np.float32(sd if bias is None else bias)))
    return out


def _desc(net, rng):
    d = Desc()
    d.d_s, d.n_actions, d.d_a, d.d_w, d.d_o, d.d_wz, hid, lik = NETS[net]
    aw = d.n_actions or d.d_a
    d.trans = _mlp(rng, [d.d_s + aw + d.d_w] + hid + [d.d_s])
    d.obs = _mlp(rng, [d.d_s + aw + d.d_wz] + hid + [d.d_o])
    d.lik = _mlp(rng, [d.d_s + aw + d.d_o] + lik + [1])
    return d


def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a), device="cuda")


def _belief(rng, N, d_s):
    """Most of the belief near its mean, a fifth spread out (particles the last update brought in)."""
    s = rng.standard_normal((N, d_s), dtype=np.float32)
    n = N // 5
    s[N - n:] = rng.uniform(-3.0, 3.0, (n, d_s)).astype(np.float32)
    return s


def _actions(rng, d, shape):
    if d.n_actions:
        return rng.integers(0, d.n_actions, shape).astype(np.int32)
    return rng.uniform(-1.0, 1.0, tuple(shape) + (d.d_a,)).astype(np.float32)


def _goal(rng, d):
    g = np.zeros(d.d_s, np.float32)
    g[:2] = 1.0
    return g + 0.1 * rng.standard_normal(d.d_s).astype(np.float32)


def _seed(rng):
    return int(rng.integers(1, 2**63))


def _u32(rng, n):
    return rng.integers(0, 2**32, n, dtype=np.uint64).astype(np.uint32)


def _instance(case, rng):
    """One batched instance: its own networks, belief, candidates and update."""
    N = int(rng.integers(case["n_lo"], case["n_hi"] + 1))
    H = int(rng.integers(case["h_lo"], case["h_hi"] + 1))
    K = int(rng.integers(case["k_lo"], case["k_hi"] + 1))
    d = _desc(case["net"], rng)
    return dict(d=d, S=_belief(rng, N, d.d_s), C=_actions(rng, d, (K, H)), goal=_goal(rng, d), seed=_seed(rng),
                update_seed=_seed(rng), action=_actions(rng, d, (1,)),
                obs=rng.standard_normal(d.d_o).astype(np.float32), U=_u32(rng, 1))


def _sizes(case):
    """Instance sizes of a batched case (those of seed 0: the amount of work only)."""
    out, rng = [], np.random.default_rng(0)
    for _ in range(case["n"]):
        N = int(rng.integers(case["n_lo"], case["n_hi"] + 1))
        H = int(rng.integers(case["h_lo"], case["h_hi"] + 1))
        out.append((N, int(rng.integers(case["k_lo"], case["k_hi"] + 1)), H))
    return out


def _inputs(case, seed):
    """Host arrays (and, for the largest beliefs, device tensors) of a case."""
    rng = np.random.default_rng([seed, 2606])
    kind, x = case["kind"], {}
    if kind == "batch":
        sizes = _sizes(case)  # sizes by the case, values by the seed
        insts = [dict(case, n_lo=N, n_hi=N, k_lo=K, k_hi=K, h_lo=H, h_hi=H) for N, K, H in sizes]
        return dict(instances=[_instance(c, rng) for c in insts])
    if kind == "teacher":
        d_x, d_c, n_act, d_a, hid = DENOISERS[case["net"]]
        x.update(layers=_mlp(rng, [d_c + (n_act or d_a) + d_x + 1] + hid + [d_x], gain=2.0, bias=0.1),
                 cond=rng.standard_normal((case["N"], d_c), dtype=np.float32),
                 x1=rng.standard_normal((case["N"], d_x), dtype=np.float32),
                 action=int(rng.integers(0, n_act)) if n_act else rng.uniform(-1, 1, d_a).astype(np.float32))
        return x
    if kind == "reweight":
        g = torch.Generator(device="cuda").manual_seed(seed)
        x["loglik"] = torch.randn(case["N"], generator=g, device="cuda")
        x["src"] = torch.randn(case["N"], case["rows"], generator=g, device="cuda")
        if case["weighted"]:
            p = torch.rand(case["N"], generator=g, device="cuda", dtype=torch.float64) + 0.05
            x["prior"] = p / case["N"]
        x["U"] = int(_u32(rng, 1)[0])
        return x
    d = x["d"] = _desc(case["net"], rng)
    if kind in ("plan", "simulate"):
        x.update(S=_belief(rng, case["N"], d.d_s), C=_actions(rng, d, (case["K"], case["H"])), goal=_goal(rng, d),
                 seed=_seed(rng))
        if case.get("weighted"):
            w = rng.uniform(0.2, 1.0, case["N"])
            x["w"] = w / w.sum()
    elif kind == "update":
        x.update(S=_belief(rng, case["N"], d.d_s), action=_actions(rng, d, (1,)),
                 obs=rng.standard_normal(d.d_o).astype(np.float32), seed=_seed(rng), U=int(_u32(rng, 1)[0]))
    elif kind == "widen":
        M, cap = case["M"], 8
        sizes = np.random.default_rng(1).integers(1, case["group"] + 1, M)
        children = rng.integers(0, cap + 1, M).astype(np.int32)
        T = int(sizes.sum())
        x.update(seg=np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32), actions=_actions(rng, d, (M,)),
                 succ=rng.standard_normal((T, d.d_s), dtype=np.float32), children=children,
                 visits=(children.astype(np.int64) ** 2 + rng.integers(-2, 3, M)).clip(0).astype(np.int32),
                 table=rng.standard_normal((M, cap, d.d_o), dtype=np.float32), U=_u32(rng, M), seed=_seed(rng))
    elif kind == "distill":
        B, H = case["B"], case["H"]
        s0 = rng.standard_normal((B, d.d_s), dtype=np.float32)
        walk = 0.3 * rng.standard_normal((B, H, d.d_s), dtype=np.float32)
        x.update(s0=s0, actions=_actions(rng, d, (B, H)), targets=s0[:, None] + np.cumsum(walk, 1, dtype=np.float32),
                 seed=_seed(rng))
    elif kind == "return":
        B, H = case["B"], case["H"]
        x.update(s0=rng.standard_normal((B, d.d_s), dtype=np.float32), actions=_actions(rng, d, (B // 64, H)),
                 goal=_goal(rng, d), seed=_seed(rng))
    elif kind == "contrast":
        B = case["B"]
        x.update(S=_belief(rng, B, d.d_s), A=_actions(rng, d, (B,)),
                 O=rng.standard_normal((B, d.d_o), dtype=np.float32))
    return x


class State:
    pass


def prepare(case, seed):
    x, s = _inputs(case, seed), State()
    s.case, s.x, kind = case, x, case["kind"]
    if kind == "batch":
        s.models = [V.Model(i["d"], compute=case["compute"]) for i in x["instances"]]
        s.actions = torch.cat([_dev(i["action"]) for i in x["instances"]])
        s.obs = torch.stack([_dev(i["obs"]) for i in x["instances"]])
        s.u = _dev(np.concatenate([i["U"] for i in x["instances"]]).view(np.int32))
        s.batch = V.Batch([dict(model=m, states=_dev(i["S"]), cands=_dev(i["C"]), gamma=0.95, goal=i["goal"],
                                seed=i["seed"], lam=1.0, update_seed=i["update_seed"])
                           for m, i in zip(s.models, x["instances"])])
        s.batch.capture(actions=s.actions, obs=s.obs, resample_u=s.u)
        return s
    if kind == "teacher":
        d_x, d_c, n_act, d_a, _ = DENOISERS[case["net"]]
        s.den = V.Denoiser(x["layers"], d_c, d_x, n_act, d_a, compute=case["compute"])
        s.cond, s.x1, s.out = _dev(x["cond"]), _dev(x["x1"]), torch.empty((case["N"], d_x), device="cuda")
        s.ws = torch.empty(max(1, int(V.lib.voila_ddim_workspace_size(s.den.handle, case["steps"]))),
                           dtype=torch.uint8, device="cuda")
        return s
    if kind == "reweight":
        s.ws = V.weights_workspace(case["N"], x["loglik"].device)
        s.idx = torch.empty(case["N"], dtype=torch.int32, device="cuda")
        s.dst = torch.empty_like(x["src"])
        s.stats = torch.empty(2, dtype=torch.float64, device="cuda")
        return s
    d = x["d"]
    s.model = V.Model(d, compute=case["compute"])
    if kind in ("plan", "simulate"):
        K, N, H = case["K"], case["N"], case["H"]
        s.S, s.C, s.w = _dev(x["S"]), _dev(x["C"]), _dev(x["w"]) if "w" in x else None
        s.q, s.ws = torch.empty(K, device="cuda"), s.model.plan_workspace(N, K, H)
        if kind == "simulate":
            s.traj = torch.empty((K, N, H, d.d_s), device="cuda")
            s.o = torch.empty((K, N, H, d.d_o), device="cuda")
            s.wso = torch.empty(max(1, int(V.lib.voila_plan_observe_workspace_size(s.model.handle, K, H))),
                                dtype=torch.uint8, device="cuda")
    elif kind == "update":
        N = case["N"]
        s.S, s.a, s.o, s.ws = _dev(x["S"]), _dev(x["action"]), _dev(x["obs"]), s.model.update_workspace(N)
        s.a = s.a.reshape(-1)
        s.out = {"states": torch.empty((N, d.d_s), device="cuda"), "prop": torch.empty((N, d.d_s), device="cuda"),
                 "idx": torch.empty(N, dtype=torch.int32, device="cuda"), "loglik": torch.empty(N, device="cuda"),
                 "w": torch.empty(N, dtype=torch.float64, device="cuda"),
                 "stats": torch.empty(2, dtype=torch.float64, device="cuda")}
    elif kind == "widen":
        for k in ("succ", "seg", "actions", "visits", "children", "table"):
            setattr(s, k, _dev(x[k]))
        s.u = _dev(x["U"].view(np.int32))
        s.out = None
        s.ws = torch.empty(max(1, int(V.lib.voila_pw_step_workspace_size(s.model.handle, int(s.succ.shape[0]),
                                                                         case["M"]))),
                           dtype=torch.uint8, device="cuda")
    elif kind in ("distill", "return"):
        s.s0, s.actions = _dev(x["s0"]), _dev(x["actions"])
        s.targets = _dev(x["targets"]) if kind == "distill" else None
    elif kind == "contrast":
        s.S, s.A, s.O = _dev(x["S"]), _dev(x["A"]), _dev(x["O"])
        s.ws = torch.empty(max(1, int(V.lib.voila_info_nce_grad_workspace_size(s.model.handle, case["B"]))),
                           dtype=torch.uint8, device="cuda")
        s.out = None
    return s


def run(s):
    case, x, kind = s.case, s.x, s.case["kind"]
    if kind == "plan":
        return {"q": V.plan(s.model, s.S, s.C, 0.99, x["goal"], belief_w=s.w, seed=x["seed"], q_out=s.q,
                            workspace=s.ws)}
    if kind == "simulate":
        q, traj = V.plan(s.model, s.S, s.C, 0.99, x["goal"], seed=x["seed"], q_out=s.q, workspace=s.ws,
                         return_traj=True, traj_out=s.traj)
        return {"q": q, "traj": traj,
                "obs": V.plan_observe(s.model, traj, s.C, seed=x["seed"], out=s.o, workspace=s.wso)}
    if kind == "update":
        return V.update(s.model, s.S, s.a, s.o, lam=1.0, seed=x["seed"], U=x["U"], out=s.out, workspace=s.ws)
    if kind == "batch":
        b = s.batch
        b.replay()
        return {"q": b.q, "w": b.w, "states": b.new_states, "stats": b.stats}
    if kind == "widen":
        # the step updates the nodes' branch tables in place: each pass takes
        # them as they stood before it
        children, table = s.children.clone(), s.table.clone()
        s.out = V.pw_step(s.model, s.succ, s.seg, s.actions, s.visits, children, table, s.u, 1.0, 0.5, lam=1.0,
                          seed=x["seed"], out=s.out, workspace=s.ws)
        return dict(s.out, children=children, table=table)
    if kind == "distill":
        loss, grad, _ = V.rollout_grad(s.model, s.s0, s.actions, case["H"], V.VOILA_OBJ_DISTILL, targets=s.targets,
                                       seed=x["seed"])
        return {"loss": loss, "grad": grad}
    if kind == "return":
        loss, _, grad = V.rollout_grad(s.model, s.s0, s.actions, case["H"], V.VOILA_OBJ_RETURN, gamma=0.99,
                                       goal=x["goal"], particles=64, seed=x["seed"], want_params=False,
                                       want_actions=True)
        return {"loss": loss, "grad": grad}
    if kind == "contrast":
        s.out = V.info_nce_grad(s.model, s.S, s.A, s.O, out=s.out, workspace=s.ws)
        return s.out
    if kind == "teacher":
        return V.ddim_sample(s.den, s.cond, x["action"], s.x1, case["steps"], out=s.out, workspace=s.ws)
    return V.reweight_resample(x["loglik"], x["U"], lam=1.0, prior_w=x.get("prior"), src=x["src"], workspace=s.ws,
                               idx=s.idx, dst=s.dst, stats=s.stats)


# ---------------------------------------------------------------------------
# the work a pass cannot do without
# ---------------------------------------------------------------------------
def _macs(dims):
    return sum(a * b for a, b in zip(dims[:-1], dims[1:]))


def _pbytes(dims, compute):
    return _macs(dims) * (4 if compute == "f32" else 2) + 4 * sum(dims[1:])


def work(case):
    kind, c = case["kind"], case["compute"]
    if kind == "reweight":  # log-likelihoods (and prior) in, rows in and out, indices out
        return {"bytes": case["N"] * (4.0 + 8 * case["rows"] + 4 + (8 if case["weighted"] else 0)), "flops": 0.0}
    if kind == "teacher":
        d_x, d_c, n_act, d_a, hid = DENOISERS[case["net"]]
        dims = [d_c + d_x] + hid + [d_x]  # action and time are the same for every sample
        return {"bytes": 4.0 * case["N"] * (d_c + 2 * d_x) + _pbytes(dims, c),
                "flops": 2.0 * _macs(dims) * case["N"] * case["steps"]}
    d_s, n_act, d_a, d_w, d_o, d_wz, hid, lik = NETS[case["net"]]
    trans, obs = [d_s + d_a + d_w] + hid + [d_s], [d_s + d_wz] + hid + [d_o]  # a one-hot action is a bias row
    lik1 = [d_s] + lik + [1]
    act = 4.0 * (d_a or 1)

    def plan(N, K, H):
        return 4.0 * N * d_s + K * H * act + 4 * K + _pbytes(trans, c), 2.0 * _macs(trans) * K * N * H

    def update(N):
        return N * (4.0 * 3 * d_s + 16) + _pbytes(trans, c) + _pbytes(lik1, c), 2.0 * N * (_macs(trans) + _macs(lik1))

    if kind == "plan":
        b, f = plan(case["N"], case["K"], case["H"])
        return {"bytes": b + (8 * case["N"] if case["weighted"] else 0), "flops": f}
    if kind == "simulate":
        b, f = plan(case["N"], case["K"], case["H"])
        rows = float(case["K"] * case["N"] * case["H"])
        return {"bytes": b + 4 * rows * (2 * d_s + d_o) + _pbytes(obs, c), "flops": f + 2 * _macs(obs) * rows}
    if kind == "update":
        b, f = update(case["N"])
        return {"bytes": b, "flops": f}
    if kind == "batch":
        parts = [plan(*s) for s in _sizes(case)] + [update(s[0]) for s in _sizes(case)]
        return {"bytes": float(sum(p[0] for p in parts)), "flops": float(sum(p[1] for p in parts))}
    if kind == "widen":
        T = case["M"] * (case["group"] + 1) / 2.0
        return {"bytes": T * (8.0 * d_s + 16) + _pbytes(lik1, c), "flops": 2.0 * T * _macs(lik1)}
    if kind in ("distill", "return"):  # forward, input adjoints and (distillation) weight adjoints of every step
        n = float(case["B"] * case["H"])
        per = 3 if kind == "distill" else 2
        return {"bytes": 4.0 * case["B"] * d_s + (n * (4 * d_s + 4) if kind == "distill" else n / 64 * 2 * act),
                "flops": per * 2.0 * _macs(trans) * n}
    # contrast: forward from the observations, hidden adjoints, weight derivatives
    fwd, hidden = _macs([d_o] + lik + [1]), _macs(lik)
    full = _macs([d_o] + lik) + lik[-1]
    return {"bytes": 4.0 * case["B"] * (d_s + d_o) + case["B"] * act + 2 * 4 * _macs([d_s + (n_act or d_a) + d_o] + lik),
            "flops": 2.0 * (fwd + hidden + full) * float(case["B"]) ** 2}


# ---------------------------------------------------------------------------
# the same in binary64
# ---------------------------------------------------------------------------
_MASK = 0xFFFFFFFF


def _philox(seed, c0, c1, c2, c3):
    """The four words of Philox4x32-10 (Salmon et al., SC'11) at broadcast int64 counters."""
    c = [t.expand(torch.broadcast_shapes(*[u.shape for u in (c0, c1, c2, c3)])) for t in (c0, c1, c2, c3)]
    k0, k1 = seed & _MASK, (seed >> 32) & _MASK
    for _ in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [((p1 >> 32) & _MASK) ^ c[1] ^ k0, p1 & _MASK, ((p0 >> 32) & _MASK) ^ c[3] ^ k1, p0 & _MASK]
        k0, k1 = (k0 + 0x9E3779B9) & _MASK, (k1 + 0xBB67AE85) & _MASK
    return c


def _uniform(w):
    return (2.0 * (w >> 9).double() + 1.0) * 2.0**-24


def _normals(seed, c0, c1, c2, stream, d):
    """[..., d] standard normals of the counters (Box-Muller on the word pairs)."""
    dev = torch.device("cuda")
    as_t = lambda v: torch.as_tensor(v, dtype=torch.int64, device=dev)[..., None]  # noqa: E731
    blocks = torch.arange((d + 3) // 4, device=dev) + (stream << 16)
    u = [_uniform(w) for w in _philox(seed, as_t(c0), as_t(c1), as_t(c2), blocks)]
    r0, r1 = (torch.sqrt(-2.0 * torch.log(v)) for v in (u[0], u[2]))
    t0, t1 = 2.0 * math.pi * u[1], 2.0 * math.pi * u[3]
    z = torch.stack([r0 * torch.cos(t0), r0 * torch.sin(t0), r1 * torch.cos(t1), r1 * torch.sin(t1)], -1)
    return z.flatten(-2)[..., :d]


def _f64(layers):
    return [(_dev(w).double(), _dev(b).double()) for w, b in layers]


def _net(layers, x):
    for j, (w, b) in enumerate(layers):
        x = torch.addmm(b, x, w.t())
        if j + 1 < len(layers):
            x = torch.relu(x)
    return x


def _act(d, a):
    """Network input of actions [n] (one-hot) or [n, d_a]."""
    return torch.nn.functional.one_hot(a.long(), d.n_actions).double() if d.n_actions else a.double()


def _rollouts(d, S, C, goal, seed, gamma=0.99, keep=False):
    """Returns [K, N] (and the states and observations of every step if keep)."""
    T, Z = _f64(d.trans), _f64(d.obs)
    S, C, goal = _dev(S).double(), _dev(C), _dev(goal).double()
    N, K, H = S.shape[0], C.shape[0], C.shape[1]
    G = torch.zeros((K, N), dtype=torch.float64, device="cuda")
    traj = torch.empty((K, N, H, d.d_s), dtype=torch.float32, device="cuda") if keep else None
    obs = torch.empty((K, N, H, d.d_o), dtype=torch.float32, device="cuda") if keep else None
    per = max(1, (1 << 18) // N)
    for k0 in range(0, K, per):
        k1 = min(K, k0 + per)
        s = S.repeat(k1 - k0, 1)
        i = torch.arange(N, device="cuda").repeat(k1 - k0)
        k = torch.arange(k0, k1, device="cuda").repeat_interleave(N)
        g = torch.zeros(len(i), dtype=torch.float64, device="cuda")
        for t in range(H):
            a = _act(d, C[k, t])
            s = s + _net(T, torch.cat([s, a, _normals(seed, i, k, t, STREAM_PLAN, d.d_w)], 1))
            g = g - gamma**t * ((s - goal) ** 2).sum(1)
            if keep:
                traj[k0:k1, :, t] = s.view(k1 - k0, N, -1).float()
                z = torch.cat([s, a, _normals(seed, i, k, t, STREAM_OBSERVE, d.d_wz)], 1)
                obs[k0:k1, :, t] = _net(Z, z).view(k1 - k0, N, -1).float()
        G[k0:k1] = g.view(k1 - k0, N)
    return G, traj, obs


def _normalised(x):
    """Weights, log evidence (uniform prior over x) and effective sample size."""
    e = torch.exp(x - x.max())
    w = e / e.sum()
    return w, torch.stack([x.max() + torch.log(e.sum()) - math.log(x.numel()), 1.0 / (w * w).sum()])


def _updated(d, S, action, obs, seed):
    S = _dev(S).double()
    N = S.shape[0]
    a = _act(d, _dev(action).reshape(1, -1) if not d.n_actions else _dev(action).reshape(1)).expand(N, -1)
    w = _normals(seed, torch.arange(N, device="cuda"), 0, 0, STREAM_UPDATE, d.d_w)
    prop = S + _net(_f64(d.trans), torch.cat([S, a, w], 1))
    ll = _net(_f64(d.lik), torch.cat([prop, a, _dev(obs).double().expand(N, -1)], 1))[:, 0]
    wn, st = _normalised(ll)
    return prop, ll, wn, st


def _widened(case, x):
    d, M = x["d"], case["M"]
    seg, succ = x["seg"].astype(np.int64), _dev(x["succ"]).double()
    lo, cap = torch.as_tensor(seg[:-1], device="cuda"), x["table"].shape[1]
    ch, vis = x["children"].astype(np.float64), x["visits"].astype(np.float64)
    widen = (ch < cap) & ((ch == 0) | (ch < np.sqrt(vis)))
    m = torch.arange(M, device="cuda")
    a = _act(d, _dev(x["actions"]))
    new = _net(_f64(d.obs), torch.cat([succ[lo], a, _normals(x["seed"], 0, m, 0, STREAM_OBSERVE, d.d_wz)], 1))
    z = torch.zeros_like(m)
    u = _uniform(_philox(x["seed"], m, z + 1, z, z + (STREAM_BRANCH << 16))[0])
    wid, ch = _dev(widen), _dev(x["children"]).long()
    branch = torch.where(wid, ch, torch.floor(u * ch).long())
    table = _dev(x["table"]).double()
    table[m[wid], branch[wid]] = new[wid]
    node = torch.repeat_interleave(m, torch.as_tensor(np.diff(seg), device="cuda"))
    net, ll = _f64(d.lik), torch.empty(len(succ), dtype=torch.float64, device="cuda")
    for r in range(0, len(succ), 1 << 18):
        n = node[r:r + (1 << 18)]
        ll[r:r + (1 << 18)] = _net(net, torch.cat([succ[r:r + (1 << 18)], a[n], table[n, branch[n]]], 1))[:, 0]
    top = torch.full((M,), -math.inf, dtype=torch.float64, device="cuda").scatter_reduce(0, node, ll, "amax")
    e = torch.exp(ll - top[node])
    tot = torch.zeros(M, dtype=torch.float64, device="cuda").index_add(0, node, e)
    w = e / tot[node]
    sq = torch.zeros(M, dtype=torch.float64, device="cuda").index_add(0, node, w * w)
    n = torch.as_tensor(np.diff(seg), device="cuda").double()
    return {"widen": None, "branch": None, "idx": None, "children": None, "succ": None, "loglik": ll, "w": w,
            "stats": torch.stack([top + torch.log(tot) - torch.log(n), 1.0 / sq], 1), "table": table}


def _flat(grads):
    return torch.cat([g.reshape(-1) for g in grads])


def _rollout_gradient(case, x):
    d, B, H = x["d"], case["B"], case["H"]
    distill = case["kind"] == "distill"
    net = [(w.requires_grad_(distill), b.requires_grad_(distill)) for w, b in _f64(d.trans)]
    s0, A = _dev(x["s0"]).double(), _dev(x["actions"])
    if not distill:
        A = A.double().requires_grad_()
    leaves = [p for layer in net for p in layer] if distill else [A]
    loss, total = 0.0, [torch.zeros_like(p) for p in leaves]
    for r in range(0, B, 16384):
        b = torch.arange(r, min(B, r + 16384), device="cuda")
        s, part = s0[b], 0.0
        for t in range(H):
            a = _act(d, A[b, t]) if distill else A[b // 64, t]
            s = s + _net(net, torch.cat([s, a, _normals(x["seed"], b, 0, t, STREAM_PLAN, d.d_w)], 1))
            if distill:
                part = part + ((s - _dev(x["targets"][r:r + 16384, t]).double()) ** 2).sum() / (B * H)
            else:
                part = part - 0.99**t * ((s - _dev(x["goal"]).double()) ** 2).sum() / B
        for acc, g in zip(total, torch.autograd.grad(part, leaves)):
            acc += g
        loss += part.detach()
    return {"loss": loss.reshape(1), "grad": _flat(total) if distill else total[0]}


def _contrast(case, x):
    d, B = x["d"], case["B"]
    net = [(w.requires_grad_(), b.requires_grad_()) for w, b in _f64(d.lik)]
    S, A, O = _dev(x["S"]).double(), _act(d, _dev(x["A"])), _dev(x["O"]).double()
    per = max(1, (1 << 17) // B)

    def scores(r):
        n = min(B, r + per) - r
        rows = torch.cat([S[r:r + n], A[r:r + n]], 1).repeat_interleave(B, 0)
        return _net(net, torch.cat([rows, O.repeat(n, 1)], 1)).view(n, B)

    with torch.no_grad():
        L = torch.cat([scores(r) for r in range(0, B, per)])
        G = (torch.softmax(L, 1) - torch.eye(B, dtype=torch.float64, device="cuda")) / B
        loss = (torch.logsumexp(L, 1) - L.diagonal()).mean()
    leaves = [p for layer in net for p in layer]
    total = [torch.zeros_like(p) for p in leaves]
    for r in range(0, B, per):
        out = scores(r)
        for acc, g in zip(total, torch.autograd.grad((out * G[r:r + out.shape[0]]).sum(), leaves)):
            acc += g
    return {"loss": loss.reshape(1), "grad": _flat(total)}


def _abar(tau):
    c, c0 = math.cos(math.pi / 2 * (tau + 0.008) / 1.008), math.cos(math.pi / 2 * 0.008 / 1.008)
    return min(1.0, max(0.0, (c / c0) ** 2))


def _teacher(case, x):
    d_x, d_c, n_act, d_a, _ = DENOISERS[case["net"]]
    net, n = _f64(x["layers"]), case["steps"]
    a = _dev(np.asarray(x["action"])).reshape(1, -1)
    a = torch.nn.functional.one_hot(a[0].long(), n_act).double() if n_act else a.double()
    c, v = _dev(x["cond"]).double(), _dev(x["x1"]).double()
    for k in range(n):
        tau = 1.0 - k / n
        p, q = _abar(tau), _abar(1.0 - (k + 1) / n)
        t = torch.full((len(c), 1), tau, dtype=torch.float64, device="cuda")
        y = _net(net, torch.cat([c, a.expand(len(c), -1), v, t], 1))
        x0, eps = math.sqrt(p) * v - math.sqrt(1 - p) * y, math.sqrt(1 - p) * v + math.sqrt(p) * y
        v = math.sqrt(q) * x0 + math.sqrt(1 - q) * eps
    return v


def exact(case, seed):
    x, kind = _inputs(case, seed), case["kind"]
    if kind in ("distill", "return"):
        return _rollout_gradient(case, x)
    if kind == "contrast":
        return _contrast(case, x)
    with torch.no_grad():
        if kind in ("plan", "simulate"):
            G, traj, obs = _rollouts(x["d"], x["S"], x["C"], x["goal"], x["seed"], keep=kind == "simulate")
            q = G @ _dev(x["w"]) if "w" in x else G.mean(1)
            return {"q": q} if kind == "plan" else {"q": q, "traj": traj, "obs": obs}
        if kind == "update":
            prop, ll, w, st = _updated(x["d"], x["S"], x["action"], x["obs"], x["seed"])
            return {"states": None, "idx": None, "w": w, "loglik": ll, "prop": prop, "stats": st}
        if kind == "batch":
            out = {"q": [], "w": [], "states": None, "stats": []}
            for i in x["instances"]:
                G = _rollouts(i["d"], i["S"], i["C"], i["goal"], i["seed"], gamma=0.95)[0]
                _, _, w, st = _updated(i["d"], i["S"], i["action"], i["obs"], i["update_seed"])
                out["q"].append(G.mean(1))
                out["w"].append(w)
                out["stats"].append(st)
            return out
        if kind == "widen":
            return _widened(case, x)
        if kind == "teacher":
            return _teacher(case, x)
        v = x["loglik"].double()
        if "prior" in x:
            v = v + torch.log(x["prior"])
        st = _normalised(v)[1]
        if "prior" in x:
            st[0] += math.log(v.numel())
        return {"idx": None, "w": None, "stats": st, "dst": None}
