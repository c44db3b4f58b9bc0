"""The work a user of this library has it do, as cases that can be timed.

Each case is one call, or one short sequence of calls, of the public binding
(paper_2308_02329_amd.api) on inputs drawn on the GPU from a seed:

    listed()             the cases
    draw(rng)            one more case from the same ranges
    prepare(case, seed)  inputs, plans and weights a program holds before the call
    run(state)           one pass; its outputs
    work(case)           bytes and operations one pass cannot do without
    exact(case, seed)    the same outputs in 64 bits from plain torch

The sizes are those of the library's own workloads (bench.py, learned.py,
stats.py, xy.py and the tests) and the ranges around them; step counts are
cut so that a pass stays short.  exact() gives None for spins, integer
energies and indices.
"""
import math
import random

import numpy as np
import torch

from paper_2308_02329_amd import api, synth

DT, BTIL, ETA = 0.01, 1.0, 2e-4  # the library's default run inputs
MAP = dict(b=0.01, loss=0.01, kl=0.1)  # the map's parameters (the statistics' choice)
BB2 = 25.0
LR = 2e-3


# ------------------------------------------------------------------- cases
def listed():
    return [
        # the first call of a new user: a small problem, few runs; latency and launches count
        {"name": "solve_n16", "kind": "solve", "n": 16, "d": 2, "r": 32, "steps": 400, "prec": "f32", "j": "i8",
         "graph": "sk", "want": "all"},
        # one instance of the default workload: 100 initial states x 20 pumps, every output
        {"name": "solve_sk100", "kind": "solve", "n": 100, "d": 3, "r": 2000, "steps": 1000, "prec": "f32",
         "j": "i8", "graph": "sk", "want": "all"},
        # real-valued couplings and a ragged shape: both split in three bf16 terms
        {"name": "solve_gauss75", "kind": "solve", "n": 75, "d": 4, "r": 333, "steps": 1000, "prec": "f32",
         "j": "f32", "graph": "gauss", "want": "all"},
        # the learned restart's ground-state search: many runs of an N = 200 instance in bf16
        {"name": "search_sk200", "kind": "solve", "n": 200, "d": 3, "r": 20000, "steps": 500, "prec": "bf16",
         "j": "i8", "graph": "sk", "want": "energies"},
        # the precision workload: N = 1000 at D = 4, bf16 couplings, workspace kept
        {"name": "integrate_n1000", "kind": "integrate", "n": 1000, "d": 4, "r": 4096, "steps": 250, "prec": "bf16",
         "j": "bf16", "graph": "gauss"},
        # the default workload, 24 of its 1000 instances: tuned plans, one graph launch, every run scored
        {"name": "batch_sk100", "kind": "batch", "n": 100, "insts": 24, "r": 2000, "steps": 400, "prec": "f32"},
        # solves of mixed size, D and graph family, 32 runs each, in one launch with the default plans
        {"name": "batch_mixed", "kind": "mixed", "solves": 150, "r": 32, "steps": 400, "prec": "bf16", "mix": 0},
        # the round-trip map over a dense pump scan of one instance
        {"name": "map_n100", "kind": "map", "n": 100, "d": 3, "r": 65536, "steps": 200, "prec": "f32", "graph": "sk"},
        # the statistical harness: graphs of the paper's family as the CIM, readout and energies of every run
        {"name": "map_batch_stats", "kind": "map_batch", "n": 100, "d": 1, "graphs": 10, "r": 5100, "steps": 500,
         "prec": "f32"},
        # sparse rows: a 3-regular graph through the gather integrator
        {"name": "sparse_reg3_800", "kind": "integrate", "n": 800, "d": 3, "r": 4096, "steps": 500, "prec": "f32",
         "j": "ell", "graph": "reg3"},
        # the restart decision on 20 pump batches of 1000 runs: features, scores, the kept runs gathered
        {"name": "restart_decision", "kind": "restart", "n": 200, "d": 3, "groups": 20, "group": 1000, "keep": 50,
         "ckpts": 8},
        # one training step of the restart network at its default batch
        {"name": "train_step", "kind": "train", "batch": 8192},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_COST = 8.0e12  # matrix operations of a pass above which a drawn case takes fewer steps


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "integrate", "integrate", "sparse", "batch", "mixed", "map",
                       "map_batch", "restart", "train"])
    if kind == "solve":
        c = {"kind": "solve", "n": _log(rng, 8, 260), "d": rng.randint(1, 4), "r": _log(rng, 16, 20000),
             "steps": 400, "prec": rng.choice(["f32", "bf16"]), "j": rng.choice(["i8", "i8", "f32", "bf16"]),
             "want": rng.choice(["all", "energies"])}
        c["graph"] = "gauss" if c["j"] != "i8" else rng.choice(["sk", "er"])
    elif kind == "integrate":
        c = {"kind": "integrate", "n": _log(rng, 200, 1024), "d": rng.randint(1, 4), "r": _log(rng, 16, 4096),
             "steps": 200, "prec": rng.choice(["f32", "bf16", "bf16"]), "j": rng.choice(["i8", "f32", "bf16", "fp8"])}
        c["graph"] = "sk" if c["j"] == "i8" else "gauss"
    elif kind == "sparse":
        g = rng.choice(["reg3", "reg3", "er"])
        n = 2 * _log(rng, 25, 400) if g == "reg3" else _log(rng, 20, 200)
        c = {"kind": "integrate", "n": n, "d": rng.randint(1, 4), "r": _log(rng, 32, 4096), "steps": 300,
             "prec": "f32", "j": "ell", "graph": g}
    elif kind == "batch":
        c = {"kind": "batch", "n": _log(rng, 20, 128), "insts": _log(rng, 2, 24), "r": _log(rng, 100, 2000),
             "steps": 300, "prec": rng.choice(["f32", "bf16"])}
    elif kind == "mixed":
        c = {"kind": "mixed", "solves": _log(rng, 10, 150), "r": _log(rng, 8, 64), "steps": 300,
             "prec": rng.choice(["f32", "bf16"]), "mix": rng.randint(1, 1 << 20)}
    elif kind == "map":
        c = {"kind": "map", "n": _log(rng, 10, 112), "d": rng.randint(1, 4), "r": _log(rng, 64, 65536), "steps": 200,
             "prec": rng.choice(["f32", "f32", "bf16"]), "graph": rng.choice(["sk", "er"])}
    elif kind == "map_batch":
        d = rng.choice([1, 2])
        c = {"kind": "map_batch", "n": _log(rng, 10, 100), "d": d, "graphs": _log(rng, 2, 20),
             "r": (51 if d == 1 else 21) * _log(rng, 10, 100), "steps": 300, "prec": "f32"}
    elif kind == "restart":
        group = _log(rng, 100, 4000)
        c = {"kind": "restart", "n": _log(rng, 50, 400), "d": rng.randint(2, 4), "groups": rng.randint(1, 20),
             "group": group, "keep": max(1, group * rng.choice([1, 5, 20, 50]) // 100), "ckpts": rng.randint(1, 8)}
        while c["groups"] * group > 20000:
            c["groups"] = max(1, c["groups"] // 2)
            if c["groups"] == 1:
                break
    else:
        c = {"kind": "train", "batch": _log(rng, 64, 16384)}
    if "steps" in c:
        # float32 products are made of three bf16 ones (six with float couplings)
        f = work(c)["flops"] * (1 if c["prec"] == "bf16" else 6 if c.get("j") == "f32" else 3)
        if f > _COST:
            c["steps"] = max(20, int(c["steps"] * _COST / f))
    return c


# ------------------------------------------------------------------ inputs
def _gen(seed, *key):
    g = torch.Generator(device="cuda")
    g.manual_seed(hash((int(seed),) + tuple(int(k) for k in key)) & 0x7FFFFFFFFFFF)
    return g


def _f32(v):
    return float(np.float32(v))


def _density(graph, n):
    return {"sk": 1.0, "gauss": 1.0, "er": 0.2, "reg3": 3.0 / n}[graph]


def _eps(graph, n):
    """Half the inverse of the coupling matrix's largest eigenvalue, from the
    semicircle (3-regular: Kesten-McKay) edge."""
    edge = 2.0 * math.sqrt(2.0) if graph == "reg3" else 2.0 * math.sqrt(n * _density(graph, n))
    return _f32(0.5 / max(edge, 1.0))


def _couplings(graph, n, seed, key=0):
    """Symmetric zero-diagonal couplings, float32 on the GPU."""
    if graph == "reg3":
        return torch.from_numpy(synth.regular3_pm1(n, int(seed) & 0xFFFFFF, key).astype(np.float32)).cuda()
    g = _gen(seed, 11, key)
    if graph == "gauss":
        a = torch.randn((n, n), generator=g, device="cuda")
    else:
        a = (torch.randint(0, 2, (n, n), generator=g, device="cuda") * 2 - 1).float()
        if graph == "er":
            a = a * (torch.rand((n, n), generator=g, device="cuda") < 0.2)
    a = torch.triu(a, 1)
    return (a + a.T).contiguous()


def _stored(Jf, j):
    if j == "i8":
        return Jf.to(torch.int8)
    if j == "bf16":
        return Jf.to(torch.bfloat16)
    if j == "fp8":
        return api.chym_quantize_fp8(Jf)
    if j == "ell":
        return torch.from_numpy(api.ell_pack(Jf.cpu().numpy())).cuda()
    return Jf


def _pumps(r):
    """Pump-major grid over [0.5, 2], as many pumps as divide the runs evenly up to 20."""
    k = max(v for v in range(1, 21) if r % v == 0)
    return torch.from_numpy(synth.pump_grid(r // k, np.linspace(0.5, 2.0, k) if k > 1 else [1.2])).cuda()


def _x0(seed, n, r, d, sigma=1e-3, key=0):
    return torch.randn((n, r, d), generator=_gen(seed, 12, key), device="cuda") * sigma


def _alpha(steps, d):
    return torch.from_numpy(synth.anneal_schedule(steps, d)[0]).cuda()


def _ode_inputs(c, seed):
    n, r, d = c["n"], c["r"], c["d"]
    return dict(Jf=_couplings(c["graph"], n, seed), pump=_pumps(r), x0=_x0(seed, n, r, d), alpha=_alpha(c["steps"], d),
                eps=_eps(c["graph"], n))


def _mixed_tasks(c):
    """(n, d, sparse) of every solve: five sizes (50 .. 800 for mix 0, else
    drawn from 20 .. 800), D in 2 .. 4, half of them 3-regular."""
    rng = random.Random(c["mix"])
    sizes = [50, 100, 200, 400, 800] if c["mix"] == 0 else [2 * _log(rng, 10, 400) for _ in range(5)]
    return [(rng.choice(sizes), rng.choice([2, 3, 4]), rng.random() < 0.5) for _ in range(c["solves"])]


def _mixed_inputs(c, seed):
    tasks = _mixed_tasks(c)
    r, out, graphs = c["r"], [], {}
    g = _gen(seed, 13)
    pump = torch.rand(len(tasks), generator=g, device="cuda") * 1.5 + 0.5
    x0 = torch.randn(sum(n * r * d for n, d, _ in tasks), generator=g, device="cuda") * 1e-3
    off = 0
    for i, (n, d, sparse) in enumerate(tasks):
        # 3-regular graphs are drawn on the host: two per size, shared by its solves
        key = (n, i % 2) if sparse else (n, 100 + i)
        if key not in graphs:
            graphs[key] = _couplings("reg3" if sparse else "sk", n, seed, key[1])
        out.append(dict(n=n, d=d, sparse=sparse, Jf=graphs[key], key=key, off=off, x0=x0[off:off + n * r * d],
                        pump=pump[i].expand(r).contiguous(), eps=_eps("reg3" if sparse else "sk", n)))
        off += n * r * d
    return out, x0


def _map_inputs(c, seed, key=0):
    n, r, d = c["n"], c["r"], c["d"]
    graph = c.get("graph", "er")
    jmag = _f32(_eps(graph, n) * (MAP["b"] + MAP["loss"]) / MAP["b"])
    hth = -math.log((1 - MAP["b"]) * (1 - MAP["loss"])) / MAP["kl"]
    dh = torch.linspace(0.1, 1.0, r) if c["kind"] == "map" else torch.linspace(-0.5, 1.0, 51 if d == 1 else 21) \
        .repeat_interleave(r // (51 if d == 1 else 21))
    return dict(Jf=_couplings(graph, n, seed, key), h=(hth * (1.0 + dh)).float().cuda(),
                A0=_x0(seed, n, r, d, 0.1 * math.sqrt((MAP["b"] + MAP["loss"]) / BB2), key),
                alpha=_alpha(c["steps"], d) if d > 1 else torch.ones((c["steps"], 1), device="cuda"),
                jmag=jmag, beta_b2=BB2 if d > 1 or c["kind"] == "map" else 0.0)


def _net(seed):
    g = _gen(seed, 14)
    rn = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    return torch.cat([rn(128 * 32) * math.sqrt(2.0 / 32), rn(128) * 0.05, rn(128 * 128) * math.sqrt(2.0 / 128),
                      rn(128) * 0.05, rn(128) * math.sqrt(1.0 / 128), rn(1) * 0.05])


def _restart_inputs(c, seed):
    n, d, r = c["n"], c["d"], c["groups"] * c["group"]
    # amplitudes as the machine leaves them: clustered hyperspins with a run-dependent part
    base = _x0(seed, n, 1, d, 0.7, 1)
    xs = [(base * s + _x0(seed, n, r, d, 0.5, 2 + k)).contiguous() for k, s in enumerate((0.5, 0.9))]
    return dict(Jf=_couplings("sk", n, seed), xs=xs, pump=_pumps(r), w=_net(seed))


def _train_inputs(c, seed):
    g = _gen(seed, 15)
    b = c["batch"]
    rn = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    return dict(xs=rn(b, 32), y=(torch.rand(b, generator=g, device="cuda") < 0.1).float(), w=_net(seed),
                m=rn(20865) * 1e-4, v=(rn(20865) * 1e-4) ** 2 + 1e-8)


# ----------------------------------------------------------------- prepare
def _tune(n, d, prec):
    """Times the launch plans of a variant once per process, as bench.py does."""
    if api.chym_plan_get(n, d, prec, torch.int8)["ms"] == 0.0:
        api.chym_plan_autotune(n, d, prec, torch.int8, steps=100)


def prepare(case, seed):
    c, kind = case, case["kind"]
    if kind in ("solve", "integrate"):
        s = _ode_inputs(c, seed)
        s["J"] = _stored(s.pop("Jf"), c["j"])
        s["x"] = torch.empty_like(s["x0"])
        if kind == "integrate":
            nb = api.chym_integrate_workspace_size(s["J"], s["x"], precision=c["prec"])
            s["ws"] = torch.empty(nb + 256, dtype=torch.uint8, device="cuda") if nb else None
        return dict(s, case=c)
    if kind == "batch":
        n, r, dims = c["n"], c["r"], (2, 3)
        for d in dims:
            _tune(n, d, c["prec"])
        x0 = torch.randn(c["insts"] * n * r * sum(dims), generator=_gen(seed, 12), device="cuda") * 1e-3
        s = dict(x0=x0, x=torch.empty_like(x0), pump=_pumps(r), alphas={d: _alpha(c["steps"], d) for d in dims})
        m = c["insts"] * len(dims)
        w = api.spin_words(n)
        s["out"] = dict(spins=torch.empty((m, r, w), dtype=torch.int64, device="cuda"),
                        e_ising=torch.empty((m, r), dtype=torch.int32, device="cuda"),
                        e_hs=torch.empty((m, r), dtype=torch.float64, device="cuda"),
                        diverged=torch.empty((m, r), dtype=torch.uint8, device="cuda"))
        tasks, off = [], 0
        for i in range(c["insts"]):
            J = _couplings("sk", n, seed, i).to(torch.int8)
            for d in dims:
                tasks.append(dict(J=J, pump=s["pump"], x=s["x"][off:off + n * r * d].view(n, r, d),
                                  alpha=s["alphas"][d], eps=_eps("sk", n), btil=BTIL, eta=ETA, dt=DT,
                                  steps=c["steps"], precision=c["prec"],
                                  **{k: v[len(tasks)] for k, v in s["out"].items()}))
                off += n * r * d
        s["plan"] = api.chym_batch_create(tasks)
        return dict(s, case=c)
    if kind == "mixed":
        ins, x0 = _mixed_inputs(c, seed)
        r, x = c["r"], torch.empty_like(x0)
        spins = torch.empty(sum(r * api.spin_words(t["n"]) for t in ins), dtype=torch.int64, device="cuda")
        e_i = torch.zeros((len(ins), r), dtype=torch.int32, device="cuda")
        e_f = torch.zeros((len(ins), r), dtype=torch.float64, device="cuda")
        alphas = {d: _alpha(c["steps"], d) for d in (2, 3, 4)}
        packed, tasks, so = {}, [], 0
        for i, t in enumerate(ins):
            n, d, w = t["n"], t["d"], api.spin_words(t["n"])
            if t["key"] not in packed:
                packed[t["key"]] = _stored(t["Jf"], "ell" if t["sparse"] else "i8")
            k = dict(J=packed[t["key"]], pump=t["pump"], x=x[t["off"]:t["off"] + n * r * d].view(n, r, d),
                     alpha=alphas[d], eps=t["eps"], btil=BTIL, eta=ETA, dt=DT, steps=c["steps"], precision=c["prec"],
                     spins=spins[so:so + r * w].view(r, w))
            k["e_ising_f64" if t["sparse"] else "e_ising"] = (e_f if t["sparse"] else e_i)[i]
            tasks.append(k)
            so += r * w
        return dict(x0=x0, x=x, out=dict(spins=spins, e_ising=e_i, e_ising_f64=e_f), case=c,
                    plan=api.chym_batch_create(tasks))
    if kind == "map":
        s = _map_inputs(c, seed)
        s["J"] = s.pop("Jf").to(torch.int8)
        return dict(s, A=torch.empty_like(s["A0"]), case=c)
    if kind == "map_batch":
        tasks = []
        for g in range(c["graphs"]):
            t = _map_inputs(c, seed, g)
            t["J"] = t.pop("Jf").to(torch.int8)
            t.update(MAP, A=torch.empty_like(t["A0"]), steps=c["steps"], precision=c["prec"])
            tasks.append(t)
        m, r = c["graphs"], c["r"]
        return dict(tasks=tasks, case=c, spins=torch.empty((m, r, api.spin_words(c["n"])), dtype=torch.int64, device="cuda"),
                    e=torch.empty((m, r), dtype=torch.int32, device="cuda"))
    if kind == "restart":
        s = _restart_inputs(c, seed)
        s["J"] = s.pop("Jf").to(torch.int8)
        s["wb"] = api.chym_to_bf16(s["w"])
        return dict(s, feats=torch.zeros((s["pump"].shape[0], 32), device="cuda"), case=c)
    s = _train_inputs(c, seed)
    b = c["batch"]
    s["keep"] = {k: s[k].clone() for k in ("w", "m", "v")}
    s["wb0"] = api.chym_to_bf16(s["w"])
    s["wb"] = s["wb0"].clone()
    f = lambda *n: torch.empty(n, device="cuda")  # noqa: E731
    return dict(s, logit=f(b), h1=f(b, 128), h2=f(b, 128), loss=f(b), grad=f(20865),
                scratch=f(api.chym_mlp_scratch_floats(b)), case=c)


# --------------------------------------------------------------------- run
_ALL = ("spins", "e_ising", "e_hs", "e_hs_ss", "extra_frac", "diverged")


def run(state):
    s, c = state, state["case"]
    kind = c["kind"]
    if kind == "solve":
        s["x"].copy_(s["x0"])
        res = api.chym_solve(s["J"], s["pump"], s["x"], s["alpha"], eps=s["eps"], btil=BTIL, eta=ETA, dt=DT,
                             steps=c["steps"], precision=c["prec"],
                             **(dict(ss_step=int(0.4 * c["steps"]), want=_ALL) if c["want"] == "all"
                                else dict(want=("spins", "e_ising"))))
        return dict(res, x=s["x"])
    if kind == "integrate":
        s["x"].copy_(s["x0"])
        return api.chym_integrate(s["J"], s["pump"], s["x"], s["alpha"], eps=s["eps"], btil=BTIL, eta=ETA, dt=DT,
                                  steps=c["steps"], precision=c["prec"], workspace=s["ws"])
    if kind in ("batch", "mixed"):
        s["x"].copy_(s["x0"])
        s["plan"].launch()
        return dict(s["out"], x=s["x"])
    if kind == "map":
        s["A"].copy_(s["A0"])
        return api.chym_map_integrate(s["J"], s["h"], s["A"], s["alpha"], beta_b2=s["beta_b2"], jmag=s["jmag"],
                                      steps=c["steps"], precision=c["prec"], **MAP)
    if kind == "map_batch":
        for t in s["tasks"]:
            t["A"].copy_(t["A0"])
        s["batch_ws"] = api.chym_map_batch(s["tasks"])
        for i, t in enumerate(s["tasks"]):
            api.chym_readout(t["A"], s["spins"][i])
            api.chym_ising_energy(t["J"], s["spins"][i], s["e"][i])
        return dict(spins=s["spins"], e=s["e"], A=[t["A"] for t in s["tasks"]])
    if kind == "restart":
        words = api.chym_sign_words(s["xs"][1])
        for k in range(c["ckpts"]):
            api.chym_features(s["J"], s["xs"][k % 2], words, s["feats"], k)
        f = api.chym_feature_standardize(s["feats"], c["group"])
        logit = api.chym_mlp_forward(f, s["wb"])
        idx = api.chym_select_top(logit, c["group"], c["keep"])
        xk, pk = api.chym_gather_replicas(s["xs"][1], idx, pump=s["pump"])
        return dict(words=words, feats=s["feats"], std=f, logit=logit, idx=idx, x=xk, pump=pk)
    for k, v in s["keep"].items():
        s[k].copy_(v)
    s["wb"].copy_(s["wb0"])
    api.chym_mlp_forward(s["xs"], s["wb"], s["logit"], s["h1"], s["h2"])
    api.chym_mlp_backward(s["xs"], s["y"], s["wb"], s["logit"], s["h1"], s["h2"], s["scratch"], s["grad"], s["loss"])
    api.chym_mlp_adam(s["w"], s["wb"], s["m"], s["v"], s["grad"], lr=LR, t=50)
    return dict(logit=s["logit"], loss=s["loss"], grad=s["grad"], w=s["w"], m=s["m"], v=s["v"],
                wb=s["wb"].view(torch.bfloat16))


# -------------------------------------------------------------------- work
def _j_bytes(j, n, w=3):
    return {"i8": n * n, "f32": 4 * n * n, "bf16": 2 * n * n, "fp8": n * (n + 1), "ell": 8 * w * (n + 1)}[j]


def _ode_work(n, d, r, steps, j, graph):
    """One coupling row times the state per update, the state in and out once."""
    per = n - 1 if j != "ell" else _density(graph, n) * n
    return 2.0 * per * n * r * d * steps, 8.0 * n * r * d + _j_bytes(j, n, max(1, int(per))) + 4.0 * r + 4.0 * steps * d


def work(case):
    c, kind = case, case["kind"]
    if kind in ("solve", "integrate"):
        n, d, r = c["n"], c["d"], c["r"]
        f, b = _ode_work(n, d, r, c["steps"], c["j"], c["graph"])
        if kind == "solve":
            f += 2.0 * n * n * r * (1 if c["want"] != "all" else 1 + 2 * d)
            b += r * (8.0 * ((n + 63) // 64) + 4 + (25 if c["want"] == "all" else 0))
        return dict(flops=f, bytes=b)
    if kind in ("batch", "mixed"):
        f = b = 0.0
        each = [(c["n"], d, False) for d in (2, 3)] * c["insts"] if kind == "batch" else _mixed_tasks(c)
        for n, d, sparse in each:
            df, db = _ode_work(n, d, c["r"], c["steps"], "ell" if sparse else "i8", "reg3" if sparse else "sk")
            e = (6.0 * n if sparse else 2.0 * n * n) * c["r"]
            f += df + e * (1 + d if kind == "batch" else 1)
            b += db + c["r"] * (8.0 * ((n + 63) // 64) + 4 + (9 if kind == "batch" else 0))
        return dict(flops=f, bytes=b)
    if kind in ("map", "map_batch"):
        n, d, r = c["n"], c["d"], c["r"]
        f, b = _ode_work(n, d, r, c["steps"], "i8", "sk")
        m = 1
        if kind == "map_batch":
            m = c["graphs"]
            f += 2.0 * n * n * r
            b += r * (8.0 * ((n + 63) // 64) + 4)
        return dict(flops=m * f, bytes=m * b)
    if kind == "restart":
        n, d, r, g = c["n"], c["d"], c["groups"] * c["group"], c["groups"] * c["keep"]
        f = c["ckpts"] * 4.0 * n * n * r + 2.0 * 20865 * r
        b = 4.0 * n * r * d * (1 + c["ckpts"]) + 8.0 * r * ((n + 63) // 64) + 2 * 128.0 * r + 4.0 * r \
            + g * (8.0 * n * d + 12) + n * n
        return dict(flops=f, bytes=b)
    b = c["batch"]
    return dict(flops=6.0 * 20865 * b, bytes=4.0 * b * (32 + 3) + 20865 * (4.0 * 7 + 4))


# ------------------------------------------------------------------- exact
def _decoded(Jf, j):
    """The couplings as stored, in 64 bits."""
    if j == "bf16":
        return Jf.to(torch.bfloat16).double()
    if j == "fp8":
        amax = Jf.double().abs().amax(dim=1, keepdim=True)
        sc = torch.where(amax > 0, torch.exp2(torch.ceil(torch.log2(amax / 448.0))), torch.ones_like(amax))
        return (Jf.double() / sc).float().to(torch.float8_e4m3fn).double() * sc
    return Jf.double()


def _ode64(J, x0, pump, alpha, eps, steps, bf16, ss=None):
    """Euler steps in 64 bits on [m, n, r, d] (J [m, n, n]); bf16: the
    contraction's inputs rounded to bf16, as the caller of that form asks.
    Also returns the state after step ss."""
    m, n, r, d = x0.shape
    x, mid = x0.double(), None
    dt, btil, eta = _f32(DT), _f32(BTIL), _f32(ETA)
    if bf16:
        J = J.to(torch.bfloat16).double()
    gain = (pump.double() - 1.0).view(m, 1, r, 1)
    al = alpha.double()
    for k in range(steps):
        xin = x.float().to(torch.bfloat16).double() if bf16 else x
        G = torch.bmm(J, xin.reshape(m, n, r * d)).view(m, n, r, d)
        S = (x * x).sum(dim=3, keepdim=True)
        x = x + dt * (gain * x + eps * al[k] * G - btil * x * S - eta * x * x * x)
        if ss is not None and k + 1 == ss:
            mid = x
    return x, mid


def _hs64(J, x):
    """Hyperspin energies of [m, n, r, d]."""
    m, n, r, d = x.shape
    nrm = x.norm(dim=3, keepdim=True)
    u = torch.where(nrm > 0, x / nrm, torch.zeros_like(x))
    return -(u * torch.bmm(J, u.reshape(m, n, r * d)).view(m, n, r, d)).sum(dim=(1, 3))


def _map64(J, A, h, alpha, jmag, beta_b2, steps, bf16):
    m, n, r, d = A.shape
    b, loss, kl = (_f32(MAP[k]) for k in ("b", "loss", "kl"))
    A, h, al = A.double(), h.double().view(m, 1, r, 1), alpha.double()
    for k in range(steps):
        P = torch.sqrt(h * h + A * A)
        B = A * P / (P * torch.cosh(kl * P) - h * torch.sinh(kl * P))
        Bin = B.float().to(torch.bfloat16).double() if bf16 else B
        G = torch.bmm(J, Bin.reshape(m, n, r * d)).view(m, n, r, d)
        S = (B * B).sum(dim=3, keepdim=True)
        A = (1 - loss) * ((1 - b) * B + b * jmag * al[k] * G - beta_b2 * B * S)
    return A


def _bf(v):
    return v.float().to(torch.bfloat16).double()


class _Round(torch.autograd.Function):
    """Rounding to bf16 whose derivative is the identity."""

    @staticmethod
    def forward(ctx, v):
        return _bf(v)

    @staticmethod
    def backward(ctx, g):
        return g


def _mlp64(xs, p):
    """Hidden layers on bf16-rounded inputs, in 64 bits; p: the flat weights."""
    w1, b1, w2, b2, w3, b3 = torch.split(p, [4096, 128, 16384, 128, 128, 1])
    h1 = _Round.apply(torch.relu(_Round.apply(xs) @ w1.view(128, 32).T + b1))
    return torch.relu(h1 @ w2.view(128, 128).T + b2) @ w3 + b3


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind in ("solve", "integrate"):
        s = _ode_inputs(c, seed)
        J = _decoded(s["Jf"], c["j"])[None]
        bf16 = c["prec"] == "bf16" and c["j"] != "ell"
        ss = int(0.4 * c["steps"])
        x, mid = _ode64(J, s["x0"][None], s["pump"], s["alpha"], s["eps"], c["steps"], bf16, ss)
        if kind == "integrate":
            return x[0]
        out = dict(spins=None, x=x[0])
        out["e_ising" if c["j"] == "i8" else "e_ising_f64"] = None
        if c["want"] == "all":
            x2 = x[0] * x[0]
            ext = (x2.sum(2) - x2[:, :, 0]) / x2.sum(2)
            out.update(e_hs=_hs64(J, x)[0], e_hs_ss=_hs64(J, mid)[0] if ss else None,
                       extra_frac=ext.amax(0) if c["d"] > 1 else torch.zeros_like(ext.amax(0)), diverged=None)
        return out
    if kind == "batch":
        n, r, dims = c["n"], c["r"], (2, 3)
        x0 = torch.randn(c["insts"] * n * r * sum(dims), generator=_gen(seed, 12), device="cuda") * 1e-3
        J = torch.stack([_couplings("sk", n, seed, i) for i in range(c["insts"])]).double()
        each, x = n * r * sum(dims), torch.empty_like(x0, dtype=torch.float64)
        e = torch.empty((c["insts"], len(dims), r), dtype=torch.float64, device="cuda")
        for i, d in enumerate(dims):
            part = (slice(None), slice(sum(dims[:i]) * n * r, sum(dims[:i + 1]) * n * r))
            v, _ = _ode64(J, x0.view(c["insts"], each)[part].reshape(-1, n, r, d), _pumps(r).repeat(c["insts"], 1),
                          _alpha(c["steps"], d), _eps("sk", n), c["steps"], c["prec"] == "bf16")
            x.view(c["insts"], each)[part] = v.reshape(c["insts"], -1)
            e[:, i] = _hs64(J, v)
        return dict(spins=None, e_ising=None, e_hs=e.view(-1, r), diverged=None, x=x)
    if kind == "mixed":
        ins, x0 = _mixed_inputs(c, seed)
        r, x = c["r"], torch.empty_like(x0, dtype=torch.float64)
        for key in sorted({(t["n"], t["d"], t["sparse"]) for t in ins}):
            n, d, sparse = key
            mine = [t for t in ins if (t["n"], t["d"], t["sparse"]) == key]
            v, _ = _ode64(torch.stack([t["Jf"] for t in mine]).double(),
                          torch.stack([t["x0"].view(n, r, d) for t in mine]), torch.stack([t["pump"] for t in mine]),
                          _alpha(c["steps"], d), mine[0]["eps"], c["steps"], c["prec"] == "bf16" and not sparse)
            for t, u in zip(mine, v):
                x[t["off"]:t["off"] + n * r * d] = u.reshape(-1)
        return dict(spins=None, e_ising=None, e_ising_f64=None, x=x)
    if kind == "map":
        s = _map_inputs(c, seed)
        return _map64(s["Jf"].double()[None], s["A0"][None], s["h"], s["alpha"], s["jmag"], s["beta_b2"], c["steps"],
                      c["prec"] == "bf16")[0]
    if kind == "map_batch":
        ts = [_map_inputs(c, seed, g) for g in range(c["graphs"])]
        A = _map64(torch.stack([t["Jf"] for t in ts]).double(), torch.stack([t["A0"] for t in ts]),
                   torch.stack([t["h"] for t in ts]), ts[0]["alpha"], ts[0]["jmag"], ts[0]["beta_b2"], c["steps"], False)
        return dict(spins=None, e=None, A=list(A))
    if kind == "restart":
        s = _restart_inputs(c, seed)
        n, r, J = c["n"], c["groups"] * c["group"], s["Jf"].double()
        sg = [torch.where(x[:, :, 0] >= 0, 1.0, -1.0).double() for x in s["xs"]]
        f = torch.zeros((r, 32), dtype=torch.float64, device="cuda")
        for k in range(c["ckpts"]):
            x, g, old = s["xs"][k % 2].double(), sg[k % 2], sg[(k + 1) % 2]
            x1 = x[:, :, 0].contiguous()
            q = (x1 * x1).sum(0)
            f[:, 4 * k] = -(x1 * (J @ x1)).sum(0) / (n * q)
            f[:, 4 * k + 1] = -(g * (J @ g)).sum(0) / n
            f[:, 4 * k + 2] = q / (x * x).sum((0, 2))
            f[:, 4 * k + 3] = (g != old).sum(0).double() / n
        v = f.view(c["groups"], c["group"], 32)
        sd = v.std(dim=1, keepdim=True, unbiased=False)
        std = torch.where(sd > 0, (v - v.mean(1, keepdim=True)) / sd, torch.zeros_like(v)).view(r, 32)
        return dict(words=None, feats=f, std=std, logit=_mlp64(std, _bf(s["w"])), idx=None, x=None, pump=None)
    s = _train_inputs(c, seed)
    p = _bf(s["w"]).requires_grad_(True)
    z = _mlp64(s["xs"].double(), p)
    loss = torch.nn.functional.softplus(z) - s["y"].double() * z
    g, = torch.autograd.grad(loss.mean(), p)
    lr, b1, b2, eps = (_f32(v) for v in (LR, 0.9, 0.999, 1e-8))
    m = b1 * s["m"].double() + (1 - b1) * g
    v = b2 * s["v"].double() + (1 - b2) * g * g
    w = s["w"].double() - lr * (m / (1 - b1 ** 50)) / (torch.sqrt(v / (1 - b2 ** 50)) + eps)
    return dict(logit=z.detach(), loss=loss.detach(), grad=g, w=w, m=m, v=v, wb=_bf(w))
