"""The work a program gives this library, as timed cases.

Four kinds of call, each through the entry points of the binding:

  layer       one MoE layer of one server over one batch: routing and
              server-expert selection with the dispatch list
              (ordermoe_route_select), then the local expert FFN and combine
              (ordermoe_local_moe_forward).  Decode (1 to 128 tokens),
              prefill chunks (a few hundred tokens, ragged) and whole prefill
              batches, in bf16 and in fp32.
  similarity  the similarity model of a layer from its calibration tokens
              (ordermoe_build_similarity: device part and host grouping).
  replan      the transition statistics and the look-ahead tables of a stack
              (ordermoe_estimate_transitions_device,
              ordermoe_build_lookahead_device), rebuilt whenever the cost
              weights or the deployment change.
  pack        the weights of a server's experts into the layout the forward
              reads (ordermoe_pack_gate_up, ordermoe_pack_down), at load time
              and whenever an expert moves.

The layer shapes are those of the library's own workloads (Mixtral-, Qwen-MoE-
and DeepSeek-MoE-shaped layers, the 128-expert decode layer, the small fp32
layer).  Inputs follow the same recipe: N(0, 1) tokens, router rows in planted
clusters, N(0, 0.02^2) expert weights, the deployment spread over the servers,
a synthetic network in the testbed's ranges.  A token whose router logits lie
within rounding distance of a tie has no single right decision (the library
flags it), so such tokens are drawn again: every other decision is the same
for every correct implementation.
"""
import functools
import math

import numpy as np
import torch

from paper_2607_17154_amd import ordermoe as om

GMAX = om.MAX_SUBS
MARGIN = 1.0e-4               # the library's own tie margin

# The layers: hidden size, routed experts, FFN width, top-k, shared experts,
# experts per planted cluster, router noise, servers, copies of each expert
# over the servers, where tokens start, most tokens of a batch.
SHAPES = {
    "mixtral": dict(d=4096, E=8, f=14336, k=2, n_shared=0, csize=2, sigma=0.1, M=4, copies=1, loc="zero"),
    "qwen": dict(d=2048, E=60, f=1408, k=4, n_shared=4, csize=5, sigma=0.15, M=4, copies=1, loc="uniform"),
    "deepseek": dict(d=2048, E=64, f=1408, k=6, n_shared=2, csize=4, sigma=0.2, M=8, copies=1, loc="zero"),
    "stack": dict(d=4096, E=128, f=1536, k=8, n_shared=0, csize=4, sigma=0.15, M=8, copies=2, loc="zero"),
    "small": dict(d=512, E=8, f=1024, k=2, n_shared=0, csize=2, sigma=0.1, M=2, copies=1, loc="zero"),
    "medium": dict(d=1024, E=40, f=640, k=5, n_shared=1, csize=4, sigma=0.3, M=5, copies=1, loc="uniform"),
}


def _layer(shape, T, dtype="bf16", Qbar=0.25, spent=0.0, pin=1, allow_sub=1, renorm=1):
    c = dict(kind="layer", shape=shape, dtype=dtype, T=T, Qbar=Qbar, spent=spent, pin=pin,
             allow_sub=allow_sub, renorm=renorm)
    c.update(SHAPES[shape])
    return c


def listed():
    return [
        # one user's next token at a 128-expert layer: the smallest call, where
        # launches and the weights of eight experts are all there is
        dict(_layer("stack", 1, Qbar=1.0), name="decode_T1"),
        # a decode batch at the same layer: every local expert has a few rows
        dict(_layer("stack", 64, Qbar=1.0), name="decode_T64"),
        # a chunk of a chunked prefill, a ragged number of tokens on all
        # servers with part of their quality budget spent
        dict(_layer("qwen", 501, spent=0.2), name="chunk_qwen_T501"),
        # whole prefill batches of the three layer shapes
        dict(_layer("mixtral", 4096), name="prefill_mixtral_T4096"),
        dict(_layer("qwen", 8192), name="prefill_qwen_T8192"),
        dict(_layer("deepseek", 16384), name="prefill_deepseek_T16384"),
        # fp32 storage: the small layer used for verification, and a ragged
        # batch of a middling layer with a shared expert
        dict(_layer("small", 256, dtype="f32"), name="f32_small_T256"),
        dict(_layer("medium", 1001, dtype="f32"), name="f32_medium_T1001"),
        # similarity model of a 128-expert layer (bf16) and of the small fp32 layer
        dict(kind="similarity", dtype="bf16", T=65536, d=4096, E=128, k=8, csize=4, sigma=0.15,
             name="similarity_T65536_E128"),
        dict(kind="similarity", dtype="f32", T=2048, d=512, E=8, k=2, csize=2, sigma=0.1,
             name="similarity_f32_T2048_E8"),
        # tables of a 32-layer stack of 128 experts on 8 servers, look-ahead depth 3
        dict(kind="replan", N=32, E=128, M=8, H=3, T=2048, csize=4, copies=2, Qbar=1.0, pin=1, allow_sub=1,
             name="replan_N32_E128_H3"),
        # a server's two Mixtral-shaped experts at load time
        dict(kind="pack", dtype="bf16", n=2, d=4096, f=14336, name="pack_mixtral_n2"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    r = rng.random()
    if r < 0.64:
        # bf16 layers from one token to a whole prefill batch
        shape = rng.choice(["mixtral", "qwen", "deepseek", "stack", "medium"])
        top = {"mixtral": 4000, "qwen": 8000, "deepseek": 16000, "stack": 4000, "medium": 8000}[shape]
        return _layer(shape, _log(rng, 1, top), Qbar=rng.choice([0.12, 0.25, 1.0]), spent=rng.choice([0.0, 0.1]),
                      pin=rng.choice([1, 1, 0]), allow_sub=rng.choice([1, 1, 1, 0, 2]), renorm=rng.choice([1, 1, 0]))
    if r < 0.76:
        return _layer(rng.choice(["small", "medium"]), _log(rng, 1, 2049), dtype="f32", Qbar=rng.choice([0.12, 0.25]),
                      spent=rng.choice([0.0, 0.1]), allow_sub=rng.choice([1, 1, 0]))
    if r < 0.87:
        if rng.random() < 0.7:
            s = SHAPES[rng.choice(["mixtral", "qwen", "deepseek", "stack"])]
            return dict(kind="similarity", dtype="bf16", T=_log(rng, 1024, 60000), d=s["d"], E=s["E"], k=s["k"],
                        csize=s["csize"], sigma=s["sigma"])
        s = SHAPES[rng.choice(["small", "medium"])]
        return dict(kind="similarity", dtype="f32", T=_log(rng, 512, 8192), d=s["d"], E=s["E"], k=s["k"],
                    csize=s["csize"], sigma=s["sigma"])
    if r < 0.94:
        E = 4 * rng.randint(2, 32)
        return dict(kind="replan", N=rng.randint(2, 32), E=E, M=rng.choice([2, 4, 8]), H=rng.randint(2, 5),
                    T=_log(rng, 512, 4096), csize=4, copies=rng.choice([1, 2]), Qbar=rng.choice([0.25, 1.0]),
                    pin=rng.choice([1, 1, 0]), allow_sub=rng.choice([1, 1, 0, 2]))
    s = SHAPES[rng.choice(["qwen", "deepseek", "stack", "medium"])]
    dtype = rng.choice(["bf16", "bf16", "f32"])
    return dict(kind="pack", dtype=dtype, n=rng.randint(1, 16), d=s["d"], f=s["f"])


# ---------------------------------------------------------------- inputs
def _dt(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _gen(seed, device):
    g = torch.Generator(device=device)
    g.manual_seed(int(seed))
    return g


def _np_rng(seed):
    return np.random.default_rng([int(seed), 77])


def _router(case, g, dtype):
    """Rows in planted clusters: centre + sigma * noise, scaled so that logits are O(1)."""
    E, d, cs = case["E"], case["d"], case["csize"]
    c = torch.randn((E + cs - 1) // cs, d, generator=g, device=g.device)
    n = torch.randn(E, d, generator=g, device=g.device)
    cl = torch.arange(E, device=g.device) // cs
    return ((c[cl] + case["sigma"] * n) * d ** -0.5).to(dtype)


def _tokens(case, g, w, T, dtype):
    """N(0, 1) tokens; those within the tie margin of the router are drawn again."""
    x = torch.randn(T, case["d"], generator=g, device=g.device).to(dtype)
    k1 = min(case["k"] + 1, case["E"])
    if k1 < 2:
        return x
    wt = w.double().t().contiguous()
    todo = torch.arange(T, device=g.device)
    for _ in range(12):
        top = torch.topk(x[todo].double() @ wt, k1, dim=1).values
        todo = todo[(top[:, :-1] - top[:, 1:]).min(1).values < 2 * MARGIN]
        if todo.numel() == 0:
            break
        x[todo] = torch.randn(todo.numel(), case["d"], generator=g, device=g.device).to(dtype)
    return x


def _deployment(E, M, copies):
    """Experts spread over the servers, group mates apart; further copies one or more servers on."""
    x = np.zeros((M, E), np.uint8)
    for j in range(E):
        for c in range(copies):
            x[(j + c * (1 + (j // M) % max(M - 1, 1))) % M, j] = 1
    return x


def _network(M, rng):
    B = rng.uniform(1e9, 10e9, (M, M))
    tau = rng.uniform(0.2e-3, 20e-3, (M, M))
    B, tau = np.triu(B, 1) + np.triu(B, 1).T, np.triu(tau, 1) + np.triu(tau, 1).T
    np.fill_diagonal(B, 10e9)
    return B, tau, rng.uniform(20e12, 110e12, M)


def _plan(case, w, seed):
    """The layer's decision tables (numpy): substitutes, server masks, static costs."""
    E, M, cs = case["E"], case["M"], case["csize"]
    h = w.double().cpu().numpy()
    nrm = np.linalg.norm(h, axis=1)
    sim = ((h @ h.T) / np.outer(nrm, nrm)).astype(np.float32)
    group = np.arange(E) // cs
    x = _deployment(E, M, case["copies"])
    B, tau, F = _network(M, _np_rng(seed))
    c = np.full(E, 6.0 * case["d"] * case["f"])
    d_ref = c.mean() / F.mean()
    z = 8.0 * case["d"] * (2 if case["dtype"] == "bf16" else 4)
    t1_k = np.full((E, GMAX), -1, np.int32)
    t1_q = np.full((E, GMAX), np.inf, np.float32)
    t1_n = np.zeros(E, np.int32)
    for r in range(E):
        q = (np.float32(1) - sim[r]) * np.float32(0.5)
        ks = sorted((j for j in range(E) if j != r and group[j] == group[r] and sim[r, j] >= np.float32(0.7)),
                    key=lambda j: (q[j], j))[:GMAX]
        t1_k[r, :len(ks)], t1_q[r, :len(ks)], t1_n[r] = ks, q[ks], len(ks)
    mask = (x.astype(np.uint64) << np.arange(M, dtype=np.uint64)[:, None]).sum(0).astype(np.uint32)
    S = np.empty((M, M, E), np.float32)
    for s in range(M):
        for m in range(M):
            t = z / B[s, m] + tau[s, m] if s != m else 0.0
            S[s, m] = (0.5 * (t + c / F[m]) / d_ref).astype(np.float32)
    return dict(t1_k=t1_k, t1_q=t1_q, t1_n=t1_n, srvmask=mask, S=S, x=x)


def _batch(case, g, w, T):
    x = _tokens(case, g, w, T, _dt(case))
    if case["loc"] == "zero":
        loc = torch.zeros(T, dtype=torch.uint8, device=g.device)
    else:
        loc = torch.randint(0, case["M"], (T,), generator=g, device=g.device).to(torch.uint8)
    qhat = torch.rand(T, generator=g, device=g.device) * case["spent"]
    return x, loc, qhat


def _experts(case, g, n):
    """Weights of n experts in the Linear layout [out][in]."""
    dt, d, f = _dt(case), case["d"], case["f"]
    mk = lambda *s: torch.randn(*s, generator=g, device=g.device, dtype=dt) * 0.02  # noqa: E731
    return mk(n, f, d), mk(n, f, d), mk(n, d, f)


def _weights(case, g, plan):
    """Server 0's routed experts, and the shared experts as one wide one."""
    routed = _experts(case, g, max(int(plan["x"][0].sum()), 1))
    ns = case["n_shared"]
    shared = _experts(dict(case, f=ns * case["f"]), g, 1) if ns else None
    return routed, shared


def _pack(wg, wu, wd):
    n, f, d = wg.shape
    gu = torch.empty((n, 2 * f, d), dtype=wg.dtype, device=wg.device)
    dn = torch.empty_like(wd)
    om.ordermoe_pack_gate_up(wg, wu, gu)
    om.ordermoe_pack_down(wd, dn)
    return gu, dn


def prepare(case, seed):
    return {"layer": _prepare_layer, "similarity": _prepare_similarity, "replan": _prepare_replan,
            "pack": _prepare_pack}[case["kind"]](case, seed)


def _prepare_layer(case, seed):
    T, k, M = case["T"], case["k"], case["M"]
    g = _gen(seed, "cuda")
    w = _router(case, g, _dt(case))
    plan = _plan(case, w, seed)
    x, loc, qhat = _batch(case, g, w, T)
    routed, shared = _weights(case, g, plan)
    gu, dn = _pack(*routed)
    sgu, sdn = _pack(*shared) if shared else (None, None)
    tabs = {n: torch.from_numpy(plan[n].view(np.int32) if n == "srvmask" else plan[n]).cuda()
            for n in ("t1_k", "t1_q", "t1_n", "srvmask", "S")}
    code = om.BF16 if case["dtype"] == "bf16" else om.F32
    layer = om.make_layer(code, case["d"], case["E"], k, M, GMAX, w, tabs, case["Qbar"], 0.5, case["pin"],
                          case["allow_sub"], case["renorm"])
    local = [int(j) for j in np.nonzero(plan["x"][0])[0]]
    ex = om.make_experts(code, case["d"], case["f"], case["E"], local, gu, dn, case["n_shared"], sgu, sdn)
    out = om.alloc_route_out(T, k, M, "cuda")
    out["dispatch"].zero_()       # only the entries of the list are written
    need = max(om.ordermoe_route_workspace_size(T, k, M), 1), max(om.ordermoe_forward_workspace_size(ex, T, k), 1)
    ws = [torch.empty(n, dtype=torch.uint8, device="cuda") for n in need]
    return dict(kind="layer", T=T, k=k, layer=layer, ex=ex, x=x, loc=loc, qhat=qhat, out=out,
                outs=om.route_out_struct(out), ws=ws, y=torch.empty((T, case["d"]), dtype=_dt(case), device="cuda"),
                ro=torch.empty(len(local) + 2, dtype=torch.int32, device="cuda"), keep=(w, tabs, gu, dn, sgu, sdn))


def _calibration(case, seed):
    g = _gen(seed, "cuda")
    w = _router(case, g, _dt(case))
    return w, _tokens(case, g, w, case["T"], _dt(case))


def _prepare_similarity(case, seed):
    w, x = _calibration(case, seed)
    ws = torch.empty(om.ordermoe_similarity_workspace_size(case["T"], case["d"], case["E"]), dtype=torch.uint8,
                     device="cuda")
    return dict(kind="similarity", x=x, w=w, k=case["k"], ws=ws,
                top1=torch.empty(case["T"], dtype=torch.int32, device="cuda"))


def _stack_model(case, seed):
    """What a stack's look-ahead is built from: top-1 experts of the calibration
    tokens (mostly staying in their cluster from layer to layer), similarities
    by cluster, deployment, network, thresholds from 0.9 down to 0.5."""
    N, E, M, cs, T = (case[n] for n in ("N", "E", "M", "csize", "T"))
    rng = _np_rng(seed)
    group = np.stack([rng.permutation(E) for _ in range(N)]).argsort(1) // cs
    top1 = np.empty((N, T), np.int32)
    top1[0] = rng.integers(0, E, T)
    for l in range(1, N):
        order = np.argsort(group[l], kind="stable").reshape(-1, cs)
        stay = order[group[l - 1][top1[l - 1]], rng.integers(0, cs, T)]
        top1[l] = np.where(rng.random(T) < 0.7, stay, rng.integers(0, E, T))
    sim = rng.uniform(-0.1, 0.1, (N, E, E))
    same = group[:, :, None] == group[:, None, :]
    sim = np.where(same, rng.uniform(0.55, 0.99, (N, E, E)), sim)
    sim = (sim + sim.transpose(0, 2, 1)) / 2
    sim[:, np.arange(E), np.arange(E)] = 1.0
    x = np.stack([np.roll(_deployment(E, M, case["copies"]), l, axis=0) for l in range(N)])
    B, tau, F = _network(M, rng)
    c = rng.uniform(0.8, 1.2, (N, E)) * 6.0 * 4096 * 1536
    theta = np.array([0.5 + 0.4 * (N - 1 - l) / (N - 1) for l in range(N)], np.float32)
    return dict(top1=top1, x=x, sim=sim.astype(np.float32), group_of=group.astype(np.int32), theta=theta,
                z_bits=np.full(N, 8.0 * 4096 * 2), c=c, d_ref=c.mean(1) / F.mean(), B=B, tau=tau, F=F)


def _prepare_replan(case, seed):
    m = {n: torch.from_numpy(np.ascontiguousarray(v)).cuda() for n, v in _stack_model(case, seed).items()}
    N, E, M = case["N"], case["E"], case["M"]
    L = om.lib()
    mk = lambda n: torch.empty(max(int(n), 1), dtype=torch.uint8, device="cuda")  # noqa: E731
    return dict(kind="replan", case=case, m=m, P=torch.empty((N - 1, E, E), dtype=torch.float64, device="cuda"),
                phi=torch.empty((N, M, E), dtype=torch.float64, device="cuda"),
                ws_t=mk(L.ordermoe_transitions_device_workspace_size(N, E)),
                ws_l=mk(L.ordermoe_lookahead_device_workspace_size(N, E, M)))


def _prepare_pack(case, seed):
    wg, wu, wd = _experts(case, _gen(seed, "cuda"), case["n"])
    n, f, d = wg.shape
    return dict(kind="pack", w=(wg, wu, wd), gu=torch.empty((n, 2 * f, d), dtype=wg.dtype, device="cuda"),
                dn=torch.empty_like(wd))


# ---------------------------------------------------------------- the calls
def run(s):
    if s["kind"] == "layer":
        o = s["out"]
        om.ordermoe_route_select(s["layer"], s["x"], s["T"], s["loc"], s["qhat"], o, s["ws"][0],
                                 out_struct=s["outs"])
        om.ordermoe_local_moe_forward(s["ex"], s["x"], s["T"], s["k"], o["w"], o["exec_k"], o["exec_m"], s["loc"], 0,
                                      s["y"], s["ro"], s["ws"][1])
        return dict(o, y=s["y"], row_offsets=s["ro"])
    if s["kind"] == "similarity":
        r = om.ordermoe_build_similarity(s["x"], s["w"], s["k"], 0.7, 0.5, s["ws"], top1=s["top1"])
        return dict(sim=r["sim_dev"], counts=r["counts_dev"], group_of=r["group_of"], importance=r["importance"],
                    top1=s["top1"])
    if s["kind"] == "replan":
        c, m = s["case"], s["m"]
        om.ordermoe_estimate_transitions_device(m["top1"], c["E"], s["P"], s["ws_t"])
        om.ordermoe_build_lookahead_device(c["H"], s["P"], m["x"], m["sim"], m["group_of"], m["theta"], m["z_bits"],
                                           m["c"], m["d_ref"], m["B"], m["tau"], m["F"], 0.5, 0.5, c["Qbar"],
                                           c["pin"], c["allow_sub"], s["phi"], s["ws_l"])
        return dict(P=s["P"], phi=s["phi"])
    om.ordermoe_pack_gate_up(s["w"][0], s["w"][1], s["gu"])
    om.ordermoe_pack_down(s["w"][2], s["dn"])
    return dict(gate_up=s["gu"], down=s["dn"])


# ---------------------------------------------------------------- plain reference
def _decide(case, plan, lg, loc, qhat):
    """Decisions of a batch from its fp64 logits: per slot in rank order, the
    target if it is local (pin), else the cheapest (server, expert) of the
    target and its substitutes within the budget, in fp32 as the tables are."""
    dev = lg.device
    k, M, E = case["k"], case["M"], case["E"]
    t = {n: torch.from_numpy(plan[n].astype(np.int64) if n in ("t1_k", "t1_n") else plan[n]).to(dev)
         for n in ("t1_k", "t1_q", "t1_n", "S", "x")}
    v, idx = torch.sort(lg, dim=1, descending=True, stable=True)
    v, idx = v[:, :min(k + 1, E)], idx[:, :k]
    margin = (v[:, :-1] - v[:, 1:]).min(1).values if v.shape[1] > 1 else torch.full_like(v[:, 0], math.inf)
    e = torch.exp(v[:, :k] - v[:, :1])
    den = e.sum(1) if case["renorm"] else torch.exp(lg - v[:, :1]).sum(1)
    locl = loc.long()
    on = bool(case["allow_sub"]) and case["Qbar"] > 0
    cq = float(np.float32(0.5) / np.float32(case["Qbar"])) if case["Qbar"] > 0 else 0.0
    Qbar = float(np.float32(case["Qbar"]))
    rows = torch.arange(lg.shape[0], device=dev)
    ms = torch.arange(M, device=dev)
    qh = qhat.clone()
    exec_k, exec_m = [], []
    for s in range(k):
        r = idx[:, s]
        cand = torch.cat([r[:, None], t["t1_k"][r]], 1)
        q = torch.cat([torch.zeros_like(qh)[:, None], t["t1_q"][r]], 1)
        j = torch.arange(1 + GMAX, device=dev)[None]
        ok = (j == 0) | ((j <= t["t1_n"][r][:, None]) & on & (qh[:, None] + q <= Qbar))
        cand, q = torch.where(ok, cand, r[:, None]), torch.where(ok, q, torch.zeros_like(q))
        held = ok[:, :, None] & (t["x"].t()[cand] > 0)
        if case["allow_sub"] == 2:
            held &= (j[:, :, None] == 0) | (ms[None, None] == locl[:, None, None])
        J = (cq * q.double()[:, :, None] + t["S"][locl[:, None, None], ms[None, None], cand[:, :, None]].double()).float()
        J = torch.where(held, J, torch.full_like(J, math.inf))
        order = j[:, :, None] * 64 + (ms[None, None] != locl[:, None, None]) * 32 + ms[None, None]
        best = torch.where(J == J.amin((1, 2), keepdim=True), order, torch.full_like(order, 1 << 20)).flatten(1).argmin(1)
        pos, m = best // M, best % M
        kk = cand[rows, pos]
        if case["pin"]:
            keep = t["x"][locl, r] > 0
            pos, m, kk = torch.where(keep, 0, pos), torch.where(keep, locl, m), torch.where(keep, r, kk)
        qh = qh + torch.where(pos > 0, q[rows, pos], torch.zeros_like(qh))
        exec_k.append(kk)
        exec_m.append(m)
    return dict(idx=idx, w=e / den[:, None], margin=margin, exec_k=torch.stack(exec_k, 1),
                exec_m=torch.stack(exec_m, 1), qhat_out=qh.double())


def _exact_layer(case, seed):
    g = _gen(seed, "cuda")
    w = _router(case, g, _dt(case))
    plan = _plan(case, w, seed)
    x, loc, qhat = _batch(case, g, w, case["T"])
    routed, shared = _weights(case, g, plan)
    x = x.double()
    dec = _decide(case, plan, x @ w.double().t().contiguous(), loc, qhat)
    y = torch.zeros_like(x)

    def ffn(xs, wg, wu, wd):
        a = xs @ wg.double().t().contiguous()
        return (a / (1 + torch.exp(-a)) * (xs @ wu.double().t().contiguous())) @ wd.double().t().contiguous()

    for i, e in enumerate(np.nonzero(plan["x"][0])[0]):
        wt = (dec["w"] * ((dec["exec_k"] == int(e)) & (dec["exec_m"] == 0))).sum(1)
        at = torch.nonzero(wt > 0).flatten()
        if at.numel():
            y[at] += wt[at, None] * ffn(x[at], *(v[i] for v in routed))
    if shared:
        at = torch.nonzero(loc == 0).flatten()
        if at.numel():
            y[at] += ffn(x[at], *(v[0] for v in shared))
    names = ("idx", "w", "margin", "flag", "exec_k", "exec_m", "cls", "qhat_out", "loc_out", "dispatch", "dst_count",
             "counters", "row_offsets")
    return dict({n: dec[n] if n in ("w", "margin", "qhat_out") else None for n in names}, y=y)


def _exact_similarity(case, seed):
    w, x = _calibration(case, seed)
    gram = torch.zeros((case["E"], case["E"]), dtype=torch.float64, device="cuda")
    wt = w.double().t().contiguous()
    cnt = torch.zeros(case["E"], dtype=torch.float64, device="cuda")
    for i in range(0, case["T"], 8192):
        h = x[i:i + 8192].double() @ wt
        gram += h.t().contiguous() @ h
        cnt += torch.bincount(torch.topk(h, case["k"], dim=1).indices.flatten(), minlength=case["E"])
    n = gram.diagonal().sqrt()
    sim = gram / (n[:, None] * n[None])
    sim.fill_diagonal_(1.0)
    return dict(sim=sim, counts=None, group_of=None, importance=None, top1=None)


def _exact_replan(case, seed):
    m = _stack_model(case, seed)
    N, E, M, H = (case[n] for n in ("N", "E", "M", "H"))
    P = np.zeros((N - 1, E, E))
    for l in range(N - 1):
        np.add.at(P[l], (m["top1"][l], m["top1"][l + 1]), 1.0)
        P[l] /= np.maximum(P[l].sum(1, keepdims=True), 1.0)
    phi = np.zeros((N, M, E))
    Qbar = float(np.float32(case["Qbar"]))
    subs = bool(case["allow_sub"]) and Qbar > 0
    off = ~np.eye(M, dtype=bool)
    for _ in range(H - 1):
        new = np.zeros_like(phi)
        for l in range(N - 1):
            n = l + 1
            delay = np.where(off, m["z_bits"][n] / m["B"] + m["tau"], 0.0)[:, :, None] + m["c"][n] / m["F"][:, None]
            cost = 0.5 * delay / m["d_ref"][n] + phi[n][None]                      # [s, m', k']
            q = ((np.float32(1) - m["sim"][n]) * np.float32(0.5)).astype(np.float64)
            np.fill_diagonal(q, 0.0)
            cand = (m["group_of"][n][:, None] == m["group_of"][n][None]) & (m["sim"][n] >= m["theta"][n]) & subs
            np.fill_diagonal(cand, True)
            held = np.where(m["x"][n] > 0, 0.0, np.inf)                            # [m', k']
            V = np.empty((M, E))
            for s in range(M):
                hs = np.broadcast_to(held[None], (E, M, E)).copy()                 # [r', m', k']
                if case["allow_sub"] == 2:
                    far = (np.arange(M) != s)[None, :, None] & ~np.eye(E, dtype=bool)[:, None, :]
                    hs[far] = np.inf
                v = cost[s][None] + hs + (0.5 * q / Qbar if Qbar > 0 else q * 0)[:, None, :]
                v = np.where(cand[:, None, :], v, np.inf).min((1, 2))
                own = cost[s, s]
                V[s] = np.where((m["x"][n][s] > 0) & bool(case["pin"]), own, v)
            new[l] = V @ P[l].T
        phi = new
    return dict(P=P, phi=phi)


def exact(case, seed):
    if case["kind"] == "layer":
        return _exact_layer(case, seed)
    if case["kind"] == "similarity":
        return _exact_similarity(case, seed)
    if case["kind"] == "replan":
        return _exact_replan(case, seed)
    wg, wu, wd = _experts(case, _gen(seed, "cuda"), case["n"])
    n, f, d = wg.shape
    gu = torch.stack([wg.view(n, f // 32, 32, d), wu.view(n, f // 32, 32, d)], 2).reshape(n, 2 * f, d)
    if case["dtype"] == "bf16":
        blk = lambda t, N, K: t.view(n, N // 256, 256, K // 64, 64).transpose(2, 3).reshape(n, N, K)  # noqa: E731
        gu, wd = blk(gu, 2 * f, d), blk(wd, d, f)
    return dict(gate_up=gu.double(), down=wd.double())


# ---------------------------------------------------------------- work and tolerance
@functools.lru_cache(maxsize=None)
def _local_work(key):
    """(rows, shared rows, experts with a row) of server 0, from a sample of at
    most 512 tokens of the layer."""
    case = dict(key)
    T = min(case["T"], 512)
    g = _gen(1, "cpu")
    w = _router(case, g, torch.float32)
    plan = _plan(case, w, 1)
    x = torch.randn(T, case["d"], generator=g)
    loc = torch.zeros(T, dtype=torch.uint8) if case["loc"] == "zero" else (torch.arange(T) % case["M"]).to(torch.uint8)
    dec = _decide(case, plan, (x @ w.t()).double(), loc, torch.full((T,), case["spent"] / 2))
    here = torch.zeros(T, case["E"], dtype=torch.bool)
    for s in range(case["k"]):
        at = torch.nonzero(dec["exec_m"][:, s] == 0).flatten()
        here[at, dec["exec_k"][at, s]] = True
    scale = case["T"] / T
    return int(here.sum()) * scale, (int((loc == 0).sum()) * scale if case["n_shared"] else 0.0), int(here.any(0).sum())


def work(case):
    if case["kind"] == "pack":
        return {"bytes": 2.0 * 3 * case["n"] * case["d"] * case["f"] * (2 if case["dtype"] == "bf16" else 4), "flops": 0}
    if case["kind"] == "replan":
        N, E, M, H = (case[n] for n in ("N", "E", "M", "H"))
        read = 4 * N * case["T"] + N * M * E + N * E * E * 4 + N * E * 12
        return {"bytes": float(read + (N - 1) * E * E * 8 + N * M * E * 8),
                "flops": float((H - 1) * (N - 1) * M * E * (2 * E + 4 * case["csize"] * case["copies"]))}
    esz = 2 if case["dtype"] == "bf16" else 4
    T, d, E, k = case["T"], case["d"], case["E"], case["k"]
    if case["kind"] == "similarity":
        return {"bytes": float((T + E) * d * esz + T * 4 + E * E * 4), "flops": 2.0 * T * E * d + 2.0 * T * E * E}
    rows, shared, active = _local_work(tuple(sorted((n, v) for n, v in case.items() if n != "name")))
    f, ns = case["f"], case["n_shared"]
    byt = (2 * T + E) * d * esz + T * k * 14 + T * 15 + (active + (ns if shared else 0)) * 3 * d * f * esz
    return {"bytes": float(byt), "flops": 2.0 * T * E * d + 6.0 * d * f * (rows + ns * shared)}


def tolerance(case):
    if case["kind"] in ("replan", "pack"):
        return "exact"
    if case["kind"] == "similarity":
        return {"rel": 1e-5}
    # bf16: the activations and the row outputs are rounded to 8 bits of mantissa
    return {"rel": 1e-2, "max": 0.2} if case["dtype"] == "bf16" else {"rel": 1e-5, "max": 1e-3}
