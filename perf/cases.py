"""The workloads this library's performance is measured on.

Each case is one pass through the public entry points as a user's program
calls them: an interior-point solver evaluating the callbacks of one model
(small and large, static, multi-period, security-constrained, rectangular),
a batch of load scenarios, and the learned warm-start proxy (its layers, its
loss, a training step, a prediction).  Sizes are those of the repository's
configurations, tests and benchmark; ``draw`` spreads over the same ranges.

  listed()            the named cases
  draw(rng)           one more case of the same ranges
  prepare(case, s)    models, weights and inputs in device memory, from seed s
  run(state)          one pass; returns its outputs
  work(case)          bytes and floating-point operations it cannot do without
  exact(case, s)      the same outputs from plain torch in 64 bits
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2510_12897_amd import opf, proxy, synth

F64 = torch.float64
RHO, OBJ_SCALE, VA_SPAN, LR = 10.0, 1e-3, 0.3, 3e-4


def listed():
    return [
        # the smallest call: one callback set of the 14-bus parity network, issued by itself
        dict(name="set_14", kind="set", N=14, L=20, G=5, form="polar"),
        # what a solver asks for in one iteration on a small network: the
        # trial point's f and c, then gradient, Jacobian and Hessian values
        # and the J^T y of its dual residual, each its own call
        dict(name="iter_300", kind="iter", N=300, L=410, G=60, form="polar"),
        # back-to-back sets of the 10,000-bus network from a HIP graph, as the benchmark's headline issues them
        dict(name="sets_10k", kind="graph", N=10000, L=13500, G=2000, form="polar", sets=16),
        # the rectangular form of the same network, one call
        dict(name="rect_10k", kind="set", N=10000, L=13500, G=2000, form="rect"),
        # 48 half-hour periods with storage units and user devices
        dict(name="mp48_storage", kind="mp", N=2000, L=2700, G=400, T=48, S=1, D=100),
        # security constraints: 200 branch-outage copies
        dict(name="n1_200", kind="n1", N=1000, L=1350, G=200, K=200),
        # 64 load scenarios of eight networks of 500 to 20,000 buses, one batched evaluation
        dict(name="batch_64", kind="batch", first=500, nets=8, scen=8),
        # the penalty and its gradient on a network beyond the one-launch loss: squashing,
        # arc flows, batched rows, penalty, batched J^T v
        dict(name="chain_1000", kind="chain", N=1000, L=1350, G=200, B=256),
        # a hidden layer of the proxy's network: forward (product, bias, GELU) and backward
        # (weight gradient, input gradient through the GELU below, bias sums)
        dict(name="layer_fwd", kind="layer_fwd", B=4096, fi=1024, fo=1024),
        dict(name="layer_bwd", kind="layer_bwd", B=4096, fi=1024, fo=1024),
        # one training step of the proxy at its benchmark shape
        dict(name="train_4096", kind="train", N=300, L=410, G=60, B=4096, width=1024, depth=3),
        # predictions for a small set of scenarios, as a solver asks for starts
        dict(name="predict_64", kind="predict", N=300, L=410, G=60, B=64, width=1024, depth=3),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _net_sizes(rng, lo, hi, even=False):
    N = _log(rng, lo, hi)
    G = max(1, int(N * rng.uniform(0.1, 0.3)))
    if even:
        N, G = N // 2 * 2, max(2, G // 2 * 2)
    return dict(N=N, L=min(int(N * rng.uniform(1.2, 1.5)) + 1, N * (N - 1) // 2), G=G)


def draw(rng):
    kind = rng.choice(["set", "iter", "graph", "mp", "n1", "batch", "chain", "layer_fwd", "layer_bwd", "train",
                       "predict"])
    form = rng.choice(["polar", "polar", "rect"])
    if kind in ("set", "iter"):
        return dict(kind=kind, form=form, **_net_sizes(rng, 14, 10000 if kind == "set" else 2000))
    if kind == "graph":
        return dict(kind=kind, form=form, sets=rng.randint(2, 16), **_net_sizes(rng, 100, 10000))
    if kind == "mp":
        return dict(kind=kind, T=rng.randint(2, 48), S=rng.randint(0, 1), D=rng.choice([0, rng.randint(1, 100)]),
                    **_net_sizes(rng, 100, 2000))
    if kind == "n1":
        return dict(kind=kind, K=_log(rng, 4, 200), **_net_sizes(rng, 100, 1000))
    if kind == "batch":
        return dict(kind=kind, first=rng.randint(20, 500), nets=rng.randint(1, 8), scen=rng.randint(1, 8))
    if kind == "chain":
        return dict(kind=kind, B=_log(rng, 4, 256), **_net_sizes(rng, 14, 1000, even=True))
    B = 4 * _log(rng, 4, 1024)
    if kind in ("layer_fwd", "layer_bwd"):
        return dict(kind=kind, B=B, fi=8 * _log(rng, 8, 128), fo=8 * _log(rng, 8, 128))
    return dict(kind=kind, B=B, width=4 * _log(rng, 32, 256), depth=rng.randint(1, 3),
                **_net_sizes(rng, 14, 300, even=True))


# ------------------------------------------------------------------ inputs
def _dev():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _gen(seed, dev):
    return torch.Generator(device=dev).manual_seed(int(seed))


@functools.lru_cache(maxsize=32)
def _network(N, L, G, variant=False):
    """The network a program loads from its files: its topology and branch data by size alone."""
    return synth.network(N, L, G, 1000 + N, variant=variant)


def _case_opts(case):
    """(network, model options) of a callback case."""
    cs = _network(case["N"], case["L"], case["G"], case["kind"] in ("set", "iter"))
    kw = {}
    if case.get("form", "polar") == "rect":
        kw["form"] = "rect"
    if case["kind"] == "mp":
        T = case["T"]
        pd_t, qd_t = synth.mp_loads(cs, T, 5)
        kw.update(n_periods=T, pd_t=pd_t, qd_t=qd_t, ramp_ratio=0.2)
        if case["S"]:
            kw.update(storage=synth.storage(cs, 6), stor_dt=0.5, stor_comp=True)
        if case["D"]:
            kw.update(devices=synth.devices(cs, case["D"], 7))
    if case["kind"] == "n1":
        K = min(case["K"], len(cs["extra_branches"]))
        kw.update(n_cont=K, outaged=synth.outages(cs, K, 8))
    return cs, kw


def _batch_nets(case):
    nets = []
    for k in range(case["nets"]):
        N = synth.BATCH_SIZES[k] if case["first"] == 500 else int(case["first"] * 1.5 ** k)
        nets.append(_network(N, int(round(1.35 * N)), int(round(0.2 * N))))
    return nets


def _dims(cs, nrep=1, npg=None, form="polar", kw=None):
    """(n, m) of a model."""
    kw = kw or {}
    N, L, G = cs["n_bus"], cs["n_branch"], cs["n_gen"]
    npg = nrep if npg is None else npg
    S = len(kw["storage"]["bus"]) if kw.get("storage") is not None else 0
    D = len(kw["devices"]["bus"]) if kw.get("devices") is not None else 0
    rows = 1 + 7 * L + 2 * N + (L + N if form == "rect" else 0) + S * (4 + bool(kw.get("stor_comp")))
    m = rows * nrep + (D * nrep if D else 0) + (G * (nrep - 1) if kw.get("n_periods", 1) > 1 else 0)
    return (2 * N + G + 4 * L + 6 * S + D) * nrep + G * npg, m


def _replicas(kw):
    T, K = kw.get("n_periods", 1), kw.get("n_cont", 0)
    return (K + 1, 1) if K else (T, T)


def _point(cs, kw, g, dev):
    """An evaluation point within the variable bounds, blocks in the model's order."""
    nrep, npg = _replicas(kw)
    N, L, G = cs["n_bus"], cs["n_branch"], cs["n_gen"]

    def uni(lo, hi, reps=1):
        lo = torch.as_tensor(np.asarray(lo, np.float64), device=dev).repeat(reps)
        hi = torch.as_tensor(np.asarray(hi, np.float64), device=dev).repeat(reps)
        return lo + (hi - lo) * torch.rand(lo.numel(), generator=g, device=dev, dtype=F64)

    va = uni(np.full(N, -math.pi / 6), np.full(N, math.pi / 6), nrep)
    vm = uni(cs["vmin"], cs["vmax"], nrep)
    if kw.get("form") == "rect":
        va, vm = vm * torch.cos(va), vm * torch.sin(va)
    arc = np.concatenate([cs["rate_a"], cs["rate_a"]])
    blocks = [va, vm, uni(cs["pmin"], cs["pmax"], npg), uni(cs["qmin"], cs["qmax"], nrep), uni(-arc, arc, nrep),
              uni(-arc, arc, nrep)]
    st, dv = kw.get("storage"), kw.get("devices")
    if st is not None:
        z = np.zeros(len(st["bus"]))
        for lo, hi in ((-st["rating"], st["rating"]), (st["qmin"], st["qmax"]), (-st["rating"], st["rating"]),
                       (z, st["emax"]), (z, st["chmax"]), (z, st["dismax"])):
            blocks.append(uni(lo, hi, nrep))
    if dv is not None:
        blocks.append(uni(dv["lo"], dv["hi"], nrep))
    return torch.cat(blocks)


def _callback_inputs(case, seed, dev):
    """[(x, y)] of every set of a callback case."""
    cs, kw = _case_opts(case)
    g = _gen(seed, dev)
    nrep, npg = _replicas(kw)
    n, m = _dims(cs, nrep, npg, kw.get("form", "polar"), kw)
    out = []
    for _ in range(case.get("sets", 1)):
        x = _point(cs, kw, g, dev)
        assert x.numel() == n
        out.append((x, torch.randn(m, generator=g, device=dev, dtype=F64)))
    return cs, kw, out


def _batch_inputs(case, seed, dev):
    """Per instance (network, pd, qd, x, y); objective weight 1."""
    g, rng = _gen(seed, dev), np.random.default_rng(seed)
    out = []
    for cs in _batch_nets(case):
        n, m = _dims(cs)
        for _ in range(case["scen"]):
            pd = rng.uniform(0.0, 0.5, cs["n_bus"])
            x = _point(cs, {}, g, dev)
            out.append((cs, pd, 0.3 * pd, x, torch.randn(m, generator=g, device=dev, dtype=F64)))
    return out


def _loads(cs, B, g, dev):
    """B load samples [B, 2N] (+-30 % per bus) and the proxy's features of them."""
    base = torch.as_tensor(np.concatenate([cs["pd"], cs["qd"]]), device=dev)
    u = torch.rand(B, cs["n_bus"], generator=g, device=dev, dtype=F64) * 2.0 - 1.0
    loads = base * (1.0 + 0.3 * torch.cat([u, u], dim=1))
    feats = torch.cat([u, u], dim=1) * math.sqrt(3.0)
    return loads, feats.to(torch.float32)


def _mlp_state(dims, g, dev):
    """Parameters and Adam moments of a network some way into its training,
    as a program resuming from its checkpoint holds them."""
    w, m1, m2 = [], [], []
    for k, (fi, fo) in enumerate(zip(dims[:-1], dims[1:])):
        s = math.sqrt(2.0 / fi) * (0.2 if k == len(dims) - 2 else 1.0)
        for cnt, scale in ((fo * fi, s), (fo, 0.05)):
            w.append(torch.randn(cnt, generator=g, device=dev) * scale)
            m1.append(torch.randn(cnt, generator=g, device=dev) * 0.05)
            m2.append(0.01 + 0.01 * torch.rand(cnt, generator=g, device=dev))
    return torch.cat(w), torch.cat(m1), torch.cat(m2)


def _proxy_dims(case):
    N, G = case["N"], case["G"]
    return [2 * N] + [case["width"]] * case["depth"] + [2 * N + 2 * G]


def _proxy_inputs(case, seed, dev):
    cs, g = _network(case["N"], case["L"], case["G"]), _gen(seed, dev)
    w, m1, m2 = _mlp_state(_proxy_dims(case), g, dev)
    loads, feats = _loads(cs, case["B"], g, dev)
    return cs, w, m1, m2, loads, feats


def _chain_inputs(case, seed, dev):
    cs, g = _network(case["N"], case["L"], case["G"]), _gen(seed, dev)
    loads, _ = _loads(cs, case["B"], g, dev)
    z = torch.randn(case["B"], 2 * case["N"] + 2 * case["G"], generator=g, device=dev)
    return cs, loads, z


def _layer_inputs(case, seed, dev):
    B, fi, fo, g = case["B"], case["fi"], case["fo"], _gen(seed, dev)
    bf = torch.bfloat16
    pre = torch.randn(B, fi, generator=g, device=dev)
    h = torch.nn.functional.gelu(pre).to(bf)
    W = (torch.randn(fo, fi, generator=g, device=dev) * math.sqrt(2.0 / fi)).to(bf)
    bias = torch.randn(fo, generator=g, device=dev) * 0.05
    dpre = (torch.randn(B, fo, generator=g, device=dev) / B).to(bf)
    return h, W, bias, pre, dpre


# ----------------------------------------------------------------- passes
def _outs(model, sets, dev):
    e = lambda *s: torch.empty(*s, dtype=F64, device=dev)  # noqa: E731
    return dict(f=e(sets), g=e(sets, model.n), c=e(sets, model.m), J=e(sets, model.nnzj), H=e(sets, model.nnzh))


def prepare(case, seed):
    kind, dev = case["kind"], _dev()
    st = dict(kind=kind)
    if kind in ("set", "iter", "graph", "mp", "n1"):
        cs, kw, st["xy"] = _callback_inputs(case, seed, dev)
        st["model"] = model = opf.Model(cs, device=0, **kw)
        if kind == "iter":
            return st
        st["out"] = _outs(model, len(st["xy"]), dev)
        if kind == "graph":  # the program's captured evaluation loop
            s = torch.cuda.Stream()
            s.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(s):
                _sets(st)
            torch.cuda.synchronize()
            st["graph"] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(st["graph"], stream=s):
                _sets(st)
            torch.cuda.synchronize()
    elif kind == "batch":
        inst = _batch_inputs(case, seed, dev)
        models = [opf.Model(cs, device=0) for cs in _batch_nets(case)]
        idx = [k for k in range(case["nets"]) for _ in range(case["scen"])]
        st["batch"] = b = opf.Batch(models, idx, np.concatenate([i[1] for i in inst]),
                                    np.concatenate([i[2] for i in inst]))
        st["X"], st["Y"] = torch.cat([i[3] for i in inst]), torch.cat([i[4] for i in inst])
        st["sigma"] = torch.ones(len(inst), dtype=F64, device=dev)
        st["out"] = [torch.empty(k, dtype=F64, device=dev) for k in (b.n_inst, b.n, b.m, b.nnzj, b.nnzh)]
    elif kind == "chain":
        cs, st["loads"], z = _chain_inputs(case, seed, dev)
        st["pen"] = proxy.Penalty(cs, case["B"], rho=RHO, obj_scale=OBJ_SCALE)
        st["squash"] = proxy.Squash(st["pen"].model, VA_SPAN)
        st["z"] = z.requires_grad_(True)
    elif kind in ("layer_fwd", "layer_bwd"):
        st["h"], st["W"], st["bias"], st["pre"], st["dpre"] = _layer_inputs(case, seed, dev)
        B, fi, fo = case["B"], case["fi"], case["fo"]
        if kind == "layer_fwd":
            st["z"] = torch.empty(B, fo, device=dev)
            st["act"] = torch.empty(B, fo, dtype=torch.bfloat16, device=dev)
        else:
            st["splits"] = proxy.gemm_splits(fo, fi, B)
            st["work"] = torch.empty(max(st["splits"] * fo * fi, 4), device=dev)
            st["dW"] = torch.empty(fo, fi, device=dev)
            st["d"] = torch.empty(B, fi, dtype=torch.bfloat16, device=dev)
            st["part"] = torch.empty((B + 127) // 128, fi, device=dev)
            st["db"] = torch.empty(fi, device=dev)
    else:
        cs, w, m1, m2, st["loads"], st["feats"] = _proxy_inputs(case, seed, dev)
        st["px"] = px = proxy.WarmStartProxy(cs, B=case["B"], width=case["width"], depth=case["depth"], rho=RHO,
                                             obj_scale=OBJ_SCALE, va_span=VA_SPAN)
        with torch.no_grad():
            for t, v in ((px.mlp.flat, w), (px.mlp.m1, m1), (px.mlp.m2, m2)):
                t.copy_(v)
        px.mlp.step = 100
        px.mlp.step_dev.fill_(100)
        px.mlp.sync_bf16()
    return st


def _sets(st):
    o = st["out"]
    for k, (x, y) in enumerate(st["xy"]):
        st["model"].eval_set(x, y, 1.0, o["f"][k:k + 1], o["g"][k], o["c"][k], o["J"][k], o["H"][k])


def run(st):
    kind = st["kind"]
    if kind in ("set", "mp", "n1"):
        _sets(st)
        return st["out"]
    if kind == "graph":
        st["graph"].replay()
        return st["out"]
    if kind == "iter":
        m, (x, y) = st["model"], st["xy"][0]
        f, c = m.obj(x), m.cons(x)
        g, J, H = m.grad(x), m.jac_coord(x), m.hess_coord(x, y, 1.0)
        return dict(f=f, c=c, g=g, J=J, H=H, jty=m.jtprod(x, y))
    if kind == "batch":
        return list(st["batch"].eval(st["X"], st["Y"], st["sigma"], *st["out"]))
    if kind == "chain":
        pen, N = st["pen"], st["pen"].N
        pen.set_loads(st["loads"][:, :N], st["loads"][:, N:])
        loss = pen(st["squash"](st["z"]))
        (dz,) = torch.autograd.grad(loss.sum(), st["z"])
        return dict(loss=loss.detach(), cvio=pen.last["cvio"], dz=dz)
    if kind == "layer_fwd":
        B, fi = st["h"].shape
        fo = st["W"].shape[0]
        proxy.gemm_mixed(0, st["h"], True, fi, st["W"], True, fi, st["z"], fo, B, fo, fi, bias=st["bias"],
                         act=st["act"], act_bf16=True)
        return dict(z=st["z"], act=st["act"])
    if kind == "layer_bwd":
        B, fi = st["h"].shape
        fo = st["W"].shape[0]
        proxy.gemm_mixed(2, st["dpre"], True, fo, st["h"], True, fi, st["dW"], fi, fo, fi, B, splits=st["splits"],
                         work=st["work"])
        proxy.gemm_gelu_bwd(st["dpre"], True, fo, st["W"], True, fi, st["pre"], fi, st["d"], fi, B, fi, fo, st["part"])
        proxy._check(proxy.lib().prox_colsum_parts(proxy._p(st["part"]), st["part"].shape[0], fi, proxy._p(st["db"]),
                                                   1.0, proxy._stream()))
        return dict(dW=st["dW"], d=st["d"], db=st["db"])
    px = st["px"]
    if kind == "train":
        loss = px.train_step(st["loads"], st["feats"], lr=LR)
        return dict(loss=loss, flat=px.mlp.flat, m1=px.mlp.m1, m2=px.mlp.m2)
    x, cvio = px.predict(st["loads"], st["feats"])
    return dict(x=x, cvio=cvio)


# ------------------------------------------------------------------- work
def _set_bytes(cs, kw, shared=False):
    """Bytes of one callback set: every input read once, every output written
    once (shared: without the network's own data, read once for a whole batch)."""
    nrep, npg = _replicas(kw)
    rect = kw.get("form") == "rect"
    n, m = _dims(cs, nrep, npg, "rect" if rect else "polar", kw)
    N, L, G = cs["n_bus"], cs["n_branch"], cs["n_gen"]
    S = len(kw["storage"]["bus"]) if kw.get("storage") is not None else 0
    D = len(kw["devices"]["bus"]) if kw.get("devices") is not None else 0
    comp, T = bool(kw.get("stor_comp")), kw.get("n_periods", 1)
    # Jacobian: reference 1, flows 5, angle 2 (rectangular: 4 + 4), balance (bus entries, arcs, generators), thermal 2
    nnzj = 1 + 20 * L + (8 * L + 2 * N if rect else 2 * L) + 2 * ((2 if rect else 1) * N + 2 * L + G) + 4 * L
    nnzh = (2 * N + 4 * L if rect else 3 * N + 4 * L) + 4 * L
    nnzj += S * (4 + 5 + 4 + 2 + 2 + 2 * comp) + 2 * D
    nnzh += S * (4 + comp)
    nnzj, nnzh = nnzj * nrep - S, nnzh * nrep + G * npg
    if T > 1:
        nnzj += 2 * G * (T - 1) + D * (2 * T - 1)
    elif D:
        nnzj += D
    loads = 16 * N * (T if kw.get("pd_t") is not None else 1)
    model = (96 if rect else 80) * L + 16 * N + 28 * G + 4 * (2 * L + 2 * N + 2 + G) + 4 * kw.get("n_cont", 0)
    model += 108 * S + 28 * D
    return 8 * (2 * n + 2 * m + nnzj + nnzh) + loads + (0 if shared else model)


def _loss_bytes(case):
    N, L, G, B = case["N"], case["L"], case["G"], case["B"]
    return B * (4 * (2 * N + 2 * G) + 16 * N + 16) + 80 * L + 100 * N + 60 * G


def work(case):
    kind = case["kind"]
    if kind in ("set", "iter", "graph", "mp", "n1"):
        cs, kw = _case_opts(case)
        b = _set_bytes(cs, kw)
        if kind == "iter":  # and J^T y: x and y read, a vector of n written
            n, m = _dims(cs, 1, 1, kw.get("form", "polar"), kw)
            b += 8 * (2 * n + m)
        nrep = _replicas(kw)[0]
        return dict(bytes=b * case.get("sets", 1), flops=300.0 * cs["n_branch"] * nrep * case.get("sets", 1))
    if kind == "batch":
        nets = _batch_nets(case)
        b = sum(_set_bytes(cs, {}) + (case["scen"] - 1) * _set_bytes(cs, {}, shared=True) for cs in nets)
        return dict(bytes=b, flops=300.0 * case["scen"] * sum(cs["n_branch"] for cs in nets))
    if kind == "chain":
        N, L, G, B = case["N"], case["L"], case["G"], case["B"]
        return dict(bytes=_loss_bytes(case) + B * 4 * (2 * N + 2 * G), flops=B * (250.0 * L + 150.0 * N))
    if kind in ("layer_fwd", "layer_bwd"):
        B, fi, fo = case["B"], case["fi"], case["fo"]
        if kind == "layer_fwd":
            return dict(bytes=2 * (B * fi + fo * fi) + 4 * fo + 6 * B * fo, flops=2.0 * B * fi * fo)
        return dict(bytes=2 * (B * fo + B * fi + fo * fi) + 4 * B * fi + 4 * fo * fi + 2 * B * fi + 4 * fi,
                    flops=4.0 * B * fi * fo)
    dims, B = _proxy_dims(case), case["B"]
    mac = sum(a * b for a, b in zip(dims[:-1], dims[1:]))
    par = mac + sum(dims[1:])
    loss_flops = B * (250.0 * case["L"] + 150.0 * case["N"])
    if kind == "train":  # weights, both moments read and written, BF16 copy read and written
        return dict(bytes=28 * par + _loss_bytes(case) + 8 * B * case["N"], flops=6.0 * B * mac + loss_flops)
    n = 2 * case["N"] + 2 * case["G"] + 4 * case["L"]
    return dict(bytes=2 * par + B * (24 * case["N"] + 8 * n + 8), flops=2.0 * B * mac + loss_flops / 2)


# ------------------------------------------------- the same in plain torch
def _admittance(cs, dev):
    t = lambda k: torch.as_tensor(np.asarray(cs[k], np.float64), device=dev)  # noqa: E731
    y = 1.0 / torch.complex(t("r"), t("x"))
    half = torch.complex(torch.zeros_like(t("b")), t("b") / 2)
    tap = torch.polar(t("tap"), t("shift"))
    return (y + half) / t("tap") ** 2, -y / tap.conj(), -y / tap, y + half


class _Rows:
    """The rows of one model: each block an elementwise function of a few
    variables per row (derivatives by autograd), plus linear entries."""

    def __init__(self, x, y):
        self.x, self.y, self.dev = x, y, x.device
        self.c = torch.zeros(0, dtype=F64, device=self.dev)
        self.j, self.h = [], []

    def add(self, cols, fn, pairs=(), linear=()):
        """cols: column indices per argument of fn; pairs: its second
        derivatives; linear: (row in the block, column, coefficient)."""
        r0, v = self.c.numel(), [self.x[k].clone().requires_grad_(True) for k in cols]
        c = fn(*v)
        rows = torch.arange(r0, r0 + c.numel(), device=self.dev)
        gr = torch.autograd.grad(c.sum(), v, create_graph=bool(pairs))
        for k, gk in zip(cols, gr):
            self.j.append((rows, k, gk.detach()))
        for a, b in pairs:
            d = torch.autograd.grad(gr[a].sum(), v[b], retain_graph=True, allow_unused=True)[0] \
                if gr[a].requires_grad else None
            d = torch.zeros_like(c) if d is None else d
            self.h.append((torch.maximum(cols[a], cols[b]), torch.minimum(cols[a], cols[b]), (self.y[rows] * d).detach()))
        c = c.detach()
        for row, col, coef in linear:
            c = c.index_add(0, row, coef * self.x[col])
            self.j.append((row + r0, col, coef))
        self.c = torch.cat([self.c, c])

    @staticmethod
    def _merge(parts, n):
        key = torch.cat([r * n + k for r, k, _ in parts])
        u, inv = torch.unique(key, return_inverse=True)
        return torch.zeros(u.numel(), dtype=F64, device=key.device).index_add_(0, inv, torch.cat([v for _, _, v in parts]))

    def values(self):
        n = self.x.numel()
        return self.c, self._merge(self.j, n), self._merge(self.h, n)

    def jty(self):
        out = torch.zeros_like(self.x)
        for r, k, v in self.j:
            out.index_add_(0, k, v * self.y[r])
        return out


def _exact_set(cs, kw, x, y, pd=None, qd=None):
    """(f, g, c, J, H, rows) of one callback set, objective weight 1."""
    dev = x.device
    nrep, npg = _replicas(kw)
    T, rect = kw.get("n_periods", 1), kw.get("form") == "rect"
    N, L, G = cs["n_bus"], cs["n_branch"], cs["n_gen"]
    ix = lambda a: torch.as_tensor(np.asarray(a, np.int64), device=dev)  # noqa: E731
    dv = lambda a: torch.as_tensor(np.asarray(a, np.float64), device=dev)  # noqa: E731
    rep = torch.arange(nrep, device=dev)[:, None]
    over = lambda off, cnt, idx, r=rep: (off + cnt * r + idx[None, :]).reshape(-1)  # noqa: E731  per replica
    tile = lambda a: a.repeat(nrep)  # noqa: E731
    o_va, o_vm, o_pg = 0, N * nrep, 2 * N * nrep
    o_qg = o_pg + G * npg
    o_p = o_qg + G * nrep
    o_q = o_p + 2 * L * nrep
    o_s = o_q + 2 * L * nrep
    fb, tb, gb, ref, ln, bn, gn = (ix(cs["f_bus"]), ix(cs["t_bus"]), ix(cs["gen_bus"]), ix(cs["ref_bus"]),
                                   torch.arange(L, device=dev), torch.arange(N, device=dev),
                                   torch.arange(G, device=dev))
    Yff, Yft, Ytf, Ytt = _admittance(cs, dev)
    on = torch.ones(nrep, L, dtype=F64, device=dev)
    if kw.get("n_cont"):
        on[torch.arange(1, nrep, device=dev), ix(kw["outaged"])] = 0.0
    on = on.reshape(-1)
    A = lambda t: tile(t) * on  # noqa: E731  admittance terms, zero where a branch is out
    pf, pt = over(o_p, 2 * L, ln), over(o_p + L, 2 * L, ln)
    qf, qt = over(o_q, 2 * L, ln), over(o_q + L, 2 * L, ln)
    c2, c1, c0 = dv(cs["c2"]).repeat(npg), dv(cs["c1"]).repeat(npg), dv(cs["c0"]).repeat(npg)
    pgv = x[o_pg:o_qg]
    f = (c2 * pgv ** 2 + c1 * pgv + c0).sum()
    g = torch.zeros_like(x)
    g[o_pg:o_qg] = 2 * c2 * pgv + c1
    R = _Rows(x, y)
    pgc = torch.arange(o_pg, o_qg, device=dev)
    R.h.append((pgc, pgc, 2 * c2))
    bf, bt = over(o_va, N, fb), over(o_va, N, tb)
    mf, mt = over(o_vm, N, fb), over(o_vm, N, tb)
    R.add([over(o_vm if rect else o_va, N, ref)], lambda v: v)
    flows = (("f", Yff, Yft, pf, qf), ("t", Ytt, Ytf, pt, qt))
    pairs = [(0, 0), (1, 0), (1, 1), (2, 0), (2, 1), (2, 2), (3, 0), (3, 1), (3, 2), (3, 3)]
    rpairs = [(0, 0), (1, 0), (1, 1), (2, 2), (3, 2), (3, 3), (2, 1), (3, 0)]
    for side, Ys, Ym, pc, qc in flows:
        gs_, bs_, gm, bm = A(Ys.real), A(Ys.imag), A(Ym.real), A(Ym.imag)
        for re in (True, False):
            def row(a, b, u, w, arc, side=side, re=re, gs_=gs_, bs_=bs_, gm=gm, bm=bm):
                if rect:  # a, b = vr_f, vr_t; u, w = vi_f, vi_t
                    own = (a * a + u * u) if side == "f" else (b * b + w * w)
                    cr, si = a * b + u * w, (u * b - a * w) if side == "f" else (a * w - u * b)
                else:
                    own = u * u if side == "f" else w * w
                    th = a - b if side == "f" else b - a
                    cr, si = u * w * torch.cos(th), u * w * torch.sin(th)
                return arc - (gs_ * own + gm * cr + bm * si) if re else arc - (-bs_ * own + gm * si - bm * cr)
            R.add([bf, bt, mf, mt, pc if re else qc], row, rpairs if rect else pairs)
    if rect:
        for lim in ("angmax", "angmin"):
            tn = tile(torch.tan(dv(cs[lim])))
            R.add([bf, bt, mf, mt], lambda a, b, u, w, tn=tn: (u * b - a * w) - tn * (a * b + u * w),
                  [(1, 0), (3, 2), (2, 1), (3, 0)])
    else:
        R.add([bf, bt], lambda a, b: a - b)
    ones = torch.ones(L * nrep, dtype=F64, device=dev)
    go = torch.ones(G * nrep, dtype=F64, device=dev)
    if pd is None:
        pd, qd = (dv(kw["pd_t"]), dv(kw["qd_t"])) if kw.get("pd_t") is not None else (tile(dv(cs["pd"])), tile(dv(cs["qd"])))
    allb = over(o_vm, N, bn)
    st, de = kw.get("storage"), kw.get("devices")
    S, D = (len(st["bus"]) if st is not None else 0), (len(de["bus"]) if de is not None else 0)
    sn, dn = torch.arange(S, device=dev), torch.arange(D, device=dev)
    sv = [over(o_s + k * S * nrep, S, sn) for k in range(6)]
    o_u = o_s + 6 * S * nrep
    dc = over(o_u, D, dn)
    for k, (arc_f, arc_t, gen, sh, ld) in enumerate(((pf, pt, over(o_pg, G if npg > 1 else 0, gn), cs["gs"], pd),
                                                     (qf, qt, over(o_qg, G, gn), -np.asarray(cs["bs"]), qd))):
        lin = [(over(0, N, fb), arc_f, ones), (over(0, N, tb), arc_t, ones), (over(0, N, gb), gen, -go)]
        if S:
            lin.append((over(0, N, ix(st["bus"])), sv[k], torch.ones(S * nrep, dtype=F64, device=dev)))
        if D:
            lin.append((over(0, N, ix(de["bus"])), dc, tile(dv(de["cp" if k == 0 else "cq"]))))
        s = tile(dv(sh))
        if rect:
            R.add([over(o_va, N, bn), allb], lambda a, b, s=s, ld=ld: ld + s * (a * a + b * b), [(0, 0), (1, 1)], lin)
        else:
            R.add([allb], lambda v, s=s, ld=ld: ld + s * v * v, [(0, 0)], lin)
    r2 = tile(dv(cs["rate_a"])) ** 2
    for a, b in ((pf, qf), (pt, qt)):
        R.add([a, b], lambda p, q: p * p + q * q - r2, [(0, 0), (1, 1)])
    if rect:
        R.add([over(o_va, N, bn), allb], lambda a, b: a * a + b * b, [(0, 0), (1, 1)])
    later = torch.arange(1, nrep, device=dev)[:, None]
    if T > 1:
        R.add([over(o_pg, G, gn, later), over(o_pg, G, gn, later - 1)], lambda a, b: a - b)
    if S:
        par = {k: tile(dv(st[k])) for k in ("eta_c", "eta_d", "r", "x", "ploss", "qloss", "rating")}
        dt = kw["stor_dt"]
        first = torch.zeros(1, 1, dtype=torch.long, device=dev)
        e0, ec, ed = dv(st["e0"]), dv(st["eta_c"]), dv(st["eta_d"])
        ocol = lambda k, r: over(o_s + k * S * nrep, S, sn, r)  # noqa: E731
        R.add([ocol(3, first), ocol(4, first), ocol(5, first)], lambda se, sc, sd: se - e0 - dt * (ec * sc - sd / ed))
        if nrep > 1:
            ec1, ed1 = ec.repeat(nrep - 1), ed.repeat(nrep - 1)
            R.add([ocol(3, later), ocol(3, later - 1), ocol(4, later), ocol(5, later)],
                  lambda se, sp, sc, sd: se - sp - dt * (ec1 * sc - sd / ed1))
        vmc = over(o_vm, N, ix(st["bus"]))
        lp = [(0, 0), (1, 0), (1, 1), (2, 0), (2, 2)]
        R.add([vmc, sv[0], sv[1], sv[4], sv[5]],
              lambda v, p, q, c, d: p + d - c - par["ploss"] - par["r"] * (p * p + q * q) / v ** 2, lp)
        R.add([vmc, sv[0], sv[1], sv[2]],
              lambda v, p, q, c: q - c - par["qloss"] - par["x"] * (p * p + q * q) / v ** 2, lp)
        R.add([sv[0], sv[1]], lambda p, q: p * p + q * q - par["rating"] ** 2, [(0, 0), (1, 1)])
        if kw.get("stor_comp"):
            R.add([sv[4], sv[5]], lambda c, d: c * d, [(1, 0)])
    if D:
        cost = tile(dv(de["cost"]))
        f = f + (cost * x[dc]).sum()
        g[dc] = cost
        if nrep > 1:
            R.add([over(o_u, D, dn, later), over(o_u, D, dn, later - 1)], lambda a, b: a - b)
        R.add([over(o_u, D, dn, torch.zeros(1, 1, dtype=torch.long, device=dev))], lambda a: a)
    return (f, g, *R.values(), R)


def _exact_squash(cs, z):
    """x = (va, vm, pg, qg) [B, .] of the network output z (vm, va, pg, qg)."""
    N, G = cs["n_bus"], cs["n_gen"]
    t = lambda k: torch.as_tensor(np.asarray(cs[k], np.float64), device=z.device)  # noqa: E731
    box = lambda lo, hi, v: t(lo) + (t(hi) - t(lo)) * torch.sigmoid(v)  # noqa: E731
    keep = torch.ones(N, dtype=F64, device=z.device)
    keep[torch.as_tensor(np.asarray(cs["ref_bus"], np.int64), device=z.device)] = 0.0
    return (VA_SPAN * torch.tanh(z[:, N:2 * N]) * keep, box("vmin", "vmax", z[:, :N]),
            box("pmin", "pmax", z[:, 2 * N:2 * N + G]), box("qmin", "qmax", z[:, 2 * N + G:]))


def _exact_loss(cs, z, loads):
    """Per-sample loss, largest violation and completed x of z [B, 2N + 2G]."""
    dev, N = z.device, cs["n_bus"]
    t = lambda k: torch.as_tensor(np.asarray(cs[k], np.float64), device=dev)  # noqa: E731
    ix = lambda k: torch.as_tensor(np.asarray(cs[k], np.int64), device=dev)  # noqa: E731
    va, vm, pg, qg = _exact_squash(cs, z)
    fb, tb, gb = ix("f_bus"), ix("t_bus"), ix("gen_bus")
    Yff, Yft, Ytf, Ytt = _admittance(cs, dev)
    V = torch.polar(vm, va)
    Vf, Vt = V[:, fb], V[:, tb]
    Sf, St = Vf * (Yff * Vf + Yft * Vt).conj(), Vt * (Ytf * Vf + Ytt * Vt).conj()
    arcs = (Sf.real, St.real, Sf.imag, St.imag)
    over = lambda v, lo, hi: torch.clamp(v - hi, min=0.0) + torch.clamp(v - lo, max=0.0)  # noqa: E731
    bal = []
    for ld, a, b, gen, sh in ((loads[:, :N], arcs[0], arcs[1], pg, t("gs")), (loads[:, N:], arcs[2], arcs[3], qg, -t("bs"))):
        r = ld + sh * vm * vm
        bal.append(r.index_add(1, fb, a).index_add(1, tb, b).index_add(1, gb, -gen))
    rate = t("rate_a")
    dev_ = [over(va[:, fb] - va[:, tb], t("angmin"), t("angmax")), *bal,
            torch.clamp(arcs[0] ** 2 + arcs[2] ** 2 - rate ** 2, min=0.0),
            torch.clamp(arcs[1] ** 2 + arcs[3] ** 2 - rate ** 2, min=0.0), *[over(a, -rate, rate) for a in arcs]]
    f = (t("c2") * pg ** 2 + t("c1") * pg + t("c0")).sum(1)
    loss = RHO * sum((d * d).sum(1) for d in dev_) + OBJ_SCALE * f
    cvio = torch.stack([d.detach().abs().amax(1) for d in dev_]).amax(0)
    return loss, cvio, torch.cat([va, vm, pg, qg, *arcs], dim=1)


def _exact_mlp(dims, flat, feats):
    h, off = feats, 0
    for k, (fi, fo) in enumerate(zip(dims[:-1], dims[1:])):
        W, b = flat[off:off + fo * fi].view(fo, fi), flat[off + fo * fi:off + fo * fi + fo]
        off += fo * fi + fo
        h = h @ W.t() + b
        if k < len(dims) - 2:
            h = torch.nn.functional.gelu(h)
    return h


def exact(case, seed):
    kind, dev = case["kind"], _dev()
    if kind in ("set", "graph", "mp", "n1"):
        cs, kw, xy = _callback_inputs(case, seed, dev)
        v = [_exact_set(cs, kw, x, y)[:5] for x, y in xy]
        return {k: torch.stack([s[i] for s in v]) for i, k in enumerate("fgcJH")}
    if kind == "iter":
        cs, kw, ((x, y),) = _callback_inputs(case, seed, dev)
        f, g, c, J, H, rows = _exact_set(cs, kw, x, y)
        return dict(f=f, c=c, g=g, J=J, H=H, jty=rows.jty())
    if kind == "batch":
        v = []
        for cs, pd, qd, x, y in _batch_inputs(case, seed, dev):
            v.append(_exact_set(cs, {}, x, y, torch.as_tensor(pd, device=dev), torch.as_tensor(qd, device=dev))[:5])
        return [torch.stack([s[0] for s in v])] + [torch.cat([s[i] for s in v]) for i in range(1, 5)]
    if kind == "chain":
        cs, loads, z = _chain_inputs(case, seed, dev)
        z = z.to(F64).requires_grad_(True)
        loss, cvio, _ = _exact_loss(cs, z, loads)
        (dz,) = torch.autograd.grad(loss.sum(), z)
        return dict(loss=loss.detach(), cvio=cvio, dz=dz)
    if kind in ("layer_fwd", "layer_bwd"):
        h, W, bias, pre, dpre = (t.to(F64) for t in _layer_inputs(case, seed, dev))
        if kind == "layer_fwd":
            z = h @ W.t() + bias
            return dict(z=z, act=torch.nn.functional.gelu(z))
        pre = pre.requires_grad_(True)
        (gp,) = torch.autograd.grad(torch.nn.functional.gelu(pre).sum(), pre)
        d = (dpre @ W) * gp
        return dict(dW=dpre.t() @ h, d=d, db=d.sum(0))
    cs, w, m1, m2, loads, feats = _proxy_inputs(case, seed, dev)
    dims = _proxy_dims(case)
    w = w.to(F64).requires_grad_(kind == "train")
    loss, cvio, x = _exact_loss(cs, _exact_mlp(dims, w, feats.to(F64)), loads)
    if kind == "predict":
        return dict(x=x, cvio=cvio)
    (g,) = torch.autograd.grad(loss.mean(), w)
    m1, m2 = 0.9 * m1.to(F64) + 0.1 * g, 0.999 * m2.to(F64) + 0.001 * g * g
    step = LR * (m1 / (1 - 0.9 ** 101)) / ((m2 / (1 - 0.999 ** 101)).sqrt() + 1e-8)
    return dict(loss=loss.mean().detach(), flat=(w - step).detach(), m1=m1, m2=m2)
