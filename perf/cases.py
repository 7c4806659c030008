"""Timed cases of the framework: what a program that uses it has it do, over
the sizes it is used at.

Every case goes through the public entry points of paper_2603_14895_amd.fsg
(Simulation, Session, Batch, hk, GNN, SpreadEstimator).  Graphs are the
synthetic stand-ins of paper_2603_14895_amd.workloads: directed Erdos-Renyi,
Chung-Lu (exponent 2.5) and R-MAT; a case's graph, seed sets and keys come
from the seed alone, its sizes from the case.

listed() holds one case of each kind of use, draw() more cases of the same
kinds with their sizes spread over the kind's range.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2603_14895_amd import fsg
from paper_2603_14895_amd import workloads as W

DEV = "cuda"


# ------------------------------------------------------------------ cases --

def listed():
    return [
        # an analyst's single IC question on a small network: latency of one
        # call (directed G(1000, mean out-degree 10), p = 0.1, 100 replicates)
        dict(name="ic_small", kind="ic", graph="er", n=1000, deg=10.0, p=0.1, wc=False,
             seeds=10, B=100, out=False),
        # IC over many replicates, ragged batch, states and counts wanted
        dict(name="ic_multi", kind="ic", graph="cl", n=300_000, deg=20.0, p=0.05, wc=False,
             seeds=100, B=1000, out=False),
        # one SIR label of the surrogate's training data: counts only
        dict(name="sir_label", kind="epi", model="sir", n=20_000, deg=20.0, beta=0.03, gamma=0.1,
             steps=200, seeds=40, B=1024, out=False, states=False),
        # the large SIR workload: a million nodes, 1024 replicates, 200 steps
        dict(name="sir_large", kind="epi", model="sir", n=1_000_000, deg=20.0, beta=0.02,
             gamma=0.1, steps=200, seeds=10_000, B=1024, out=True, states=True),
        # stepwise use: a latent-state epidemic advanced in pieces with its
        # state tally after every step, then read
        dict(name="seir_session", kind="session", model="seir", n=100_000, deg=20.0, beta=0.04,
             gamma=0.1, alpha=0.3, steps=60, piece=20, seeds=1000, B=200),
        # linear threshold to absorption, ragged batch
        dict(name="lt_ragged", kind="lt", n=200_000, deg=25.0, seeds=300, B=300, out=False),
        # web-scale IC: R-MAT, weighted cascade, one word of replicates
        dict(name="ic_web", kind="web", scale=24, seeds=50, B=64),
        # Hegselmann-Krause opinions, aligned batch
        dict(name="hk", kind="hk", n=200_000, deg=20.0, eps=0.32, mu=1.0, steps=20, B=256),
        # weighted Hegselmann-Krause, a batch that no vector width divides
        dict(name="hk_ragged", kind="hk", n=20_000, deg=20.0, eps=0.32, mu=0.2, steps=20, B=50),
        # one training step of a surrogate member (forward, backward, gradient)
        dict(name="gnn_train", kind="train", n=100_000, deg=20.0, sets=8),
        # one spread query of the trained surrogate (ensemble of four)
        dict(name="spread_query", kind="query", n=100_000, deg=20.0, members=4, seeds=50,
             beta=0.03),
        # many jobs of different sizes and models in one batched run
        dict(name="batch_mixed", kind="batch", jobs=12, layout=7, n_lo=10_000, n_hi=100_000,
             b_lo=64, b_hi=1024),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["ic", "ic", "epi", "epi", "session", "lt", "web", "hk", "hk", "train",
                       "query", "batch"])
    out = rng.random() < 0.5
    deg = round(rng.uniform(5.0, 30.0), 2)
    if kind == "ic":
        n = _logint(rng, 1000, 300_000)
        B = _logint(rng, 33, min(2048, 300_000_000 // n))
        er = n < 5000 and rng.random() < 0.5
        deg = min(deg, 20.0) if er else deg
        out = out and (er or B > 64)
        return dict(kind="ic", graph="er" if er else "cl", n=n, deg=deg,
                    p=round(rng.uniform(0.02, 0.1), 4), wc=rng.random() < 0.3,
                    seeds=_logint(rng, 1, min(1000, n // 10)), B=B, out=out)
    if kind == "epi":
        n = _logint(rng, 2000, 1_000_000)
        B = _logint(rng, 33, min(2048, 400_000_000 // n))
        return dict(kind="epi", model=rng.choice(["sir", "sir", "sis", "si"]), n=n, deg=deg,
                    beta=round(rng.uniform(0.01, 0.05), 4), gamma=round(rng.uniform(0.05, 0.2), 4),
                    steps=rng.randint(30, 200), seeds=_logint(rng, 1, max(2, n // 100)), B=B,
                    out=out, states=rng.random() < 0.5)
    if kind == "session":
        n = _logint(rng, 2000, 200_000)
        steps = rng.randint(10, 80)
        return dict(kind="session", model=rng.choice(["seir", "seis", "sir"]), n=n, deg=deg,
                    beta=round(rng.uniform(0.02, 0.06), 4), gamma=round(rng.uniform(0.05, 0.2), 4),
                    alpha=round(rng.uniform(0.2, 0.6), 3), steps=steps,
                    piece=rng.randint(1, steps), seeds=_logint(rng, 1, n // 50),
                    B=_logint(rng, 33, 600))
    if kind == "lt":
        n = _logint(rng, 2000, 400_000)
        return dict(kind="lt", n=n, deg=deg, seeds=_logint(rng, 10, min(1000, n // 10)),
                    B=_logint(rng, 33, min(1024, 120_000_000 // n)), out=out)
    if kind == "web":
        return dict(kind="web", scale=rng.randint(18, 24), seeds=_logint(rng, 5, 500),
                    B=rng.randint(16, 64))
    if kind == "hk":
        n = _logint(rng, 1000, 200_000)
        B = _logint(rng, 3, min(400, 40_000_000 // n))
        if rng.random() < 0.4:
            B = max(4, B // 4 * 4)
        return dict(kind="hk", n=n, deg=deg, eps=0.32, mu=rng.choice([1.0, 0.2]),
                    steps=rng.randint(5, 20), B=B)
    if kind == "train":
        return dict(kind="train", n=_logint(rng, 2000, 100_000), deg=deg, sets=rng.randint(1, 8))
    if kind == "query":
        return dict(kind="query", n=_logint(rng, 2000, 150_000), deg=deg, members=rng.randint(2, 5),
                    seeds=_logint(rng, 5, 500), beta=round(rng.uniform(0.01, 0.05), 4))
    return dict(kind="batch", jobs=rng.randint(3, 16), layout=rng.randint(0, 1 << 20), n_lo=3000,
                n_hi=_logint(rng, 20_000, 100_000), b_lo=64, b_hi=rng.randint(200, 1024))


# ----------------------------------------------------------------- inputs --

def _sub(seed, tag):
    return (int(seed) * 1_000_003 + 7919 * tag + 12345) & 0x7FFFFFFF


def _chung_lu(n, mean_degree, seed):
    """The Chung-Lu recipe of workloads.chung_lu with the prefix sums of the
    weights formed on the host, so that the same seed always gives the same
    graph, and the pairs drawn on the GPU."""
    idx = torch.arange(n, dtype=torch.float64)
    w = (n / (idx + 1.0)) ** (1.0 / 1.5)
    cw = torch.cumsum(w * (mean_degree / w.mean()), 0)
    total = float(cw[-1])
    cw = cw.to(DEV)
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    m = int(round(n * mean_degree / 2))
    a, b = (torch.searchsorted(cw, torch.rand(m, generator=g, device=DEV, dtype=torch.float64) * total)
            .clamp_(max=n - 1) for _ in range(2))
    keep = a != b
    a, b = a[keep], b[keep]
    key = torch.unique(torch.minimum(a, b) * n + torch.maximum(a, b))
    lo = torch.div(key, n, rounding_mode="floor")
    hi = key - lo * n
    return W.pull_csr(n, torch.cat([lo, hi]), torch.cat([hi, lo]))


def _graph(case, seed):
    if case["kind"] == "web":
        return W.rmat(case["scale"], 16, 0.57, 0.19, 0.19, _sub(seed, 1), DEV)
    if case.get("graph") == "er":
        return W.erdos_renyi_directed(case["n"], case["deg"], _sub(seed, 1), DEV)
    return _chung_lu(case["n"], case["deg"], _sub(seed, 1))


def _seeds(n, k, seed):
    rng = np.random.default_rng(_sub(seed, 2))
    return np.sort(rng.choice(n, size=min(k, n), replace=False)).astype(np.int32)


def _opinions(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(_sub(seed, 3))
    return torch.rand((case["n"], case["B"]), generator=g, device=DEV) * 2.0 - 1.0


def _glorot(seed):
    """Parameters of one surrogate member: uniform Glorot weights, zero biases
    for the hidden layers (flat float32 in the library's order)."""
    rng = np.random.default_rng(seed)
    out = []
    for fan_in in (32, 128, 128):
        a = math.sqrt(6.0 / (fan_in + 64))
        out += [rng.uniform(-a, a, size=fan_in * 64), np.zeros(64)]
    a = math.sqrt(6.0 / 128)
    out += [rng.uniform(-a, a, size=64), np.zeros(1)]
    return np.concatenate(out).astype(np.float32)


def _train_inputs(case, graph, seed):
    """Masks, infection rates and targets (frequencies that grow with degree
    and rate, 1 on the seeds) of one training step."""
    n, sets = case["n"], case["sets"]
    rng = np.random.default_rng(_sub(seed, 4))
    masks = np.zeros((sets, n), dtype=np.uint8)
    for s in range(sets):
        k = max(1, int(round(math.exp(rng.uniform(0.0, math.log(min(1000, n // 2)))))))
        masks[s, rng.choice(n, size=k, replace=False)] = 1
    betas = rng.uniform(0.01, 0.05, size=sets).astype(np.float32)
    masks = torch.from_numpy(masks).to(DEV)
    g = torch.Generator(device=DEV)
    g.manual_seed(_sub(seed, 5))
    u = 0.2 + 0.8 * torch.rand((sets, n), generator=g, device=DEV)
    d = graph.indeg().to(torch.float32)[None, :]
    b = torch.from_numpy(betas).to(DEV)[:, None]
    y = 1.0 - torch.exp(d * u * torch.log1p(-b))
    y = torch.where(masks != 0, torch.ones_like(y), y).contiguous()
    return masks, [float(x) for x in betas], y


def _device_graph(graph, out=False):
    ptr, src = graph.numpy()
    return fsg.DeviceGraph(ptr, src, out=out)


def prepare(case, seed):
    kind = case["kind"]
    key = W.rng_key(_sub(seed, 6))
    st = dict(case=case, key=key)
    if kind == "batch":
        jobs = []
        for j in W.config_c3_jobs(case["jobs"], case["n_lo"], case["n_hi"], case["b_lo"],
                                  case["b_hi"], 300.0, case["layout"]):
            s = _sub(seed, 100 + j["index"])
            gr = _chung_lu(j["n"], j["mean_degree"], s)
            job = {k: j[k] for k in ("p", "ic_prob", "beta", "gamma", "max_steps") if k in j}
            job.update(graph=_device_graph(gr), model=j["model"], B=j["B"], rng_key=W.rng_key(s + 1),
                       seeds=_seeds(j["n"], j["n_seeds"], s))
            jobs.append(job)
        st["batch"] = fsg.Batch(jobs)
        st["jobs"] = jobs
        return st
    graph = _graph(case, seed)
    n = graph.n
    if kind == "hk":
        st.update(graph=_device_graph(graph), h0=_opinions(case, seed))
        return st
    if kind == "train":
        masks, betas, y = _train_inputs(case, graph, seed)
        net = fsg.GNN(1)
        net.set_params(_glorot(_sub(seed, 7)))
        st.update(graph=_device_graph(graph), reverse=_device_graph(W.reverse_graph(graph)),
                  net=net, masks=masks, betas=betas, y=y)
        return st
    st["seeds"] = _seeds(n, case["seeds"], seed)
    if kind == "query":
        members = []
        for i in range(case["members"]):
            net = fsg.GNN(i)
            net.set_params(_glorot(_sub(seed, 20 + i)))
            members.append(net)
        dg = _device_graph(graph)
        st.update(graph=dg, est=fsg.SpreadEstimator(members, dg, gamma=0.1, max_steps=200,
                                                    B_fallback=64, gate=dict(tau=float("inf"))))
        return st
    if kind == "session":
        st["graph"] = _device_graph(graph)
        return st
    dg = _device_graph(graph, out=case.get("out", False))
    if kind in ("ic", "web"):
        wc = kind == "web" or case["wc"]
        st["sim"] = fsg.Simulation(dg, "ic", case["B"], p=0.0 if wc else case["p"],
                                   ic_prob="weighted_cascade" if wc else "uniform", max_steps=-1)
    elif kind == "epi":
        st["sim"] = fsg.Simulation(dg, case["model"], case["B"], beta=case["beta"],
                                   gamma=case["gamma"], max_steps=case["steps"],
                                   want_states=case["states"])
    else:
        st["sim"] = fsg.Simulation(dg, "lt", case["B"], max_steps=-1)
    return st


# ------------------------------------------------------------------- runs --

def run(st):
    case, kind = st["case"], st["case"]["kind"]
    if kind == "batch":
        infos, _ = st["batch"].run()
        return dict(states=st["batch"].states, counts=st["batch"].counts,
                    steps=np.array([i.steps_run for i in infos]))
    if kind == "hk":
        h, counts, info = fsg.hk(st["graph"], st["h0"], case["eps"], case["steps"], mu=case["mu"])
        return dict(h=h, counts=counts, steps=int(info.steps_run))
    if kind == "train":
        loss = st["net"].train_step(st["graph"], st["reverse"], st["masks"], st["betas"], st["y"],
                                    1e-3, update=False)
        return dict(loss=loss, grads=st["net"].get_grads())
    if kind == "query":
        spread, unc, fallback = st["est"].estimate(st["seeds"], case["beta"], st["key"])
        return dict(spread=spread, uncertainty=unc, fallback=fallback)
    if kind == "session":
        s = fsg.Session(st["graph"], case["model"], st["seeds"], case["B"], st["key"],
                        beta=case["beta"], gamma=case["gamma"], alpha=case["alpha"],
                        max_steps=case["steps"])
        tallies, left = [], case["steps"]
        while left > 0:
            k = min(left, case["piece"])
            _, t = s.step(k, tally=True)
            tallies.append(t)
            left -= k
        states, counts, _ = s.read()
        s.close()
        return dict(states=states, counts=counts, tally=np.concatenate(tallies).astype(np.int64))
    sim = st["sim"]
    info = sim.run(st["seeds"], st["key"])
    return dict(states=sim.states, counts=sim.counts, steps=int(info.steps_run))


# ------------------------------------------------------- work and outputs --

def work(case):
    """Bytes and operations a pass cannot do without: the graph (row pointers
    and sources, 4 bytes each) and the other inputs read once, the outputs
    written once.  The cascades and epidemics are integer work; their
    operations are left at zero.  The web-scale cascade reaches few arcs, so
    only its outputs count."""
    kind = case["kind"]
    if kind == "batch":
        by = 0.0
        for j in W.config_c3_jobs(case["jobs"], case["n_lo"], case["n_hi"], case["b_lo"],
                                  case["b_hi"], 300.0, case["layout"]):
            by += 4.0 * j["n"] * (1 + j["mean_degree"]) + j["n"] * (j["B"] + 4.0)
        return dict(bytes=by, flops=0.0)
    if kind == "web":
        return dict(bytes=float(1 << case["scale"]) * (case["B"] + 4.0), flops=0.0)
    n, nnz = float(case["n"]), case["n"] * case["deg"]
    graph = 4.0 * (n + 1 + nnz)
    if kind == "hk":
        nb = n * case["B"]
        # per arc, replicate and step: a difference, a compare, two additions
        return dict(bytes=graph + 8.0 * nb + 4.0 * case["B"],
                    flops=4.0 * nnz * case["B"] * case["steps"])
    if kind in ("train", "query"):
        sets = case.get("sets", 1)
        reps = 3.0 if kind == "train" else float(case["members"])
        gemm = 2.0 * n * sets * 64 * (32 + 128 + 128 + 1)
        mean = nnz * sets * (16 + 64 + 64)
        by = graph * (2 if kind == "train" else 1) + n * sets * (5.0 if kind == "train" else 1.0)
        return dict(bytes=by + 4.0 * 18689 * reps, flops=(gemm + mean) * reps)
    by = graph + 4.0 * n
    if kind == "session" or case.get("states", True):
        by += n * case["B"]
    return dict(bytes=by, flops=0.0)


def _row_sums(x, graph):
    """Sums of the columns x[:, u] over the sources u of every row of the
    graph, in 64 bits ([k, n] -> [k, n]; prefix sums along the arcs)."""
    z = torch.zeros((x.shape[0], graph.nnz + 1), dtype=torch.float64, device=DEV)
    torch.cumsum(x, 1, out=z[:, 1:])
    return z[:, graph.ptr[1:]] - z[:, graph.ptr[:-1]]


def _hk_exact(case, seed):
    graph, n = _graph(case, seed), case["n"]
    if float(graph.nnz) * case["B"] * case["steps"] > 3.0e10:
        return None
    src = graph.src.to(torch.int64)
    dst = torch.repeat_interleave(torch.arange(n, device=DEV), graph.indeg())
    eps, mu = float(np.float32(case["eps"])), float(np.float32(case["mu"]))
    h0 = _opinions(case, seed)
    out = torch.empty(h0.shape, dtype=torch.float64, device=DEV)
    cols = max(1, (1 << 27) // max(1, graph.nnz))
    for c in range(0, case["B"], cols):
        h = h0[:, c:c + cols].t().to(torch.float64).contiguous()
        for _ in range(case["steps"]):
            hj = h[:, src]
            near = ((h[:, dst] - hj).abs() < eps).to(torch.float64)
            num, cnt = _row_sums(hj * near, graph), _row_sums(near, graph)
            h = torch.where(cnt > 0, (1.0 - mu) * h + mu * (num / cnt.clamp(min=1.0)), h)
        out[:, c:c + cols] = h.t()
    return dict(h=out, counts=None, steps=None)


class _Mean64(torch.autograd.Function):
    """Mean over in-neighbours of [k, n] features, 0 for an empty row."""

    @staticmethod
    def forward(ctx, x, graph, reverse, inv):
        ctx.rest = (reverse, inv)
        return _row_sums(x[:, graph.src.to(torch.int64)], graph) * inv

    @staticmethod
    def backward(ctx, g):
        reverse, inv = ctx.rest
        return _row_sums((g * inv)[:, reverse.src.to(torch.int64)], reverse), None, None, None


def _gnn_forward64(P, graph, reverse, mask, beta):
    """The surrogate's logits of one seed set in 64 bits."""
    d = graph.indeg().to(torch.float64)
    k = float(mask.sum())
    D = float(d[mask != 0].sum())
    xb, xd = 20.0 * beta, torch.log1p(d) * 0.125
    x = torch.zeros((16, graph.n), dtype=torch.float64, device=DEV)
    x[0] = mask.to(torch.float64)
    x[1] = xb
    x[2] = xd
    x[3] = 1.0
    x[4] = xb * xd
    x[5] = math.log1p(k) * 0.125
    x[6] = math.log1p(D) * 0.0625
    inv = 1.0 / d.clamp(min=1.0)
    for Wl, bl in P[:3]:
        mean = _Mean64.apply(x, graph, reverse, inv)
        x = torch.relu(Wl.t() @ torch.cat([x, mean], 0) + bl[:, None])
    wo, bo = P[3]
    return wo @ x + bo


def _params64(flat):
    t = torch.from_numpy(flat.astype(np.float64)).to(DEV).requires_grad_(True)
    P, o = [], 0
    for fan_in in (32, 128, 128):
        Wl = t[o:o + fan_in * 64].view(fan_in, 64)
        o += fan_in * 64
        P.append((Wl, t[o:o + 64]))
        o += 64
    P.append((t[o:o + 64], t[o + 64]))
    return t, P


def exact(case, seed):
    kind = case["kind"]
    if kind == "hk":
        return _hk_exact(case, seed)
    if kind not in ("train", "query"):
        return None
    graph, n = _graph(case, seed), case["n"]
    reverse = W.reverse_graph(graph)
    if kind == "query":
        mask = torch.zeros(n, dtype=torch.uint8, device=DEV)
        mask[torch.from_numpy(_seeds(n, case["seeds"], seed)).to(DEV).to(torch.int64)] = 1
        sp = []
        for i in range(case["members"]):
            with torch.no_grad():
                _, P = _params64(_glorot(_sub(seed, 20 + i)))
                z = _gnn_forward64(P, graph, reverse, mask, float(np.float32(case["beta"])))
                sp.append(float(torch.sigmoid(z).sum()))
        mean = float(np.mean(sp))
        return dict(spread=mean, uncertainty=float(np.std(sp, ddof=1)) / mean, fallback=None)
    masks, betas, y = _train_inputs(case, graph, seed)
    t, P = _params64(_glorot(_sub(seed, 7)))
    total = 0.0
    for s in range(case["sets"]):
        z = _gnn_forward64(P, graph, reverse, masks[s], betas[s])
        loss = torch.nn.functional.binary_cross_entropy_with_logits(
            z, y[s].to(torch.float64), reduction="sum") / (n * case["sets"])
        loss.backward(retain_graph=True)
        total += float(loss.detach())
    return dict(loss=total, grads=t.grad.detach())
