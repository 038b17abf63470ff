"""The work a program has this framework do, as cases that can be timed and
compared: the fused training step over a whole gradient and per layer, the
Top-k selection on its own, and the weighted aggregation on its own, from
models of a few ten thousand parameters to the largest of the workloads.

Gradients are seeded synthetic values with the models' sizes and a scale of
its own for every layer (see ``workloads``), made on the GPU.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2301_08897_amd as sc

# Parameter counts of the workloads' models; the small ones are a LeNet-sized
# model and one 128 x 128 x 3 x 3 layer.
LENET, CONV, MILLION = 61_706, 147_456, 1_048_576
RESNET18, RESNET50, RESNET152, VGG19 = 11_173_962, 25_557_032, 60_192_808, 143_667_240

STEP = {"call": "step", "ratio": 0.01, "ratio_b": 0.0, "layout": "conv", "layers": 62, "values": "normal",
        "per_layer": False, "optimizer": "sgd", "adaptive": False}


def listed():
    return [
        # A small model on four devices: below the size the sampled selection
        # starts at, where the launches and not the bytes are the cost.
        dict(STEP, name="step_lenet", K=4, n=LENET, ratio=0.1, layout="even", layers=8),
        # One layer's gradient, compressed on its own in a training hook.
        dict(STEP, name="select_conv", call="select", K=1, n=CONV, layout="even", layers=1, optimizer="none"),
        # The smallest workload of the benchmark: every launch is short.
        dict(STEP, name="step_1m", K=4, n=MILLION, layout="even", layers=8),
        # ResNet-18 on 8 devices, the ordinary training step.
        dict(STEP, name="step_resnet18", K=8, n=RESNET18),
        # The paper's own compression ratio (0.1): ten times as many kept
        # entries, heavy-tailed values.
        dict(STEP, name="step_resnet50_cr0.1", K=16, n=RESNET50, ratio=0.1, layers=161, values="laplace"),
        # The adaptive rule at work: half of the devices compress harder than
        # the threshold allows and send their dense gradients; moving averages
        # and accounting on.
        dict(STEP, name="step_resnet50_adaptive", K=16, n=RESNET50, ratio=0.1, ratio_b=0.001, layers=161,
             values="laplace", adaptive=True),
        # ResNet-152 with zeros and tied magnitudes, momentum SGD with weight
        # decay as in the paper's evaluation.
        dict(STEP, name="step_resnet152_momentum", K=16, n=RESNET152, ratio=0.001, layers=467, values="ties",
             optimizer="momentum"),
        # The largest model on nearly as many devices as the benchmark's
        # largest workload: bandwidth.
        dict(STEP, name="step_vgg19", K=30, n=VGG19, layout="vgg", layers=38),
        # Per-layer Top-k of a model of many short layers, the sets handed on
        # (to a wire, say) rather than aggregated here.
        dict(STEP, name="layers_resnet18", call="select", per_layer=True, K=8, n=RESNET18, optimizer="none"),
        # The per-layer training step of a model with five long layers and
        # many short ones.
        dict(STEP, name="layers_vgg19", per_layer=True, K=16, n=VGG19, layout="vgg", layers=38),
        # One device's whole gradient, without allocation (under capture, in
        # a serving loop).
        dict(STEP, name="select_vgg19", call="select_noalloc", K=1, n=VGG19, layout="vgg", layers=38,
             optimizer="none"),
        # Sets received from other machines: 14 compressed ones and two
        # devices that sent everything.
        dict(STEP, name="aggregate_resnet152", call="aggregate", K=16, n=RESNET152, layers=467, optimizer="none"),
    ]


def draw(rng):
    call = rng.choice(["step", "step", "step", "step", "select", "select", "select_noalloc", "aggregate"])
    n = int(math.exp(rng.uniform(math.log(LENET), math.log(VGG19))))
    if rng.random() < 0.5:
        n |= 1
    K = 1 if call == "select_noalloc" else rng.randint(1, 16)
    ratio = round(math.exp(rng.uniform(math.log(0.001), math.log(0.1))), 5)
    if call == "select_noalloc":
        n, ratio = min(n, 60_000_000 + rng.randint(0, 9999)), min(ratio, 0.01)
    layout = rng.choice(["conv", "vgg", "even"])
    c = dict(STEP, call=call, K=K, n=n, ratio=ratio, layout=layout,
             layers=max(4, min(rng.choice([8, 38, 62, 161, 467]), n // 4096)),
             values=rng.choice(["normal", "laplace", "ties"]), optimizer="none")
    c["per_layer"] = call in ("step", "select") and rng.random() < 0.4
    if call == "select" and not c["per_layer"]:
        c["K"] = 1
    if call == "step":
        c["optimizer"] = rng.choice(["none", "sgd", "sgd", "momentum"])
        if rng.random() < 0.3:
            c.update(adaptive=True, ratio_b=0.001)
    return c


# ---- inputs -----------------------------------------------------------------------------------

MOMENTUM, WEIGHT_DECAY, DELTA, BETA = 0.9, 5e-4, 0.3, 0.9


def layout(case):
    """Layer bounds [0, ..., n] and every layer's standard deviation (the model's
    own: the same for every device and seed)."""
    n, L = case["n"], case["layers"]
    r = np.random.RandomState(1000 + L)
    if case["layout"] == "even":
        w = np.ones(L)
    else:
        w = np.exp(r.uniform(math.log(64.0), math.log(2.4e6), L))
        if case["layout"] == "vgg":            # three layers hold 85% of the parameters
            w = w / w[:-3].sum() * 0.15
            w[-3:] = 0.85 * r.dirichlet(np.ones(3))
    b = np.round(np.cumsum(w) / w.sum() * n).astype(np.int64)
    for l in range(L):                         # no layer empty
        b[l] = max(b[l], l + 1)
    b[-1] = n
    for l in range(L - 2, -1, -1):
        b[l] = min(b[l], b[l + 1] - 1)
    lo = {"even": -4.0, "conv": -5.0, "vgg": -6.0}[case["layout"]]
    return [0] + [int(x) for x in b], 10.0 ** r.uniform(lo, -1.0, L)


def ratios(case):
    b = case["ratio_b"] or case["ratio"]
    return [case["ratio"] if j % 2 == 0 else b for j in range(case["K"])]


def gradients(case, seed, bounds, sigma):
    """[K, n] float32 gradients."""
    K, n = case["K"], case["n"]
    g = torch.Generator(device="cuda").manual_seed(seed * 7919 + 13)
    grads = torch.empty(K, n, dtype=torch.float32, device="cuda")
    scale = torch.repeat_interleave(torch.tensor(sigma, dtype=torch.float32, device="cuda"),
                                    torch.tensor(np.diff(bounds), device="cuda"))
    for j in range(K):
        x = grads[j]
        if case["values"] == "laplace":
            x.uniform_(-1.0, 1.0, generator=g)
            x.copy_(torch.sign(x) * torch.log1p(-x.abs().clamp(max=1.0 - 2.0**-24)) * -0.70710678)
        else:
            x.normal_(generator=g)
        x.mul_(scale)
        if case["values"] == "ties":
            # 5% zeros of either sign; 1% ties at a magnitude inside the kept set
            k = sc.topk_k(n, ratios(case)[j])
            u = torch.empty(n, dtype=torch.float32, device="cuda").uniform_(generator=g)
            m = torch.topk(x.abs(), (k + 1) // 2, sorted=False).values.min()
            x.copy_(torch.where(u < 0.05, x * 0.0, torch.where(u > 0.99, torch.sign(x) * m, x)))
    return grads


def sparse_sets(case, seed, bounds, sigma):
    """Sets as other machines send them: the entries above a magnitude that keeps
    about ratio of them, ascending; every eighth device the whole gradient."""
    grads = gradients(case, seed, bounds, sigma)
    sets = []
    for j in range(case["K"]):
        x = grads[j]
        if j % 8 == 7:
            sets.append((None, x.clone()))
            continue
        k = max(1, int(case["ratio"] * case["n"]))
        t = torch.topk(x.abs(), k, sorted=False).values.min()
        i = (x.abs() >= t).nonzero().flatten()
        sets.append((i.to(torch.int32), x[i].contiguous()))
    return sets


def weights_of(case, seed):
    """Eqn 4a weights and the scaled learning rate from streaming rates."""
    K = case["K"]
    rates = 1.0 + np.random.RandomState(seed % (1 << 31)).poisson(4.0 * 128.0 ** (np.arange(K) / max(K - 1, 1)))
    w, gamma = sc.stream_weights(rates, base_batch=64.0 * K)
    return w, 0.01 * gamma


def params_of(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed * 7919 + 17)
    return torch.empty(case["n"], dtype=torch.float32, device="cuda").normal_(0.0, 0.05, generator=g)


# ---- one pass -----------------------------------------------------------------------------------

def prepare(case, seed):
    bounds, sigma = layout(case)
    s = {"case": case, "call": case["call"]}
    if case["call"] == "aggregate":
        s["sets"] = sparse_sets(case, seed, bounds, sigma)
        s["weights"] = weights_of(case, seed)[0]
        s["out"] = torch.empty(case["n"], dtype=torch.float32, device="cuda")
        s["ws"] = torch.empty(sc.aggregate_workspace_bytes(case["K"], case["n"]), dtype=torch.uint8, device="cuda")
        return s
    grads = gradients(case, seed, bounds, sigma)
    if case["call"] == "step":
        s["weights"], s["lr"] = weights_of(case, seed)
        more = {}
        if case["optimizer"] != "none":
            more["params"] = params_of(case, seed)
        if case["optimizer"] == "momentum":
            more.update(momentum_buf=torch.zeros(case["n"], dtype=torch.float32, device="cuda"), momentum=MOMENTUM,
                        weight_decay=WEIGHT_DECAY)
        if case["adaptive"]:
            more.update(delta=DELTA, ewma_beta=BETA, track=True)
        if case["per_layer"]:
            more["seg_off"] = bounds
        f = s["step"] = sc.FusedStep(grads, ratios(case), **more)
        s["outputs"] = {"idx": [t.view(torch.int32) for t in f.idx], "val": f.val, "dense": f.dense,
                        "energies": f.energies, "compressed": f.compressed, "params": f.params,
                        "momentum": f.momentum_buf, "ewma": f.ewma, "counters": f.counters}
    elif case["per_layer"]:
        f = s["layers"] = sc.LayerSelect(grads, bounds, ratios(case))
        s["outputs"] = {"idx": [t.view(torch.int32) for t in f.idx], "val": f.val, "energies": f.energies}
    else:
        n, r = case["n"], case["ratio"]
        s["grad"], s["ratio"] = grads[0], r
        if case["call"] == "select_noalloc":
            k = sc.topk_k(n, r)
            s["idx"] = torch.empty(k, dtype=torch.int32, device="cuda")
            s["val"] = torch.empty(k, dtype=torch.float32, device="cuda")
            s["energies"] = torch.empty(2, dtype=torch.float64, device="cuda")
        else:
            s["ws"] = torch.empty(sc.workspace_bytes(1, n, [r]), dtype=torch.uint8, device="cuda")
    return s


def run(s):
    if s["call"] == "aggregate":
        return sc.weighted_aggregate(s["sets"], s["weights"], s["case"]["n"], out=s["out"], workspace=s["ws"])
    if s["call"] == "step":
        s["step"].run(s["weights"], s["lr"])
        return s["outputs"]
    if "layers" in s:
        s["layers"].run()
        return s["outputs"]
    if s["call"] == "select_noalloc":
        return sc.topk_select_noalloc(s["grad"], s["ratio"], s["idx"], s["val"], s["energies"])
    idx, val, en = sc.topk_select(s["grad"], s["ratio"], workspace=s["ws"], energies=True)
    return idx.view(torch.int32), val, en


# ---- what a pass cannot do without, and what it gives ---------------------------------------------

def kept(case):
    if case["per_layer"]:
        bounds = layout(case)[0]
        return [sc.layers_k(bounds, r) for r in ratios(case)]
    return [sc.topk_k(case["n"], r) for r in ratios(case)]


def work(case):
    """Bytes: every gradient (or set) read once, the kept pairs, the aggregate and
    the updated state written once. Operations: the energies' squares and the
    weighted terms, two each."""
    K, n = case["K"], case["n"]
    if case["call"] == "aggregate":
        k = max(1, int(case["ratio"] * n))
        dense = K // 8
        return {"bytes": 8 * k * (K - dense) + 4 * n * dense + 4 * n, "flops": 2 * (k * (K - dense) + n * dense)}
    ks = sum(kept(case))
    b, f = 4 * K * n + 8 * ks, 2 * K * n + 2 * ks
    if case["call"] == "step":
        b += 4 * n + {"none": 0, "sgd": 8 * n, "momentum": 16 * n}[case["optimizer"]]
        f += 2 * ks + {"none": 0, "sgd": 2 * n, "momentum": 6 * n}[case["optimizer"]]
    return {"bytes": b, "flops": f}


def tolerance(case):
    """Indices, values, aggregate and update are defined bit for bit (integer
    ranking; double sums in device order, rounded once); only the energies are
    double sums whose order is free: 1e-14 relative between two orders at the
    largest sizes here, a few times that stated."""
    return {"rel": 1e-12, "max": 1e-12, "differ": 0.0}


def _topk(x, k):
    """Positions of the k largest magnitudes, ties to the lower index, ascending."""
    mag = x.abs()
    t = torch.topk(mag, k, sorted=False).values.min()
    keep = mag > t
    need = k - int(keep.sum())
    eq = (mag == t).nonzero().flatten()[:need]
    keep[eq] = True
    return keep.nonzero().flatten()


def exact(case, seed):
    bounds, sigma = layout(case)
    n, K = case["n"], case["K"]
    if case["call"] == "aggregate":
        w = weights_of(case, seed)[0]
        out = torch.zeros(n, dtype=torch.float64, device="cuda")
        for wj, (i, v) in zip(w, sparse_sets(case, seed, bounds, sigma)):
            if i is None:
                out += float(wj) * v.double()
            else:
                out[i.long()] += float(wj) * v.double()
        return out
    grads = gradients(case, seed, bounds, sigma)
    idx, val, en, sent = [], [], [], []
    rs = ratios(case)
    for j in range(K):
        x = grads[j]
        if case["per_layer"]:
            i = torch.cat([_topk(x[a:b], sc.topk_k(b - a, rs[j])) + a for a, b in zip(bounds[:-1], bounds[1:])])
        else:
            i = _topk(x, sc.topk_k(n, rs[j]))
        idx.append(i.to(torch.int32))
        val.append(x[i].double())
        e_all = sum(float(c.double().square().sum()) for c in x.split(1 << 25))
        e_kept = float(val[-1].square().sum())
        en += [e_all, e_kept]
        rho = 0.0 if e_all == 0.0 else abs(e_all - e_kept) / e_all
        sent.append(1 if not case["adaptive"] or rho <= DELTA else 0)
    energies = torch.tensor(en, dtype=torch.float64, device="cuda")
    if case["call"] in ("select", "select_noalloc") and not case["per_layer"]:
        return idx[0], val[0], energies
    if case["call"] == "select":
        return {"idx": idx, "val": val, "energies": energies}
    w, lr = weights_of(case, seed)
    dense = torch.zeros(n, dtype=torch.float64, device="cuda")
    for j in range(K):
        if sent[j]:
            dense[idx[j].long()] += float(w[j]) * val[j]
        else:
            dense += float(w[j]) * grads[j].double()
    del grads
    out = {"idx": idx, "val": val, "dense": dense, "energies": energies, "compressed": None, "params": None,
           "momentum": None, "ewma": energies if case["adaptive"] else None, "counters": None}
    lr = float(np.float32(lr))
    if case["optimizer"] != "none":
        p = params_of(case, seed).double()
        if case["optimizer"] == "momentum":
            out["momentum"] = dense + float(np.float32(WEIGHT_DECAY)) * p
            out["params"] = p - lr * out["momentum"]
        else:
            out["params"] = p - lr * dense
    return out
