"""The work a program has the batched LSGD step do, as a list of cases to time and to compare.

A case is a dict of plain values.  `path` says which part of the library it goes through:

  update   gradients and losses come from the caller: one step is leader selection + pull update
  easgd    the same with the elastic-averaging update
  mc       low-rank matrix completion: one whole step (gradient, selection, update) or one iteration of Algorithm 1
  mlp      fully connected classifier: one whole step, a separate gradient call, or an objective evaluation

`prepare` draws the inputs from the seed on the GPU and builds the population a program keeps; `run` makes one
pass through the public binding; `exact` is the same pass in plain torch at 64 bits, with the rounding points
of the library's contract (MLP matrix operands are bf16) and nothing else rounded.
"""
import math

import torch

import paper_1905_10395_amd as L

DEV = "cuda:0"


def _ld(P):
    """Row stride a program uses: rows padded to 256 bytes."""
    return (P + 63) // 64 * 64


def _mlp_dims(case):
    return [int(v) for v in case["dims"].split("-")]


def _mlp_params(dims):
    return sum(dims[k + 1] * dims[k] + dims[k + 1] for k in range(len(dims) - 1))


def _params(case):
    if case["path"] == "mc":
        return (case["m"] + case["n"]) * case["r"]
    if case["path"] == "mlp":
        return _mlp_params(_mlp_dims(case))
    return case["P"]


# ------------------------------------------------------------------------------------------------
# the listed cases
# ------------------------------------------------------------------------------------------------
def listed():
    return [
        # a toy objective optimised by four workers: the cost of a step is its launches
        {"name": "update_tiny", "path": "update", "W": 4, "G": 1, "P": 1003, "momentum": 0.0, "nesterov": False, "wd": 0.0,
         "keep": False},
        # a small conv net's parameter vector, 12 workers in 3 groups, Nesterov and weight decay, in the middle of a
        # communication period: one group re-selects, the others and the global leader are the kept copies
        {"name": "update_kept_leaders", "path": "update", "W": 12, "G": 3, "P": 271_117, "momentum": 0.9, "nesterov": True,
         "wd": 1e-4, "keep": True},
        # the update stress: 32 workers of 11.7 M parameters, every leader re-selected
        {"name": "update_stress", "path": "update", "W": 32, "G": 4, "P": 11_689_512, "momentum": 0.9, "nesterov": False,
         "wd": 0.0, "keep": False},
        # the paper's comparison method on a medium population
        {"name": "easgd_medium", "path": "easgd", "W": 16, "G": 4, "P": 1_280_000, "momentum": 0.9, "nesterov": False, "wd": 0.0},
        # tiny matrix completion, batch gradient on all observed entries
        {"name": "mc_tiny_full_batch", "path": "mc", "call": "step", "m": 100, "n": 100, "r": 5, "n_obs": 3000, "B": 0,
         "W": 4, "G": 1, "packed": False},
        # matrix completion at scale, sampled batches, packed entry records, leaders re-selected at this step
        {"name": "mc_step_rank32", "path": "mc", "call": "step", "m": 20000, "n": 20000, "r": 32, "n_obs": 4_000_000,
         "B": 65536, "W": 16, "G": 4, "packed": True},
        # Algorithm 1's schedule on a rectangular problem of a rank that is no multiple of four, separate entry arrays,
        # an iteration that communicates
        {"name": "mc_alg1_rank10", "path": "mc", "call": "alg1", "m": 6001, "n": 3517, "r": 10, "n_obs": 1_000_003,
         "B": 16384, "W": 8, "G": 2, "packed": False},
        # two-layer classifier, update inside the backward pass, batch 128
        {"name": "mlp_2layer_fused", "path": "mlp", "call": "step", "dims": "3072-1024-10", "W": 16, "G": 4, "B": 128,
         "fused": True, "keep": False, "fp32_in": False},
        # four-layer classifier of hidden width 4096, update inside the backward pass, a step on which leaders are kept
        {"name": "mlp_4layer_fused", "path": "mlp", "call": "step", "dims": "3072-4096-4096-4096-10", "W": 8, "G": 2, "B": 256,
         "fused": True, "keep": True, "fp32_in": False},
        # a small classifier of sizes that are no multiples of anything, fp32 inputs, gradient through memory
        {"name": "mlp_ragged_step", "path": "mlp", "call": "step", "dims": "784-300-100-10", "W": 8, "G": 2, "B": 50,
         "fused": False, "keep": False, "fp32_in": True},
        # gradients for a program with an update of its own, batch 32 per worker
        {"name": "mlp_grad_batch32", "path": "mlp", "call": "grad", "dims": "3072-1024-512-10", "W": 16, "G": 4, "B": 32,
         "fused": False, "keep": False, "fp32_in": False},
        # objective evaluation on a larger sample (what choosing a leader costs): forward pass only
        {"name": "mlp_eval_loss", "path": "mlp", "call": "loss", "dims": "3072-1024-10", "W": 16, "G": 4, "B": 500,
         "fused": False, "keep": False, "fp32_in": False},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above: workers 2-32, groups that divide them, sizes over their logarithm."""
    G = rng.choice([1, 2, 3, 4])
    W = G * rng.randint(max(1, 2 // G), 8)
    path = rng.choice(["update", "update", "easgd", "mc", "mc", "mlp", "mlp", "mlp"])
    if path in ("update", "easgd"):
        case = {"path": path, "W": W, "G": G, "P": _log_int(rng, 500, 11_000_000),
                "momentum": rng.choice([0.0, 0.9]), "nesterov": False, "wd": rng.choice([0.0, 1e-4])}
        if path == "update":
            case["nesterov"] = case["momentum"] > 0 and rng.random() < 0.5
            case["keep"] = rng.random() < 0.5
        return case
    if path == "mc":
        r = rng.choice([1, 2, 3, 4, 5, 8, 10, 12, 16, 20, 32, 50, 64])
        m, n = _log_int(rng, 80, 20000), _log_int(rng, 80, 20000)
        n_obs = min(m * n, _log_int(rng, 2000, 4_000_000))
        full = n_obs <= 20000 and rng.random() < 0.5
        return {"path": "mc", "call": rng.choice(["step", "alg1"]), "m": m, "n": n, "r": r, "n_obs": n_obs,
                "B": 0 if full else _log_int(rng, 256, 65536), "W": min(W, 16), "G": 1 if W > 16 else G, "packed": rng.random() < 0.5}
    layers = rng.choice([1, 2, 2, 3])
    hidden = [_log_int(rng, 40, 2048) for _ in range(layers)]
    if rng.random() < 0.4:                       # round widths are common too
        hidden = [max(64, (h + 63) // 64 * 64) for h in hidden]
    d0 = rng.choice([3072, 784, 256, 617, 100])
    C = rng.choice([10, 10, 2, 7, 100])
    B = rng.choice([16, 32, 50, 64, 100, 128, 200, 256])
    call = rng.choice(["step", "step", "grad", "loss"])
    return {"path": "mlp", "call": call, "dims": "-".join(str(v) for v in [d0] + hidden + [C]), "W": min(W, 16), "G": 1 if W > 16 else G,
            "B": B, "fused": call == "step" and rng.random() < 0.5, "keep": call == "step" and rng.random() < 0.5,
            "fp32_in": rng.random() < 0.3}


# ------------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(1_000_003 * int(seed) + 17)
    return g


def _rows(W, P, gen, std):
    t = torch.zeros((W, _ld(P)), device=DEV)
    t[:, :P].normal_(std=std, generator=gen)
    return t


def _inputs(case, seed):
    """Everything drawn from the seed, on the GPU."""
    gen = _gen(seed)
    W, P = case["W"], _params(case)
    d = {}
    if case["path"] in ("update", "easgd"):
        d["x"] = _rows(W, P, gen, 0.05)
        d["g"] = _rows(W, P, gen, 1e-2)
        d["m"] = _rows(W, P, gen, 3e-2) if case["momentum"] else None
        d["losses0"] = torch.rand(W, device=DEV, generator=gen)      # selected the kept leaders
        d["losses"] = torch.rand(W, device=DEV, generator=gen)
        if case["path"] == "easgd":
            d["center"] = torch.zeros(_ld(P), device=DEV)
            d["center"][:P].normal_(std=0.05, generator=gen)
        return d
    if case["path"] == "mc":
        m, n, r = case["m"], case["n"], case["r"]
        std = r ** -0.25                                              # entries of U V^T of order one
        U = torch.empty((m, r), device=DEV).normal_(std=std, generator=gen)
        V = torch.empty((n, r), device=DEV).normal_(std=std, generator=gen)
        flat = torch.randint(0, m * n, (case["n_obs"],), device=DEV, generator=gen)
        rows, cols = flat // n, flat % n
        noise = torch.empty(case["n_obs"], device=DEV).normal_(std=0.01, generator=gen)
        d["vals"] = (U[rows] * V[cols]).sum(1) + noise
        d["rows"], d["cols"] = rows.to(torch.int32), cols.to(torch.int32)
        d["idx"] = (torch.randint(0, case["n_obs"], (W, case["B"]), device=DEV, generator=gen, dtype=torch.int32)
                    if case["B"] else None)
        d["x"] = _rows(W, P, gen, std)
        return d
    dims, B = _mlp_dims(case), case["B"]
    means = torch.empty((dims[-1], dims[0]), device=DEV).normal_(generator=gen)
    y = torch.randint(0, dims[-1], (W, B), device=DEV, generator=gen, dtype=torch.int32)
    X = means[y.long()] + torch.empty((W, B, dims[0]), device=DEV).normal_(generator=gen)
    d["X"], d["y"] = (X if case["fp32_in"] else X.to(torch.bfloat16)), y
    x = torch.zeros((W, _ld(P)), device=DEV)
    o = 0
    for k in range(len(dims) - 1):
        fin, fout = dims[k], dims[k + 1]
        x[:, o:o + fin * fout].uniform_(-fin ** -0.5, fin ** -0.5, generator=gen)
        o += fin * fout
        x[:, o:o + fout].normal_(std=0.01, generator=gen)
        o += fout
    d["x"] = x
    d["m"] = _rows(W, P, gen, 1e-3) if case["call"] == "step" else None
    d["losses0"] = torch.rand(W, device=DEV, generator=gen)
    return d


def _mc_c(case):
    return 0.5 * case["n_obs"] / case["B"] if case["B"] else 0.5


def _eta(case):
    if case["path"] != "mc":
        return 0.01
    # a step length at which a batch of this size neither diverges nor stalls: curvature of a factor row is
    # 2 c |V|^2 per entry of the batch in that row
    nb = case["B"] or case["n_obs"]
    return 0.2 / (2 * _mc_c(case) * math.sqrt(case["r"]) * (1 + 4 * nb / min(case["m"], case["n"])))


# coefficients: those of the configurations
LAM_L, LAM_G = 0.1, 0.05
GAM_L, GAM_G = 0.025, 0.0125


def prepare(case, seed):
    d = _inputs(case, seed)
    W, G, P = case["W"], case["G"], _params(case)
    s = {"case": case, "in": d}
    Z = torch.zeros((G + 1, _ld(P)), device=DEV)
    if case["path"] in ("update", "easgd"):
        keep = bool(case.get("keep"))
        needs_z = keep or case["path"] == "easgd"
        flags = L.NESTEROV if case["nesterov"] else 0
        pop = L.Population(d["x"], d["g"], G, m=d["m"], z_snapshot=Z if needs_z else None, P=P, momentum=case["momentum"],
                           flags=flags, weight_decay=case["wd"])
        s["batch"] = L.ExternalBatch(d["losses"])
        if keep:
            pop.select_leaders(d["losses0"])
            pop.leader_pull(0.0, 0.0)                                 # takes the leader copies, moves nobody
        s["mask"], s["glob"] = ([1] + [0] * (G - 1), 0) if keep else (None, 1)
        s["Z"] = Z if keep else None
    elif case["path"] == "mc":
        d["g"] = torch.zeros_like(d["x"])
        entries = L.mc_pack_entries(d["rows"], d["cols"], d["vals"]) if case["packed"] else None
        s["batch"] = L.MCBatch(case["m"], case["n"], case["r"], d["rows"], d["cols"], d["vals"], d["idx"], _mc_c(case), entries=entries)
        pop = L.Population(d["x"], d["g"], G, z_snapshot=Z, P=P, largest_batch=s["batch"])
        if case["call"] == "alg1":                                    # the initialisation block of Algorithm 1
            pop.grad_loss(s["batch"])
            pop.select_leaders()
            pop.leader_pull(0.0, 0.0)
        s["Z"] = Z
    else:
        d["g"] = torch.zeros_like(d["x"])
        xb = torch.zeros((W, _ld(P)), dtype=torch.bfloat16, device=DEV)
        s["batch"] = L.MLPBatch(_mlp_dims(case), d["X"], d["y"])
        step = case["call"] == "step"
        pop = L.Population(d["x"], d["g"], G, m=d["m"], z_snapshot=Z if step else None, x_bf16=xb, P=P,
                           momentum=0.9 if step else 0.0, largest_batch=s["batch"],
                           flags=L.WRITE_BF16_SHADOW | (L.FUSED_MLP_UPDATE if case["fused"] else 0))
        if case["keep"]:
            pop.select_leaders(d["losses0"])
            pop.leader_pull(0.0, 0.0)
        pop.sync_shadow()                                             # as after any earlier step
        s["mask"], s["glob"] = ([0] * G, 0) if case["keep"] else (None, 1)
        s["xb"], s["Z"] = xb, Z
        s["losses"] = torch.zeros(W, device=DEV)
    s["pop"] = pop
    return s


def run(s):
    case, d, pop = s["case"], s["in"], s["pop"]
    eta = _eta(case)
    if case["path"] == "update":
        pop.step(s["batch"], eta, LAM_L, LAM_G, s["mask"], s["glob"])
        return {"x": d["x"], "m": d["m"], "Z": s["Z"]}
    if case["path"] == "easgd":
        pop.easgd_step(s["batch"], d["center"], eta, LAM_L)
        return {"x": d["x"], "m": d["m"], "center": d["center"]}
    if case["path"] == "mc":
        if case["call"] == "step":
            pop.step(s["batch"], eta, LAM_L, LAM_G)
        else:
            pop.step_alg1(s["batch"], eta, GAM_L, GAM_G, LAM_L, LAM_G, L.COMM_LOCAL | L.COMM_GLOBAL)
        return {"x": d["x"], "g": d["g"], "Z": s["Z"]}
    if case["call"] == "step":
        pop.step(s["batch"], eta, LAM_L, LAM_G, s["mask"], s["glob"])
        return {"x": d["x"], "m": d["m"], "xb": s["xb"], "Z": s["Z"], "g": None if case["fused"] else d["g"]}
    if case["call"] == "grad":
        pop.grad_loss(s["batch"], s["losses"])
        return {"g": d["g"], "losses": s["losses"]}
    pop.loss(s["batch"], s["losses"])
    return {"losses": s["losses"]}


# ------------------------------------------------------------------------------------------------
# what one pass cannot do without, and what two correct implementations may differ by
# ------------------------------------------------------------------------------------------------
def work(case):
    W, G, P = case["W"], case["G"], _params(case)
    if case["path"] in ("update", "easgd"):
        per = 20 if case["momentum"] else 12                          # x, g (, m) read, x (, m) written
        extra = 8.0 * P if case["path"] == "easgd" else (4.0 * P * (G + 1) if case["keep"] else 0.0)
        return {"bytes": float(W) * P * per + extra, "flops": 10.0 * W * P}
    if case["path"] == "mc":
        nb = case["B"] or case["n_obs"]
        entry = 16.0 if case["B"] else 12.0                           # (index,) row, column, value
        extra = 4.0 * P * (G + 1) * (2 if case["call"] == "alg1" else 1)
        return {"bytes": W * (12.0 * P + (entry * nb if case["B"] else 0.0)) + (0.0 if case["B"] else entry * nb) + extra,
                "flops": 6.0 * W * nb * case["r"] + 8.0 * W * P}
    dims, B = _mlp_dims(case), case["B"]
    weights = sum(dims[k] * dims[k + 1] for k in range(len(dims) - 1))
    hidden = weights - dims[0] * dims[1]
    inp = W * B * (dims[0] * (4.0 if case["fp32_in"] else 2.0) + 4.0)
    if case["call"] == "loss":
        return {"bytes": 2.0 * W * P + inp, "flops": 2.0 * W * B * weights}
    flops = 2.0 * W * B * (2 * weights + hidden)
    if case["call"] == "grad":
        return {"bytes": 6.0 * W * P + inp, "flops": flops}           # bf16 weights read, fp32 gradient written
    per = 20.0 if case["fused"] else 24.0                             # bf16 copy, x, m read and written (gradient written)
    return {"bytes": per * W * P + inp + 4.0 * (G + 1) * P, "flops": flops}


def tolerance(case):
    if case["path"] in ("update", "easgd"):
        return {"rel": 1e-6, "max": 1e-5}
    if case["path"] == "mc":
        return {"rel": 1e-5, "max": 1e-4}
    if case["call"] == "loss":
        return {"rel": 1e-4}
    return {"rel": 2e-2, "max": 0.9}


# ------------------------------------------------------------------------------------------------
# the same pass in 64 bits
# ------------------------------------------------------------------------------------------------
def _leaders(losses, G):
    W = losses.numel()
    per = W // G
    v = losses.cpu().tolist()
    loc = [min(range(j * per, (j + 1) * per), key=lambda i: (v[i], i)) for j in range(G)]
    return loc, min(range(W), key=lambda i: (v[i], i))


def _bf(t):
    return t.to(torch.float32).to(torch.bfloat16).to(torch.float64)


def _exact_update(case, d, g_of, losses, kept_from, mask, glob, momentum, nesterov, wd, eta):
    """x, m and the leader copies after select + pull update; g_of(i): fp64 gradient of row i."""
    W, G, P = case["W"], case["G"], _params(case)
    x = d["x"]
    loc, gl = _leaders(losses, G)
    if kept_from is not None:
        kloc, kgl = _leaders(kept_from, G)
        loc = [loc[j] if mask[j] else kloc[j] for j in range(G)]
        gl = gl if glob else kgl
    xn = torch.zeros(x.shape, dtype=torch.float64, device=DEV)
    mn = torch.zeros(x.shape, dtype=torch.float64, device=DEV) if momentum else None
    for i in range(W):
        xi = x[i, :P].double()
        dd = g_of(i) + wd * xi + LAM_L * (xi - x[loc[i // (W // G)], :P].double()) + LAM_G * (xi - x[gl, :P].double())
        if momentum:
            mi = momentum * d["m"][i, :P].double() + dd
            mn[i, :P] = mi
            step = dd + momentum * mi if nesterov else mi
        else:
            step = dd
        xn[i, :P] = xi - eta * step
    Z = torch.cat([x[loc + [gl], :P].double(), torch.zeros((G + 1, x.shape[1] - P), dtype=torch.float64, device=DEV)], 1)
    return xn, mn, Z


def _exact_mc(case, d):
    W, m, n, r = case["W"], case["m"], case["n"], case["r"]
    c = _mc_c(case)
    g = torch.zeros(d["x"].shape, dtype=torch.float64, device=DEV)
    losses = torch.zeros(W, dtype=torch.float64, device=DEV)
    for i in range(W):
        at = d["idx"][i].long() if d["idx"] is not None else torch.arange(case["n_obs"], device=DEV)
        a, b, v = d["rows"][at].long(), d["cols"][at].long(), d["vals"][at].double()
        U = d["x"][i, :m * r].double().view(m, r)
        V = d["x"][i, m * r:(m + n) * r].double().view(n, r)
        e = (U[a] * V[b]).sum(1) - v
        losses[i] = c * (e * e).sum()
        g[i, :m * r].view(m, r).index_add_(0, a, (2 * c) * e[:, None] * V[b])
        g[i, m * r:(m + n) * r].view(n, r).index_add_(0, b, (2 * c) * e[:, None] * U[a])
    return g, losses


def _exact_mlp(case, d, backward=True):
    dims, B, W = _mlp_dims(case), case["B"], case["W"]
    n = len(dims) - 1
    g = torch.zeros(d["x"].shape, dtype=torch.float64, device=DEV) if backward else None
    losses = torch.zeros(W, dtype=torch.float64, device=DEV)
    for i in range(W):
        at, Ws, bs = 0, [], []
        for k in range(n):
            fin, fout = dims[k], dims[k + 1]
            Ws.append(_bf(d["x"][i, at:at + fin * fout]).view(fout, fin))
            at += fin * fout
            bs.append(d["x"][i, at:at + fout].double())
            at += fout
        h = [_bf(d["X"][i])]
        for k in range(n):
            z = h[k] @ Ws[k].t().contiguous() + bs[k]
            h.append(_bf(z.clamp(min=0)) if k + 1 < n else z)
        y = d["y"][i].long()
        losses[i] = (torch.logsumexp(h[n], 1) - h[n].gather(1, y[:, None])[:, 0]).mean()
        if not backward:
            continue
        delta = torch.softmax(h[n], 1)
        delta[torch.arange(B, device=DEV), y] -= 1
        delta = _bf(delta / B)
        end = _params(case)
        for k in range(n - 1, -1, -1):
            fin, fout = dims[k], dims[k + 1]
            g[i, end - fout:end] = delta.sum(0)
            end -= fout
            g[i, end - fin * fout:end] = (delta.t().contiguous() @ h[k]).reshape(-1)
            end -= fin * fout
            if k:
                delta = _bf((delta @ Ws[k]) * (h[k] != 0))
    return g, losses


def exact(case, seed):
    d = _inputs(case, seed)
    eta, G, P = _eta(case), case["G"], _params(case)
    if case["path"] == "update":
        keep = case["keep"]
        x, m, Z = _exact_update(case, d, lambda i: d["g"][i, :P].double(), d["losses"], d["losses0"] if keep else None,
                                [1] + [0] * (G - 1), 0, case["momentum"], case["nesterov"], case["wd"], eta)
        return {"x": x, "m": m, "Z": Z if keep else None}
    if case["path"] == "easgd":
        x, c, mu = d["x"], d["center"].double(), case["momentum"]
        a = case["W"] * eta * LAM_L
        mean = torch.zeros_like(c)
        xn = torch.zeros(x.shape, dtype=torch.float64, device=DEV)
        mn = torch.zeros(x.shape, dtype=torch.float64, device=DEV) if mu else None
        for i in range(case["W"]):
            xi = x[i].double()
            mean += xi
            step = d["g"][i].double() + case["wd"] * xi + LAM_L * (xi - c)
            if mu:
                step = mu * d["m"][i].double() + step
                mn[i] = step
            xn[i] = xi - eta * step
        return {"x": xn, "m": mn, "center": (1 - a) * c + a * mean / case["W"]}
    if case["path"] == "mc":
        g, losses = _exact_mc(case, d)
        if case["call"] == "step":
            x, _, Z = _exact_update(case, d, lambda i: g[i, :P], losses, None, None, 1, 0.0, False, 0.0, eta)
            return {"x": x, "g": g, "Z": Z}
        # the kept copies and the communication's leaders come from the same losses
        loc, gl = _leaders(losses, G)
        x = d["x"].double()
        own = [loc[i // (case["W"] // G)] for i in range(case["W"])]
        x = x - eta * g - GAM_L * (x - x[own]) - GAM_G * (x - x[gl])
        Z = x[loc + [gl]].clone()
        x, zg = x - LAM_L * (x - x[own]), x[gl].clone()
        return {"x": x - LAM_G * (x - zg), "g": g, "Z": Z}
    g, losses = _exact_mlp(case, d, backward=case["call"] != "loss")
    if case["call"] == "loss":
        return {"losses": losses}
    if case["call"] == "grad":
        return {"g": g, "losses": losses}
    x, m, Z = _exact_update(case, d, lambda i: g[i, :P], losses, d["losses0"] if case["keep"] else None, [0] * G, 0,
                            0.9, False, 0.0, eta)
    return {"x": x, "m": m, "xb": None, "Z": Z, "g": None if case["fused"] else g}
