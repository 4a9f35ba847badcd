"""The work whose speed this repository is measured by: training steps of the sparse path, lookups for serving, table
maintenance, the first fully-connected layer, the cross network and a whole model step, each through the calls of
``des.py`` / ``model.py`` as a user's program makes them.

Sizes follow the five workloads of ``synth.py`` (the largest one with a smaller table, so that several fit the card) and
the tower the model tests use; IDs follow a Zipf law over the resident rows, optionally mixed with uniform draws and
with IDs the table has not seen.  Tables look trained: weights are drawn from a seeded normal law and the
optimizer state is that of a table some tens of steps old, so that an update is well conditioned, as it is in a run.
All inputs are made on the GPU from the seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1909_04823_amd import des, model, synth

LR, EPS = 0.05, 1e-8
ADAM = dict(beta1=0.9, beta2=0.999, step=10)
FTRL = dict(ftrl_alpha=0.05, ftrl_beta=1.0, ftrl_l1=1e-4, ftrl_l2=1e-3)
INIT_SCALE = 0.01
CHUNK = 1 << 23                      # entries per piece of the 64-bit evaluation
HEAD = 1 << 16                       # ranks whose popularity is tabulated exactly; the tail uses the inverse of the integral
BF_D_MAX = 131072 * 200 * 64         # pooled floats of the largest listed case
ENTRY_D_MAX = 131072 * 200 * 4 * 64  # gathered floats of the largest listed case


# ---------------------------------------------------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------------------------------------------------
def _step(name, B, F, D, K, opt, rows, bag, a, **more):
    """One training step of the sparse path: find -> forward -> aggregation -> backward with the row update."""
    return dict({"name": name, "kind": "step", "B": B, "F": F, "D": D, "K": K, "opt": opt, "rows": rows, "bag": bag, "zipf": a,
                 "uniform": 0.0, "new": 0.0, "min_bag": 1, "vals": False, "policy": "key"}, **more)


def listed():
    return [
        # a small online-learning step: ten one-valued fields, one entry each; launches and latency are everything
        _step("step_tiny", 256, 10, 8, 2, "sgd", 10_000, 0.0, 0.0),
        # Criteo-shaped pooled fields with Adagrad latent vectors and FTRL first-order weights, a few unseen IDs
        _step("step_pooled", 4096, 26, 16, 8, "adagrad_ftrl", 1_000_000, 9.5, 1.1, new=0.05),
        # an odd-sized batch with feature values, missing fields and the field partition, Adam
        _step("step_values_odd", 3001, 37, 32, 5, "adam", 700_001, 3.3, 1.15, new=0.02, min_bag=0, vals=True, policy="field"),
        # DeepFM-shaped: many fields, strongly skewed popularity
        _step("step_deepfm", 16384, 100, 32, 16, "adagrad", 20_000_000, 5.0, 1.2, new=0.01),
        # a streaming recommender's step: long vectors, many workers
        _step("step_streaming", 65536, 40, 64, 32, "adagrad", 8_000_000, 3.0, 1.1, new=0.03),
        # the largest step: half of the IDs uniform over a table far larger than the caches
        _step("step_large", 131072, 200, 64, 64, "adagrad", 60_000_000, 4.0, 1.05, uniform=0.5),
        # scoring one small request against a resident table (forward only, unknown IDs read as absent)
        {"name": "serve_request", "kind": "serve", "B": 48, "F": 26, "D": 16, "K": 8, "rows": 1_000_000, "bag": 5.0, "zipf": 1.1,
         "uniform": 0.0, "new": 0.05, "min_bag": 1, "vals": False, "policy": "key"},
        # a batch with a third of unseen IDs enters the table and the newcomers are evicted again
        {"name": "insert_evict", "kind": "evict", "n": 4_000_001, "D": 32, "rows": 4_000_000, "zipf": 1.1, "uniform": 0.0, "new": 0.3},
        # first fully-connected layer, forward and backward, at the DeepFM-shaped size
        {"name": "layer", "kind": "layer", "B": 16384, "F": 100, "D": 32, "H": 256, "K": 16},
        # the same with a ragged batch, width and field count
        {"name": "layer_odd", "kind": "layer", "B": 5003, "F": 27, "D": 20, "H": 300, "K": 7},
        # the cross network of a DCN model, two layers and the output term, forward and backward
        {"name": "cross_network", "kind": "cross", "B": 32768, "F": 100, "D": 32, "K": 16, "layers": 2},
        # a whole DeepFM training step, lookup to dense update
        {"name": "model_deepfm", "kind": "model", "model": "deepfm", "B": 4096, "F": 26, "D": 16, "K": 8, "H1": 256, "H2": 128,
         "rows": 1_000_000, "bag": 5.0, "zipf": 1.1, "uniform": 0.0, "new": 0.0, "min_bag": 1, "vals": False, "policy": "key"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step"] * 6 + ["serve"] * 2 + ["evict"] + ["layer"] * 3 + ["cross"] * 2 + ["model"] * 2)
    D = rng.choice([4, 8, 16, 32, 64, 128])
    if kind == "layer":
        while True:
            c = {"kind": kind, "B": _log(rng, 64, 131072), "F": _log(rng, 2, 200), "D": 4 * _log(rng, 1, 16),
                 "H": 4 * _log(rng, 4, 128), "K": rng.choice([1, 2, 3, 8, 16, 64])}
            if c["K"] * c["B"] * c["H"] <= 1 << 30 and c["B"] * c["F"] * c["D"] * c["H"] <= 1 << 37:
                return c
    if kind == "cross":
        while True:
            c = {"kind": kind, "B": _log(rng, 64, 131072), "F": _log(rng, 2, 200), "D": rng.choice([4, 8, 12, 16, 32, 64]),
                 "K": rng.choice([1, 2, 5, 16, 64]), "layers": rng.randint(1, 4)}
            if c["B"] * c["F"] * c["D"] <= BF_D_MAX // 4:
                return c
    ids = {"rows": _log(rng, 10_000, 16_000_000), "zipf": round(rng.uniform(1.02, 1.3), 3), "uniform": rng.choice([0.0, 0.0, 0.5])}
    if kind == "evict":
        return dict(ids, kind=kind, n=_log(rng, 1000, 6_000_000), D=min(D, 64), new=round(rng.uniform(0.02, 0.5), 3))
    while True:
        B, F = _log(rng, 16, 131072), _log(rng, 1, 200)
        bag, K = round(rng.uniform(1.0, 8.0), 2), rng.choice([1, 2, 3, 8, 16, 32, 64])
        if kind == "serve":
            B = min(B, 4096)
        if K * (D + 2) * 8 + (F + 1) * 4 + 4096 > 65536 or B * F * bag * D > ENTRY_D_MAX / 8 or B * F * bag > 16_000_000 or K * B * D > 1 << 28:
            continue
        c = dict(ids, kind=kind, B=B, F=F, D=D, K=K, bag=bag, min_bag=rng.choice([0, 1]), policy=rng.choice(["key", "key", "field"]),
                 vals=rng.random() < 0.3, new=round(rng.choice([0.0, 0.0, rng.uniform(0.005, 0.1)]), 4))
        if kind == "step":
            c["opt"] = rng.choice(["sgd", "adagrad", "adagrad", "adagrad_ftrl", "adam"])
        if kind == "model":
            if B < 64 or B * F * D * 256 > 1 << 36:
                continue
            c.update(model=rng.choice(["lr", "fm", "wd", "deepfm", "deepfm", "dcn"]), H1=4 * _log(rng, 8, 64), H2=4 * _log(rng, 4, 32), new=0.0)
        return c


# ---------------------------------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------------------------------
def _gen(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1_000_003 + salt) & 0x7FFFFFFFFFFFFFFF)
    return g


def _rand(g, *shape, dtype=torch.float32):
    return torch.rand(shape, generator=g, device="cuda", dtype=dtype)


def _randn(g, *shape):
    return torch.randn(shape, generator=g, device="cuda")


def _ids(ranks):
    """63-bit feature IDs of popularity ranks (a bijection, so distinct ranks are distinct IDs)."""
    m = (1 << 63) - 1
    x = (ranks * (0xD1342543DE82EF95 - (1 << 64))) & m
    x = x ^ (x >> 31)
    x = (x * (0xA0761D6478BD642F - (1 << 64))) & m
    return x ^ (x >> 29)


def _ranks(c, g, n):
    """Ranks 1..rows by popularity (Zipf, optionally mixed with uniform draws); ranks above `rows` are unseen IDs."""
    R = c["rows"]
    u = _rand(g, n, dtype=torch.float64)
    if c["zipf"] == 0.0:
        r = (u * R).long() + 1
    else:
        a, m = c["zipf"], min(HEAD, R)
        head = torch.arange(1, m + 1, device="cuda", dtype=torch.float64) ** -a
        lo, hi = (m + 0.5) ** (1 - a), (R + 0.5) ** (1 - a)
        tail = (lo - hi) / (a - 1) if R > m else 0.0
        cdf = torch.cumsum(head, 0)
        u = u * (cdf[-1] + tail)
        r = torch.searchsorted(cdf, u, right=True) + 1
        if R > m:
            t = (u - cdf[-1]).clamp_min_(0.0).div_(tail)
            far = ((lo + t * (hi - lo)) ** (1.0 / (1 - a)) + 0.5).long()
            r = torch.where(r > m, far, r)
    r.clamp_(1, R)
    if c["uniform"] > 0.0:
        pick = _rand(g, n) < c["uniform"]
        r = torch.where(pick, (_rand(g, n, dtype=torch.float64) * R).long().clamp_(0, R - 1) + 1, r)
    if c["new"] > 0.0:
        pick = _rand(g, n) < c["new"]
        r = torch.where(pick, R + 1 + (_rand(g, n, dtype=torch.float64) * (8 * n)).long(), r)
    return r


def _batch(c, seed):
    """(ranks, offsets, vals) of one batch."""
    g = _gen(seed, 1)
    nb = c["B"] * c["F"]
    if c["bag"] == 0.0:
        lens = torch.ones(nb, dtype=torch.int64, device="cuda")
    else:
        lens = torch.poisson(torch.full((nb,), float(c["bag"]), device="cuda"), generator=g).long().clamp_(c["min_bag"], 64)
        # every seed's batch has the same number of entries: a few random bags give or take one
        while (off := _entries(c) - int(lens.sum())) != 0:
            can = lens < 64 if off > 0 else lens > c["min_bag"]
            at = torch.topk(_rand(g, nb) * can, min(abs(off), int(can.sum()))).indices
            lens[at] += 1 if off > 0 else -1
    offsets = torch.zeros(nb + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(lens, 0, out=offsets[1:])
    n = int(offsets[-1])
    ranks = _ranks(c, g, n)
    vals = _rand(g, n) * 1.75 + 0.25 if c["vals"] else None
    return ranks, offsets.int(), vals


def _mean_bag(c):
    if c["bag"] == 0.0:
        return 1.0
    return c["bag"] + (math.exp(-c["bag"]) if c["min_bag"] else 0.0)


def _entries(c):
    return int(round(c["B"] * c["F"] * _mean_bag(c)))


def _capacity(c, n):
    return c["rows"] + (int(n * c["new"] * 1.2) + 4096 if c["new"] else 0)


def _state_arrays(opt):
    return {"sgd": (0, 0), "adagrad": (1, 1), "adagrad_ftrl": (1, 2), "adam": (2, 2), "none": (0, 0)}[opt]


def _grad_scale(c):
    return 1.0 / c.get("B", 1024)


def _trained(c, seed, t, rows, state):
    """Fills the tensors of a table with the weights and optimizer state of a trained one (`t`: name -> tensor)."""
    g = _gen(seed, 2)
    s = _grad_scale(c)
    for x in t.values():
        x.zero_()
    t["emb"][:rows].normal_(0.0, INIT_SCALE, generator=g)
    t["w"][:rows].normal_(0.0, INIT_SCALE, generator=g)
    for name, kind in state.items():
        x = t[name][:rows]
        if kind == "square":           # sums (or averages) of squared gradients
            x.uniform_(10 * s * s, 100 * s * s, generator=g)
        else:                           # signed: Adam's first moment, FTRL's z
            x.normal_(0.0, kind if kind != "signed" else s, generator=g)


def _state_kinds(opt):
    if opt == "adagrad":
        return {"acc_emb": "square", "acc_w": "square"}
    if opt == "adagrad_ftrl":
        return {"acc_emb": "square", "acc_w": "square", "acc2_w": 0.2}
    if opt == "adam":
        return {"acc_emb": "signed", "acc_w": "signed", "acc2_emb": "square", "acc2_w": "square"}
    return {}


def _table(c, seed, opt, max_n, capacity):
    t = des.Table(c["D"], capacity, num_shards=c.get("K", 1),
                  shard_policy=des.SHARD_FIELD_MOD if c.get("policy") == "field" else des.SHARD_KEY_HASH,
                  init_seed=7, init_scale=INIT_SCALE, max_n=max(max_n, 1 << 16), state_arrays=_state_arrays(opt))
    for lo in range(0, c["rows"], t.max_n):
        t.insert(_ids(torch.arange(lo + 1, min(lo + t.max_n, c["rows"]) + 1, device="cuda")))
    names = [k for k in ("emb", "w", "acc_emb", "acc_w", "acc2_emb", "acc2_w") if getattr(t, k) is not None]
    _trained(c, seed, {k: getattr(t, k) for k in names}, c["rows"], _state_kinds(opt))
    return t, names


def _upstream(c, seed):
    g, s = _gen(seed, 3), _grad_scale(c)
    return {"g_lr": _randn(g, c["B"]) * s, "g_fm": _randn(g, c["B"]) * s, "g_pool": _randn(g, c["B"], c["F"], c["D"]) * s}


def _optimizer(opt):
    if opt == "sgd":
        return des.Optimizer(opt_emb=des.OPT_SGD, opt_w=des.OPT_SGD, lr=LR, eps=EPS)
    if opt == "adagrad":
        return des.Optimizer(opt_emb=des.OPT_ADAGRAD, opt_w=des.OPT_ADAGRAD, lr=LR, eps=EPS)
    if opt == "adagrad_ftrl":
        return des.Optimizer(opt_emb=des.OPT_ADAGRAD, opt_w=des.OPT_FTRL, lr=LR, eps=EPS, **FTRL)
    return des.Optimizer(opt_emb=des.OPT_ADAM, opt_w=des.OPT_ADAM, lr=LR, eps=EPS, **ADAM)


def _empty(*shape):
    return torch.empty(shape, dtype=torch.float32, device="cuda")


def _forward_buffers(c):
    B, F, D, K = c["B"], c["F"], c["D"], c["K"]
    return {"P_lr": _empty(K, B), "P_sum": _empty(K, B, D), "P_sq": _empty(K, B), "pool": _empty(B, F, D), "A_lr": _empty(B),
            "A_sum": _empty(B, D), "A_sq": _empty(B), "fm2": _empty(B)}


def _layer_inputs(c, seed):
    g = _gen(seed, 4)
    B, F, D, H = c["B"], c["F"], c["D"], c["H"]
    return {"pool": _randn(g, B, F, D) * 0.05, "W": _randn(g, F * D, H) / math.sqrt(F * D), "b": _randn(g, H) * 0.01,
            "dY": _randn(g, B, H) * 0.01}


def _cross_inputs(c, seed):
    g = _gen(seed, 5)
    B, F, D, n = c["B"], c["F"], c["D"], c["layers"]
    d = F * D
    return {"x0": _randn(g, B, F, D) * 0.05, "U": _randn(g, n + 1, d) / math.sqrt(d), "bias": _randn(g, n, d) * 0.01,
            "g": _randn(g, B) / B, "g_x0": _randn(g, B, F, D) * (0.05 / B)}


def _tower(c, seed):
    if c["model"] in ("lr", "fm"):
        return {"b0": np.full(1, -1.0, np.float32)}
    t = synth.tower_init(seed, c["F"], c["D"], (c["H1"], c["H2"]))
    if c["model"] == "dcn":
        t.update(synth.cross_init(seed, c["F"], c["D"], 2))
    return t


def _labels(c, seed):
    return (_rand(_gen(seed, 6), c["B"]) < 0.2).float()


def prepare(case, seed):
    c, kind = case, case["kind"]
    if kind == "layer":
        s = _layer_inputs(c, seed)
        B, F, D, H, K = c["B"], c["F"], c["D"], c["H"], c["K"]
        s.update(Y_partial=_empty(K, B, H), Y=_empty(B, H), g_pool=_empty(B, F, D), dW=_empty(F * D, H),
                 ws=torch.empty(des.dnn_backward_bytes(B, F, D, H), dtype=torch.uint8, device="cuda"))
    elif kind == "cross":
        s = _cross_inputs(c, seed)
        B, K, m, d, n = c["B"], c["K"], c["layers"] + 1, c["F"] * c["D"], c["layers"]
        s.update(P=_empty(K, B, m), t=_empty(B, m), gamma=_empty(B, m), c=_empty(B), dU=_empty(m, d), dbias=_empty(n, d),
                 ws=torch.empty(des.cross_net_bytes(B, d, n), dtype=torch.uint8, device="cuda"))
    elif kind == "evict":
        ranks = _ranks(c, _gen(seed, 1), c["n"])
        capacity = _capacity(c, c["n"])
        t, names = _table(c, seed, "adagrad", c["n"], capacity)
        # a newcomer that came only once is not worth a row: what was resident stays, the rest goes
        keep = torch.zeros(capacity, dtype=torch.uint8, device="cuda")
        keep[:c["rows"]] = 1
        s = {"table": t, "keys": _ids(ranks), "rows": torch.empty(c["n"], dtype=torch.int32, device="cuda"), "keep": keep,
             "staging": torch.empty(16 << 20, dtype=torch.uint8, device="cuda")}
    else:
        ranks, offsets, vals = _batch(c, seed)
        n = ranks.numel()
        opt = c["opt"] if kind == "step" else "adagrad" if kind == "model" else "none"
        t, names = _table(c, seed, opt, n, _capacity(c, n))
        s = {"table": t, "names": names, "batch": des.Batch(c["B"], c["F"], _ids(ranks), offsets, vals)}
        if kind == "model":
            s["model"] = model.Model(t, c["F"], c["model"], _tower(c, seed), c["B"],
                                     dict(opt_emb=des.OPT_ADAGRAD, opt_w=des.OPT_ADAGRAD, lr=LR, eps=EPS),
                                     dict(opt_emb=des.OPT_ADAGRAD, lr=0.01, eps=EPS))
            for k in s["model"].s1:                      # dense Adagrad state of a tower some steps old
                s["model"].s1[k].fill_(1e-4)
            s["labels"] = _labels(c, seed)
        else:
            s["rows"] = torch.empty(n, dtype=torch.int32, device="cuda")
            s.update(_forward_buffers(c))
        if kind == "step":
            s.update(_upstream(c, seed), optimizer=_optimizer(opt))
    s["case"] = dict(c)
    return s


# ---------------------------------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------------------------------
def run(s):
    c, kind = s["case"], s["case"]["kind"]
    if kind == "layer":
        des.dnn_partial_forward(s["pool"], s["W"], c["K"], out=s["Y_partial"])
        des.aggregate_bias_act(s["Y_partial"], s["b"], True, s["Y"])
        des.dnn_backward(s["pool"], s["W"], s["dY"], s["g_pool"], s["dW"], s["ws"])
        return {k: s[k] for k in ("Y_partial", "Y", "g_pool", "dW")}
    if kind == "cross":
        des.cross_net_partial(s["x0"], s["U"], c["K"], out=s["P"])
        des.aggregate_partials(s["P"].view(c["K"], -1), s["t"].view(-1))
        des.cross_net_forward(s["t"], s["U"], s["bias"], s["gamma"], s["c"], s["ws"])
        des.cross_net_backward(s["x0"], s["U"], s["bias"], s["t"], s["gamma"], s["g"], s["g_x0"], True, s["dU"], s["dbias"], s["ws"])
        return {k: s[k] for k in ("t", "c", "g_x0", "dU", "dbias")}
    t = s["table"]
    if kind == "evict":
        t.find(s["keys"], des.MISS_INSERT, s["rows"])
        n = t.compact(s["keep"], s["staging"])
        return {"rows": s["rows"], "n": n, "row_keys": t.row_keys[:c["rows"]], "emb": t.emb[:c["rows"]], "w": t.w[:c["rows"]]}
    if kind == "model":
        m = s["model"]
        loss = m.train_step(s["batch"], s["labels"])
        out = {"loss": loss, "logit": m.logit, "params": dict(m.params), "grads": dict(m.grads)}
        out.update({k: getattr(t, k) for k in s["names"]})
        return out
    t.find(s["batch"].keys, des.MISS_INSERT if kind == "step" else des.MISS_ZERO, s["rows"])
    t.partial_forward(s["batch"], s["rows"], s["P_lr"], s["P_sum"], s["P_sq"], s["pool"])
    des.aggregate_forward(s["P_lr"], s["P_sum"], s["P_sq"], s["A_lr"], s["A_sum"], s["A_sq"], s["fm2"])
    out = {k: s[k] for k in ("rows", "pool", "A_lr", "A_sum", "A_sq", "fm2")}
    if kind == "serve":
        out.update({k: s[k] for k in ("P_lr", "P_sum", "P_sq")})
        return out
    t.backward_update(s["batch"], s["rows"], s["optimizer"], g_lr=s["g_lr"], g_fm=s["g_fm"], A_sum=s["A_sum"], g_pool=s["g_pool"])
    out.update({k: getattr(t, k) for k in s["names"]})
    return out


# ---------------------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------------------------------------
def _distinct(c, n):
    """Expected number of distinct resident rows among n entries, and of new ones."""
    R, n_new = c["rows"], n * c["new"]
    n_old = n - n_new
    if c["zipf"] == 0.0:
        return R * -math.expm1(-n_old / R), n_new
    edges = np.unique(np.floor(np.geomspace(1, R + 1, 4000)))
    mid, width = np.sqrt(edges[:-1] * np.maximum(edges[1:] - 1, 1)), np.diff(edges)
    p = mid ** -c["zipf"]
    p /= float((p * width).sum())
    lam = n_old * ((1 - c["uniform"]) * p + c["uniform"] / R)
    return float((width * -np.expm1(-lam)).sum()), n_new


def work(case):
    c, kind = case, case["kind"]
    if kind == "layer":
        B, FD, H = c["B"], c["F"] * c["D"], c["H"]
        return {"bytes": 4.0 * (2 * B * FD + 2 * FD * H + (c["K"] + 2) * B * H), "flops": 6.0 * B * FD * H}
    if kind == "cross":
        B, d, m = c["B"], c["F"] * c["D"], c["layers"] + 1
        return {"bytes": 4.0 * (3 * B * d + 3 * m * d + 4 * B * m), "flops": 6.0 * B * d * m}
    if kind == "evict":
        u, new = _distinct(c, c["n"])
        slots = 1 << max(10, math.ceil(math.log2(_capacity(c, c["n"]) * 4 / 3 + 1)))
        return {"bytes": 12.0 * c["n"] + 16 * u + new * (32 + 8 * (c["D"] + 1)) + 16.0 * slots + 9.0 * c["rows"], "flops": 0.0}
    B, F, D = c["B"], c["F"], c["D"]
    n = _entries(c)
    u, new = _distinct(c, n)
    b = (16.0 if c["vals"] else 12.0) * n + 4.0 * B * F + 16 * (u + new) + 4.0 * B * (D + 3)
    fl = 6.0 * n * D
    if kind == "serve":
        return {"bytes": b + u * 4.0 * (D + 1) + 4.0 * B * F * D + 4.0 * c["K"] * B * (D + 2), "flops": fl}
    arrays = 1 + _state_arrays(c.get("opt", "adagrad"))[0]
    b += (u + new) * 8.0 * (D + 1) * arrays + 8.0 * B * F * D + 8.0 * B
    if kind == "model" and c["model"] not in ("lr", "fm"):
        k = F * D * c["H1"] + c["H1"] * c["H2"]
        return {"bytes": b + 4.0 * 5 * k, "flops": 2 * fl + 6.0 * B * k}
    return {"bytes": b, "flops": 2 * fl}


def tolerance(case):
    """About four times the distance from the 64-bit results that was measured at the listed cases.  Single weights move most:
    the first Adagrad step of a new row is lr*G/(|G|+eps), so an element whose gradient cancels to the order of eps
    amplifies a last-place difference of the gradient."""
    if case["kind"] == "layer":
        return {"rel": 1.5e-6, "max": 1e-5}
    if case["kind"] in ("serve", "cross", "evict"):
        return {"rel": 4e-7, "max": 2e-6}
    return {"rel": 3e-6, "max": 8e-3}


# ---------------------------------------------------------------------------------------------------------------------
# the same results in 64 bits, in plain torch
# ---------------------------------------------------------------------------------------------------------------------
def _shr(x, k):
    return (x >> k) & ((1 << (64 - k)) - 1)


def _mix64(z):
    z = (z ^ _shr(z, 30)) * (0xBF58476D1CE4E5B9 - (1 << 64))
    z = (z ^ _shr(z, 27)) * (0x94D049BB133111EB - (1 << 64))
    return z ^ _shr(z, 31)


def _initial(keys, cols, seed=7):
    """Initial weights of rows inserted without values: [len(keys), len(cols)] in 64 bits."""
    h = _mix64(keys[:, None] ^ _mix64(cols + seed)[None, :])
    width = float(np.float32(2.0 * math.sqrt(3.0) * float(np.float32(INIT_SCALE))))
    return (_shr(h, 40).double() * 2.0 ** -24 - 0.5) * width


def _rows_of(c, ranks, insert):
    """Rows of the batch's IDs and the new rows' IDs in row order."""
    R = c["rows"]
    rows = ranks - 1
    fresh = ranks > R
    if not insert:
        return torch.where(fresh, torch.full_like(rows, -1), rows), None
    at = torch.nonzero(fresh).flatten()
    if not at.numel():
        return rows, None
    u, inv = torch.unique(ranks[at], return_inverse=True)
    first = torch.full((u.numel(),), ranks.numel(), dtype=torch.int64, device="cuda").scatter_reduce_(0, inv, at, "amin")
    order = torch.argsort(first)
    place = torch.empty_like(order)
    place[order] = torch.arange(order.numel(), device="cuda")
    rows = rows.clone()
    rows[at] = R + place[inv]
    return rows, _ids(u[order])


def _table64(c, seed, opt, n_new_ids, capacity):
    names = ["emb", "w"] + [k for k in ("acc_emb", "acc_w", "acc2_emb", "acc2_w")
                            if _state_arrays(opt)[0 if k.endswith("emb") else 1] >= (2 if "2" in k else 1)]
    t = {k: _empty(capacity, c["D"]) if k.endswith("emb") else _empty(capacity) for k in names}
    _trained(c, seed, t, c["rows"], _state_kinds(opt))
    for k in list(t):                      # one array at a time: the largest ones are tens of gigabytes
        t[k] = t[k].double()
    if n_new_ids is not None:
        lo, hi = c["rows"], c["rows"] + n_new_ids.numel()
        t["emb"][lo:hi] = _initial(n_new_ids, torch.arange(c["D"], device="cuda"))
        t["w"][lo:hi] = _initial(n_new_ids, torch.tensor([c["D"]], device="cuda"))[:, 0]
    return t


def _update64(opt, theta, G, s1, s2, ftrl=False, lr=LR):
    if ftrl:
        a, be, l1, l2 = FTRL["ftrl_alpha"], FTRL["ftrl_beta"], FTRL["ftrl_l1"], FTRL["ftrl_l2"]
        n1 = s1 + G * G
        s2.add_(G - (n1.sqrt() - s1.sqrt()) / a * theta)
        s1.copy_(n1)
        theta.copy_(torch.where(s2.abs() <= l1, torch.zeros_like(s2), -(s2 - s2.sign() * l1) / ((be + n1.sqrt()) / a + l2)))
    elif opt == "sgd":
        theta.sub_(lr * G)
    elif opt == "adam":
        b1, b2, t = float(np.float32(ADAM["beta1"])), float(np.float32(ADAM["beta2"])), ADAM["step"]
        s1.mul_(b1).add_((1 - b1) * G)
        s2.mul_(b2).add_((1 - b2) * G * G)
        theta.sub_(lr * (s1 / (1 - b1 ** t)) / ((s2 / (1 - b2 ** t)).sqrt() + EPS))
    else:
        s1.add_(G * G)
        theta.sub_(lr * G / (s1.sqrt() + EPS))


def _apply_rows64(opt, t, touched, G, gw):
    ftrl = opt == "adagrad_ftrl"
    for lo in range(0, touched.numel(), CHUNK // 4):
        r = touched[lo:lo + CHUNK // 4]
        for name, grad in (("emb", G[lo:lo + r.numel()]), ("w", gw[lo:lo + r.numel()])):
            part = [t[k][r] if k in t else None for k in (name, "acc_" + name, "acc2_" + name)]
            _update64("adagrad" if ftrl else opt, part[0], grad, part[1], part[2], ftrl=ftrl and name == "w", lr=float(np.float32(LR)))
            for k, p in zip((name, "acc_" + name, "acc2_" + name), part):
                if p is not None:
                    t[k][r] = p


def _sums(bounds, n_out, width, rows_of):
    """out[i] = sum of the rows bounds[i] .. bounds[i+1] of a [n, width] array given piece by piece: rows_of(lo, hi).
    A plain loop over each segment's rows: no atomics, whose compare-and-swap form crawls on the hot IDs."""
    out = torch.zeros((n_out, width), dtype=torch.float64, device="cuda")
    cut = torch.searchsorted(bounds, torch.arange(0, int(bounds[-1]) + CHUNK, CHUNK, device="cuda")).clamp_(0, n_out).tolist()
    for i0, i1 in zip(cut[:-1], cut[1:]):
        if i1 > i0:
            lo, hi = int(bounds[i0]), int(bounds[i1])
            if hi > lo:
                out[i0:i1] = torch.segment_reduce(rows_of(lo, hi), "sum", lengths=bounds[i0 + 1:i1 + 1] - bounds[i0:i1], axis=0, initial=0.0)
    return out


def _grouped(key, n_out):
    """(order, bounds): the entries sorted by key, and where each key's run starts."""
    order = torch.argsort(key, stable=True)
    bounds = torch.zeros(n_out + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(torch.bincount(key, minlength=n_out), 0, out=bounds[1:])
    return order, bounds


def _exact_sparse(c, seed):
    kind, B, F, D, K = c["kind"], c["B"], c["F"], c["D"], c["K"]
    ranks, offsets, vals = _batch(c, seed)
    n = ranks.numel()
    opt = c["opt"] if kind == "step" else "none"
    rows, new_ids = _rows_of(c, ranks, kind == "step")
    t = _table64(c, seed, opt, new_ids, _capacity(c, n))
    offsets = offsets.long()
    bag = torch.repeat_interleave(torch.arange(B * F, device="cuda", dtype=torch.int32), offsets[1:] - offsets[:-1])

    def terms(e):
        """x*v, x*w and <x*v, x*v> of the entries `e`, side by side (an absent ID contributes nothing)."""
        r = rows[e]
        x = (r >= 0).double() if vals is None else (r >= 0).double() * vals[e].double()
        r = r.clamp_min(0)
        v = t["emb"][r] * x[:, None]
        return torch.cat([v, (t["w"][r] * x)[:, None], (v * v).sum(1, keepdim=True)], 1)

    per_bag = _sums(offsets, B * F, D + 2, lambda lo, hi: terms(slice(lo, hi))).view(B, F, D + 2)
    per_sample = per_bag.sum(1)
    A_sum, A_lr, A_sq = per_sample[:, :D].contiguous(), per_sample[:, D], per_sample[:, D + 1]
    out = {"rows": rows.int(), "pool": per_bag[:, :, :D].contiguous(), "A_lr": A_lr, "A_sum": A_sum, "A_sq": A_sq,
           "fm2": 0.5 * ((A_sum * A_sum).sum(1) - A_sq)}
    del per_bag
    if kind == "serve":
        shard = _shr(_mix64(_ids(ranks)), 32) % K if c["policy"] == "key" else (bag % F) % K
        order, bounds = _grouped(shard.long() * B + bag // F, K * B)
        P = _sums(bounds, K * B, D + 2, lambda lo, hi: terms(order[lo:hi])).view(K, B, D + 2)
        out.update({"P_lr": P[:, :, D], "P_sum": P[:, :, :D], "P_sq": P[:, :, D + 1]})
        return out
    up = _upstream(c, seed)
    touched, inv = torch.unique(rows, return_inverse=True)
    order, bounds = _grouped(inv, touched.numel())
    del inv

    def gradient(e):
        """d/dv without the term of the row's own vector, that term's factor, and d/dw, of the entries `e`."""
        bg = bag[e].long()
        b = bg // F
        x = 1.0 if vals is None else vals[e].double()
        gf = up["g_fm"].double()[b] * x
        g = up["g_pool"].view(B * F, D)[bg].double()
        if vals is not None:
            g *= x[:, None]
        g += A_sum[b] * gf[:, None]
        return torch.cat([g, (gf * x)[:, None], (up["g_lr"].double()[b] * x)[:, None]], 1)

    G = _sums(bounds, touched.numel(), D + 2, lambda lo, hi: gradient(order[lo:hi]))
    del order
    for lo in range(0, touched.numel(), CHUNK):
        g = G[lo:lo + CHUNK]
        g[:, :D] -= t["emb"][touched[lo:lo + CHUNK]] * g[:, D:D + 1]
    _apply_rows64(c["opt"], t, touched, G[:, :D], G[:, D + 1])
    out.update(t)
    return out


def _exact_model(c, seed):
    B, F, D, kind = c["B"], c["F"], c["D"], c["model"]
    ranks, offsets, vals = _batch(c, seed)
    rows, _ = _rows_of(c, ranks, True)
    t = _table64(c, seed, "adagrad", None, _capacity(c, ranks.numel()))
    x = torch.ones(rows.numel(), dtype=torch.float64, device="cuda") if vals is None else vals.double()
    v, w = t["emb"][rows].requires_grad_(), t["w"][rows].requires_grad_()       # one leaf per entry; summed by row below
    xv = v * x[:, None]
    per = (offsets[1:] - offsets[:-1]).long()
    pool = torch.segment_reduce(xv, "sum", lengths=per, axis=0, initial=0.0).view(B, F, D)
    per_sample = lambda z: torch.segment_reduce(z, "sum", lengths=per.view(B, F).sum(1), axis=0, initial=0.0)
    p = {k: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda().double().requires_grad_() for k, a in _tower(c, seed).items()}
    logit = p["b0"].expand(B)
    parts = model.COMPONENTS[kind]
    if "lr" in parts:
        logit = logit + per_sample(w * x)
    if "fm" in parts:
        A = pool.sum(1)
        logit = logit + 0.5 * ((A * A).sum(1) - per_sample((xv * xv).sum(1)))
    if "dnn" in parts:
        h = torch.relu(pool.reshape(B, F * D) @ p["W1"] + p["b1"])
        h = torch.relu(h @ p["W2"] + p["b2"])
        logit = logit + h @ p["w_out"]
    if "cross" in parts:
        x0 = pool.reshape(B, F * D)
        y = x0
        for l in (1, 2):
            y = x0 * (y @ p["cw%d" % l])[:, None] + p["cb%d" % l] + y
        logit = logit + y @ p["w_cross"]
    lab = _labels(c, seed).double()
    loss = (torch.nn.functional.softplus(logit) - lab * logit).mean()
    loss.backward()
    grads = {k: a.grad if a.grad is not None else torch.zeros_like(a) for k, a in p.items()}
    zero_if_none = lambda a: a.grad if a.grad is not None else torch.zeros_like(a)
    with torch.no_grad():
        touched, inv = torch.unique(rows, return_inverse=True)
        order, bounds = _grouped(inv, touched.numel())
        gv, gw = zero_if_none(v), zero_if_none(w)
        G = _sums(bounds, touched.numel(), D + 1, lambda lo, hi: torch.cat([gv[order[lo:hi]], gw[order[lo:hi], None]], 1))
        _apply_rows64("adagrad", t, touched, G[:, :D], G[:, D])
        new = {}
        for k, a in p.items():
            theta, s1 = a.detach().clone(), torch.full_like(a, float(np.float32(1e-4)))
            _update64("adagrad", theta, grads[k], s1, None, lr=float(np.float32(0.01)))
            new[k] = theta
    return dict(t, loss=loss.detach().reshape(1), logit=logit.detach(), params=new, grads=grads)


def _exact_layer(c, seed):
    s = {k: a.double() for k, a in _layer_inputs(c, seed).items()}
    B, F, D, H, K = c["B"], c["F"], c["D"], c["H"], c["K"]
    part = torch.zeros((K, B, H), dtype=torch.float64, device="cuda")
    W = s["W"].view(F, D, H)
    for k in range(min(K, F)):
        part[k] = s["pool"][:, k::K].reshape(B, -1) @ W[k::K].reshape(-1, H)
    x = s["pool"].view(B, F * D)
    return {"Y_partial": part, "Y": torch.relu(part.sum(0) + s["b"]), "g_pool": (s["dY"] @ s["W"].t()).view(B, F, D), "dW": x.t() @ s["dY"]}


def _exact_cross(c, seed):
    s = {k: a.double() for k, a in _cross_inputs(c, seed).items()}
    B, d, n = c["B"], c["F"] * c["D"], c["layers"]
    x0, U, b = s["x0"].view(B, d).requires_grad_(), s["U"].requires_grad_(), s["bias"].requires_grad_()
    y = x0
    for l in range(n):
        y = x0 * (y @ U[l])[:, None] + b[l] + y
    out = y @ U[n]
    (out * s["g"]).sum().backward()
    return {"t": (x0 @ U.t()).detach(), "c": out.detach(), "g_x0": s["g_x0"] + x0.grad.view(B, c["F"], c["D"]), "dU": U.grad, "dbias": b.grad}


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "layer":
        return _exact_layer(c, seed)
    if kind == "cross":
        return _exact_cross(c, seed)
    if kind == "model":
        return _exact_model(c, seed)
    if kind == "evict":
        rows, _ = _rows_of(c, _ranks(c, _gen(seed, 1), c["n"]), True)
        t = _table64(c, seed, "adagrad", None, _capacity(c, c["n"]))
        return {"rows": rows.int(), "n": c["rows"], "row_keys": _ids(torch.arange(1, c["rows"] + 1, device="cuda")),
                "emb": t["emb"][:c["rows"]], "w": t["w"][:c["rows"]]}
    return _exact_sparse(c, seed)
