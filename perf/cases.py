"""The work a user of this framework has it do, as measurable cases.

Each case is one pass through a public entry point: an exact query, a filter,
a training evaluation of a relaxed query, a dictionary encoding, or a layer of
the label classifier.  Sizes and value distributions follow the generators and
the benchmark of this repository; inputs are drawn on the GPU from the seed.

Query cases call the prepared plan and read its answer back (the number of
groups and the status word), as a program that wants the answer does;
training evaluations only enqueue, as a training loop does.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2211_02753_amd import _lib as L
from paper_2211_02753_amd import dictenc, llp, query as Q, soft, trainable

DEV = torch.device("cuda:0")

# ---------------------------------------------------------------- the cases


def listed():
    return [
        # A dashboard panel: SUM(label) per bucket of a 120K-row label column (the swapped-in exact
        # query over a learned column); the smallest call, where launches and latency count.
        {"name": "agg_bucket_120k", "kind": "agg", "n": 120_000, "groups": 100, "value": "i8"},
        # The star join of an ordinary interactive query: 1M facts, a 10K-row dimension with the group key.
        {"name": "star_join_1m", "kind": "star", "n": 1_000_000, "n_dim": 10_000, "literal": 1278},
        # A selection vector over the largest date column.
        {"name": "filter_60m", "kind": "filter", "n": 60_000_000, "dtype": "i32", "op": "<=", "literal": 2450,
         "chained": False},
        # The headline query: the largest fact table against a dimension far beyond the caches.
        {"name": "fact_dim_60m", "kind": "fact", "n": 60_000_000, "n_dim": 15_000_000, "literal": 2450, "zipf": 0.0,
         "hit": 1.0},
        # A skewed many-to-many join aggregated over a million groups.
        {"name": "many_to_many_20m", "kind": "mn", "n_left": 20_000_000, "n_right": 20_000_000, "n_keys": 2_000_000,
         "groups": 1_000_000, "topk": 0},
        # One training evaluation of the relaxed filter and grouped sum, forward and backward.
        {"name": "soft_query_10m", "kind": "soft", "n": 10_000_000, "groups": 1000, "tau": 1.0, "dx": False},
        # The soft COUNT of the grid-of-images query: 9 x 9 tiles an image, digit and size probabilities.
        {"name": "pe_count_123k", "kind": "pe", "grids": 123_457, "tiles": 81, "k1": 10, "k2": 2},
        # One training evaluation of a relaxed two-conjunct WHERE with a grouped COUNT.
        {"name": "soft_where_10m", "kind": "where", "n": 10_000_000, "conjuncts": 2, "value": False, "dtau": False},
        # One training step of learning from label proportions.
        {"name": "llp_step_8m", "kind": "llp", "n": 8_388_608, "features": 8, "classes": 2, "bag": 64},
        # Encoding a string column on load.
        {"name": "dict_encode_10m", "kind": "dict", "n": 10_000_000, "distinct": 100_000, "width": 16},
        # The classifier's heavy layer: forward at the inference batch.
        {"name": "conv2_fwd_1024", "kind": "conv_fwd", "batch": 1024, "layer": 2},
        # The same layer's gradients at the training batch.
        {"name": "conv2_bwd_256", "kind": "conv_bwd", "batch": 256, "layer": 2},
    ]


def _log_int(rng, lo, hi):
    """A whole number spread over the logarithm of [lo, hi]; mostly odd sizes come out."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["agg", "star", "filter", "fact", "mn", "soft", "pe", "where", "llp", "dict", "conv_fwd",
                       "conv_bwd"])
    c = {"kind": kind}
    if kind == "agg":
        n = _log_int(rng, 1000, 20_000_000)
        c.update(n=n, groups=_log_int(rng, 2, min(2000, n // 10)), value=rng.choice(["i8", "i32", "i64"]))
    elif kind == "star":
        c.update(n=_log_int(rng, 10_000, 20_000_000), n_dim=_log_int(rng, 100, 200_000), literal=rng.randrange(400, 2556))
    elif kind == "filter":
        dt = rng.choice(["i8", "i32", "i32", "i64"])
        lit = rng.randrange(-120, 120) if dt == "i8" else rng.randrange(10, 2550)
        c.update(n=_log_int(rng, 1000, 60_000_000), dtype=dt, op=rng.choice(["<", "<=", ">", ">=", "==", "!="]),
                 literal=lit, chained=rng.random() < 0.25)
    elif kind == "fact":
        n = _log_int(rng, 1_000_000, 60_000_000)
        c.update(n=n, n_dim=min(15_000_000, _log_int(rng, 50_000, n)), literal=rng.randrange(100, 2556),
                 zipf=rng.choice([0.0, 0.0, 1.1]), hit=rng.choice([1.0, 1.0, 0.6]))
    elif kind == "mn":
        nl, nr = _log_int(rng, 100_000, 20_000_000), _log_int(rng, 100_000, 20_000_000)
        c.update(n_left=nl, n_right=nr, n_keys=max(1000, min(2_000_000, nr // rng.randrange(4, 20))),
                 groups=_log_int(rng, 1000, nl // 20), topk=rng.choice([0, 0, 100]))
    elif kind == "soft":
        c.update(n=_log_int(rng, 10_000, 10_000_000), groups=_log_int(rng, 10, 4000), tau=rng.choice([1.0, 0.5, 0.125]),
                 dx=rng.random() < 0.3)
    elif kind == "pe":
        k1 = rng.randrange(2, 17)
        c.update(grids=_log_int(rng, 100, 123_457), tiles=rng.randrange(4, 82), k1=min(k1, 10) if rng.random() < 0.7 else k1,
                 k2=rng.randrange(1, 3))
    elif kind == "where":
        c.update(n=_log_int(rng, 10_000, 10_000_000), conjuncts=rng.randrange(1, 4), value=rng.random() < 0.4,
                 dtau=rng.random() < 0.4)
    elif kind == "llp":
        c.update(n=_log_int(rng, 4096, 8_388_608), features=rng.randrange(2, 17), classes=rng.randrange(2, 5),
                 bag=1 << rng.randrange(0, 11))
    elif kind == "dict":
        n, w = _log_int(rng, 10_000, 10_000_000), rng.choice([4, 8, 12, 16, 24, 32])
        c.update(n=n, distinct=_log_int(rng, 16, min(100_000 if w > 4 else 20_000, n // 4)), width=w)
    elif kind == "conv_fwd":
        c.update(batch=_log_int(rng, 1, 1024), layer=rng.choice([1, 2, 2]))
    else:
        c.update(batch=_log_int(rng, 1, 256), layer=2)
    return c


# ------------------------------------------------------------ drawn inputs


def _gen(seed, salt=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(1_000_003 * int(seed) + salt)
    return g


def _ints(g, n, lo, hi, dtype):
    """Uniform in the inclusive range [lo, hi]."""
    return torch.randint(lo, hi + 1, (n,), generator=g, device=DEV, dtype=dtype)


def _spread(g, n, k, dtype):
    """n values of 0 .. k-1 in a random order, each as often as the others (so answers keep their size
    from one seed to the next)."""
    return (torch.randperm(n, generator=g, device=DEV) % k).to(dtype)


def _zipf(g, n, ranks, s):
    w = torch.arange(1, ranks + 1, device=DEV, dtype=torch.float64).pow_(-s).cumsum_(0)
    w /= w[-1].clone()
    u = torch.rand(n, generator=g, device=DEV, dtype=torch.float64)
    return torch.searchsorted(w, u, right=True).clamp_(max=ranks - 1)


def _scattered_keys(n):
    """n distinct int32 keys, the image of 0..n-1 under an odd multiplier mod 2^32."""
    j = torch.arange(n, device=DEV, dtype=torch.int64)
    u = (j * 0x9E3779B1 + 0x7F4A7C15) & 0xFFFFFFFF
    return (u - ((u >> 31) << 32)).to(torch.int32)


_INT = {"i8": torch.int8, "i32": torch.int32, "i64": torch.int64}


def _inputs(c, seed):
    """The tensors a program holds before the call, from the seed alone."""
    g = _gen(seed)
    k = c["kind"]
    if k == "agg":
        dt = _INT[c["value"]]
        hi = 9 if dt == torch.int8 else 100_000
        return {"bucket": _spread(g, c["n"], c["groups"], torch.int32), "value": _ints(g, c["n"], 0, hi, dt)}
    if k == "star":
        n, nd = c["n"], c["n_dim"]
        return {"key": _ints(g, n, 0, nd - 1, torch.int32), "price": _ints(g, n, 100, 100_000, torch.int64),
                "day": _ints(g, n, 0, 2555, torch.int32), "flag": _ints(g, n, 0, 2, torch.int8),
                "pk": torch.arange(nd, device=DEV, dtype=torch.int32), "region": _ints(g, nd, 0, 24, torch.int8)}
    if k == "filter":
        n, (lo, span) = c["n"], (-128, 256) if c["dtype"] == "i8" else (0, 2556)
        order = torch.randperm(n, generator=g, device=DEV)
        col = torch.empty(n, device=DEV, dtype=_INT[c["dtype"]])
        col[order] = (torch.arange(n, device=DEV) % span + lo).to(col.dtype)
        # chained: the survivors of an earlier conjunct, half the rows, ascending
        return {"col": col, "sel": order[:n // 2].sort()[0].to(torch.int32) if c["chained"] else None}
    if k == "fact":
        n, nd = c["n"], c["n_dim"]
        pk = _scattered_keys(nd)[torch.randperm(nd, generator=g, device=DEV)]
        idx = _zipf(g, n, nd, c["zipf"]) if c["zipf"] else torch.randint(0, nd, (n,), generator=g, device=DEV)
        return {"orderkey": pk[idx], "extprice": _ints(g, n, 90_000, 10_500_000, torch.int64),
                "discount": _ints(g, n, 0, 10, torch.int64), "shipday": _ints(g, n, 0, 2555, torch.int32),
                "returnflag": _ints(g, n, 0, 2, torch.int8), "linestatus": _ints(g, n, 0, 1, torch.int8),
                # a dimension cut to hit * n_dim rows leaves some facts without a partner
                "dim_key": pk[torch.randperm(nd, generator=g, device=DEV)[:max(1, int(nd * c["hit"]))]].contiguous()}
    if k == "mn":
        perm = torch.randperm(c["n_keys"], generator=g, device=DEV).to(torch.int32)
        nl, nr = c["n_left"], c["n_right"]
        return {"lkey": perm[_zipf(g, nl, c["n_keys"], 0.8)], "gkey": _spread(g, nl, c["groups"], torch.int32),
                "lpay": _ints(g, nl, 0, (1 << 20) - 1, torch.int64), "rkey": perm[_zipf(g, nr, c["n_keys"], 0.8)],
                "rpay": _ints(g, nr, 0, (1 << 20) - 1, torch.int64)}
    if k == "soft":
        n, G = c["n"], c["groups"]
        d = {"x": torch.randn(n, generator=g, device=DEV), "v": torch.rand(n, generator=g, device=DEV),
             "g": _ints(g, n, 0, G - 1, torch.int32), "c": torch.full((1,), 0.3, device=DEV)}
        T = torch.zeros(G, device=DEV, dtype=torch.float64)  # the answer of the exact filter x < 0.5
        T.index_add_(0, d["g"].long(), torch.where(d["x"] < 0.5, d["v"].double(), 0.0))
        d["T"] = T.float()
        return d
    if k == "pe":
        n = c["grids"] * c["tiles"]
        p = torch.softmax(2 * torch.randn((n, c["k1"]), generator=g, device=DEV), 1)
        q = torch.softmax(2 * torch.randn((n, c["k2"]), generator=g, device=DEV), 1)
        seg = torch.arange(c["grids"] + 1, device=DEV, dtype=torch.int64) * c["tiles"]
        dS = torch.randn((c["grids"], c["k1"], c["k2"]), generator=g, device=DEV)
        return {"p": p, "q": q, "seg": seg, "dS": dS}
    if k == "where":
        n = c["n"]
        region, flag = _ints(g, n, 0, 24, torch.int8), _ints(g, n, 0, 2, torch.int8)
        u = torch.rand((2, n), generator=g, device=DEV, dtype=torch.float64)
        d = {"region": region, "flag": flag, "day": (50 * region.long() + (u[0] * 2000).long()).to(torch.int32),
             "qty": (1 + (u[1] * (30 + 15 * flag.long())).long()).to(torch.int32),
             "x": torch.randn(n, generator=g, device=DEV),
             "price": _ints(g, n, 100, 100_000, torch.int32) if c["value"] else None}
        hit = d["day"] < 1278
        if c["conjuncts"] > 1:
            hit &= d["qty"] >= 20
        if c["conjuncts"] > 2:
            hit &= d["x"] < 0.5
        e = d["price"].double() if c["value"] else torch.ones(n, device=DEV, dtype=torch.float64)
        T = torch.zeros(75, device=DEV, dtype=torch.float64)
        T.index_add_(0, region.long() * 3 + flag.long(), torch.where(hit, e, 0.0))
        d["T"] = T.float()
        return d
    if k == "llp":
        n, F, C = c["n"], c["features"], c["classes"]
        X = torch.randn((n, F), generator=g, device=DEV)
        y = (X @ torch.linspace(1.5, -1.0, F, device=DEV) > 0.7).long() + (X[:, 0] > 1.0).long() * (C - 2)
        nb = -(-n // c["bag"])
        T = torch.zeros(nb * C, device=DEV)
        T.index_add_(0, torch.arange(n, device=DEV) // c["bag"] * C + y, torch.ones(n, device=DEV))
        return {"X": X, "T": T, "W": 0.3 * torch.randn((C, F), generator=g, device=DEV),
                "b": 0.1 * torch.randn(C, generator=g, device=DEV)}
    if k == "dict":
        nd, w = c["distinct"], c["width"]
        m = 3 * nd + 64
        words = _ints(g, m * w, ord("a"), ord("z"), torch.uint8).view(m, w)
        length = torch.randint(1, w + 1, (m, 1), generator=g, device=DEV)
        words = torch.where(torch.arange(w, device=DEV)[None, :] < length, words, torch.zeros_like(words)).unique(dim=0)
        words = words[torch.randperm(words.shape[0], generator=g, device=DEV)[:nd]]
        return {"strs": words[_spread(g, c["n"], nd, torch.int64)].contiguous()}
    H, ci, co = (28, 1, 32) if c["layer"] == 1 else (26, 32, 64)
    B = c["batch"]
    bf = torch.bfloat16
    x = (torch.rand((B, H, H, ci), generator=g, device=DEV) if ci == 1 else
         torch.randn((B, H, H, ci), generator=g, device=DEV).relu_()).to(bf)
    d = {"x": x, "w": (torch.randn((co, 3, 3, ci), generator=g, device=DEV) * (2 / (9 * ci)) ** 0.5).to(bf),
         "bias": 0.05 * torch.randn(co, generator=g, device=DEV), "H": H, "ci": ci, "co": co}
    if k == "conv_bwd":  # about half the outputs sit behind a ReLU that closed
        dy = torch.randn((B, H - 2, H - 2, co), generator=g, device=DEV)
        d["dy"] = (1e-3 * dy * (torch.rand(dy.shape, generator=g, device=DEV) < 0.5)).to(bf)
    return d


def prepare(case, seed):
    c = dict(case)
    d = _inputs(c, seed)
    k = c["kind"]
    st = {"case": c, "in": d}
    if k == "agg":
        st["plan"] = Q.GroupbyQuery(c["n"], [Q.Key(d["bucket"], 0, c["groups"])], expr=L.EXPR_COL,
                                    a=Q.Operand(d["value"]))
    elif k == "star":
        st["plan"] = Q.GroupbyQuery(c["n"], [Q.Key(d["region"], 0, 25, L.BUILD), Q.Key(d["flag"], 0, 3)],
                                    expr=L.EXPR_COL, a=Q.Operand(d["price"]), pred=(d["day"], "<", c["literal"]),
                                    join=(d["pk"], d["key"], True))
    elif k == "fact":
        st["plan"] = Q.GroupbyQuery(c["n"], [Q.Key(d["returnflag"], 0, 3), Q.Key(d["linestatus"], 0, 2)],
                                    expr=L.EXPR_MUL_CONST_SUB, a=Q.Operand(d["extprice"]), b=Q.Operand(d["discount"]),
                                    k=100, pred=(d["shipday"], "<=", c["literal"]),
                                    join=(d["dim_key"], d["orderkey"], True))
    elif k == "mn":
        st["plan"] = Q.GroupbyQuery(c["n_left"], [Q.Key(d["gkey"], 0, c["groups"])], expr=L.EXPR_MUL,
                                    a=Q.Operand(d["lpay"]), b=Q.Operand(d["rpay"], L.BUILD),
                                    join=(d["rkey"], d["lkey"], False, 0, c["n_keys"]), topk=c["topk"])
    elif k == "soft":
        st["step"] = soft.SoftQueryStep(d["x"], d["v"], d["g"], d["c"], c["tau"], c["groups"], d["T"], want_dx=c["dx"])
    elif k == "pe":
        st["status"] = torch.zeros(1, dtype=torch.int32, device=DEV)
        soft.soft_workspace(DEV)
    elif k == "where":
        where = [trainable.Where(d["day"], "<", 1500.0), trainable.Where(d["qty"], ">=", 12.0),
                 trainable.Where(d["x"], "<", 0.75)][:c["conjuncts"]]
        st["plan"] = trainable.TrainableQuery(c["n"], [Q.Key(d["region"], 0, 25), Q.Key(d["flag"], 0, 3)], where,
                                              value=d["price"],
                                              tau=[20.0, 1.0, 0.25][:c["conjuncts"]]).compile(trainable=True)
        st["plan"].step_buffers()
        soft.soft_workspace(DEV)
    elif k == "llp":
        st["model"] = llp.LinearLLP(d["W"].clone(), d["b"].clone())
    elif k in ("conv_fwd", "conv_bwd"):
        B, H, ci, co = c["batch"], d["H"], d["ci"], d["co"]
        i16, f32 = dict(dtype=torch.int16, device=DEV), dict(dtype=torch.float32, device=DEV)
        if k == "conv_fwd":
            st["y"] = torch.empty((B, H - 2, H - 2, co), **i16)
        else:
            st["dx"] = torch.empty((B, H, H, ci), **i16)
            st["dw"], st["db"] = torch.empty((co, 3, 3, ci), **f32), torch.empty(co, **f32)
    return st


# ------------------------------------------------------------------ a pass


def run(st):
    c, d, k = st["case"], st["in"], st["case"]["kind"]
    if k in ("agg", "star", "fact", "mn"):
        return st["plan"]()
    if k == "filter":
        return Q.filter(d["col"], c["op"], c["literal"], d["sel"])
    if k == "soft":
        s = st["step"]
        s()
        return {"S": s.S, "loss": s.loss, "dS": s.dS, "dv": s.dv, "dc": s.dc, "dx": s.dx}
    if k == "pe":
        S = soft.soft_pe_groupby(d["p"], d["q"], d["seg"], c["grids"], status=st["status"])
        dp, dq = soft.soft_pe_groupby_bwd(d["p"], d["q"], d["seg"], d["dS"])
        return {"S": S, "dp": dp, "dq": dq}
    if k == "where":
        loss, dc, dtau = st["plan"].loss_and_grad(d["T"], want_dtau=c["dtau"])
        return {"loss": loss, "dc": dc, "dtau": dtau}
    if k == "llp":
        m = st["model"]
        loss = m.step(d["X"], d["T"], c["bag"], 0.05)
        return {"loss": loss, "gW": m.gW, "gb": m.gb, "W": m.W, "b": m.b}
    if k == "dict":
        words, codes = dictenc.encode(d["strs"], c["distinct"])
        return {"dict": words, "codes": codes}
    lib, s = L.load(), L.stream_handle(DEV)
    B, H, ci, co = c["batch"], d["H"], d["ci"], d["co"]
    if k == "conv_fwd":
        L.check("conv", lib.tdp_conv3x3_fwd_bf16(L.ptr(d["x"]), L.ptr(d["w"]), L.ptr(d["bias"]), B, H, H, ci, co, 1,
                                                 L.ptr(st["y"]), s))
        return {"y": st["y"].view(torch.bfloat16)}
    L.check("conv", lib.tdp_conv3x3_wgrad_bf16(L.ptr(d["x"]), L.ptr(d["dy"]), B, H, H, ci, co, L.ptr(st["dw"]),
                                               L.ptr(st["db"]), s))
    L.check("conv", lib.tdp_conv3x3_dgrad_bf16(L.ptr(d["dy"]), L.ptr(d["w"]), L.ptr(d["x"]), B, H, H, ci, co,
                                               L.ptr(st["dx"]), s))
    return {"dx": st["dx"].view(torch.bfloat16), "dw": st["dw"], "db": st["db"]}


# ---------------------------------------------- what a pass cannot do without


def work(c):
    """Each input read once, each output written once."""
    k = c["kind"]
    if k == "agg":
        return {"bytes": c["n"] * (4 + {"i8": 1, "i32": 4, "i64": 8}[c["value"]]) + 32 * c["groups"], "flops": c["n"]}
    if k == "star":  # key, price, day, flag; the dimension's key and region
        return {"bytes": 17 * c["n"] + 5 * c["n_dim"] + 40 * 75, "flops": c["n"]}
    if k == "filter":  # the column and the row ids that survive (about; "==" and "!=" keep one value or drop it)
        size, span = {"i8": (1, 256), "i32": (4, 2556), "i64": (8, 2556)}[c["dtype"]]
        at = c["literal"] + (128 if c["dtype"] == "i8" else 0)
        keep = {"<": at, "<=": at + 1, ">": span - 1 - at, ">=": span - at, "==": 1, "!=": span - 1}[c["op"]] / span
        n = c["n"] * (0.5 if c["chained"] else 1.0)
        return {"bytes": n * (size + (4 if c["chained"] else 0)) + 4 * n * keep, "flops": n}
    if k == "fact":  # orderkey, extprice, discount, shipday, two flags; the dimension's key
        return {"bytes": 26 * c["n"] + 4 * int(c["n_dim"] * c["hit"]) + 240, "flops": 3 * c["n"]}
    if k == "mn":  # key, group, payload; key, payload; the groups (or the best of them)
        groups = min(c["groups"], c["topk"]) if c["topk"] else c["groups"]
        return {"bytes": 16 * c["n_left"] + 12 * c["n_right"] + 32 * groups, "flops": 2 * c["n_left"] + 2 * c["n_right"]}
    if k == "soft":  # x, v, g read; dv (and dx) written
        return {"bytes": (16 + (4 if c["dx"] else 0)) * c["n"] + 8 * c["groups"], "flops": 20 * c["n"]}
    if k == "pe":  # p and q read, dp and dq written; S written, dS read
        n, kk = c["grids"] * c["tiles"], c["k1"] + c["k2"]
        return {"bytes": 8 * n * kk + 8 * c["grids"] * c["k1"] * c["k2"], "flops": 6 * n * c["k1"] * c["k2"]}
    if k == "where":  # the keys, the columns of the conjuncts, the value
        return {"bytes": c["n"] * (2 + 4 * c["conjuncts"] + (4 if c["value"] else 0)), "flops": 20 * c["n"] * c["conjuncts"]}
    if k == "llp":
        return {"bytes": 4 * c["n"] * c["features"] + 4 * c["classes"] * -(-c["n"] // c["bag"]),
                "flops": 6 * c["n"] * c["features"] * c["classes"]}
    if k == "dict":  # the strings read, their codes and the dictionary written
        return {"bytes": c["n"] * (c["width"] + 4) + c["distinct"] * c["width"], "flops": c["n"]}
    H, ci, co = (28, 1, 32) if c["layer"] == 1 else (26, 32, 64)
    B, macs = c["batch"], c["batch"] * (H - 2) ** 2 * 9 * ci * co
    x, y, w = 2 * B * H * H * ci, 2 * B * (H - 2) ** 2 * co, 2 * 9 * ci * co
    if k == "conv_fwd":
        return {"bytes": x + y + w, "flops": 2 * macs}
    return {"bytes": 2 * x + y + 3 * w, "flops": 4 * macs}


# --------------------------------------------------- the same in 64 bits


def _avg(gid, value, n_cells, topk=0):
    """AVG of each non-empty group in key order (or of the topk largest sums, ties to the smaller key)."""
    s = torch.zeros(n_cells, device=DEV, dtype=torch.int64).index_add_(0, gid, value)
    n = torch.zeros(n_cells, device=DEV, dtype=torch.int64).index_add_(0, gid, torch.ones_like(value))
    at = (n > 0).nonzero()[:, 0]
    if topk:
        at = at[torch.argsort(s[at], descending=True, stable=True)[:topk]]
    return s[at].double() / n[at].double()


def exact(case, seed):
    c = dict(case)
    k = c["kind"]
    if k in ("filter", "dict"):  # whole numbers and bytes
        return None
    d = _inputs(c, seed)
    if k == "agg":
        return {"k0": None, "sum": None, "count": None, "avg": _avg(d["bucket"].long(), d["value"].long(), c["groups"])}
    if k == "star":
        on = d["day"] < c["literal"]
        gid = d["region"][d["key"][on].long()].long() * 3 + d["flag"][on].long()
        return {"k0": None, "k1": None, "sum": None, "count": None, "avg": _avg(gid, d["price"][on], 75)}
    if k == "fact":
        keys = d["dim_key"].sort()[0]
        at = torch.searchsorted(keys, d["orderkey"]).clamp_(max=keys.numel() - 1)
        on = (keys[at] == d["orderkey"]) & (d["shipday"] <= c["literal"])
        gid = (d["returnflag"].long() * 2 + d["linestatus"].long())[on]
        return {"k0": None, "k1": None, "sum": None, "count": None,
                "avg": _avg(gid, (d["extprice"] * (100 - d["discount"]))[on], 6)}
    if k == "mn":
        cnt = torch.zeros(c["n_keys"], device=DEV, dtype=torch.int64)
        rsum = torch.zeros_like(cnt)
        cnt.index_add_(0, d["rkey"].long(), torch.ones_like(d["rpay"]))
        rsum.index_add_(0, d["rkey"].long(), d["rpay"])
        lk, g = d["lkey"].long(), d["gkey"].long()
        s = torch.zeros(c["groups"], device=DEV, dtype=torch.int64).index_add_(0, g, d["lpay"] * rsum[lk])
        n = torch.zeros_like(s).index_add_(0, g, cnt[lk])
        at = (n > 0).nonzero()[:, 0]
        if c["topk"]:
            at = at[torch.argsort(s[at], descending=True, stable=True)[:c["topk"]]]
        return {"k0": None, "sum": None, "count": None, "avg": s[at].double() / n[at].double()}
    if k == "soft":
        x, v, g, G, tau = d["x"].double(), d["v"].double(), d["g"].long(), c["groups"], c["tau"]
        w = torch.sigmoid((d["c"].double() - x) / tau)
        S = torch.zeros(G, device=DEV, dtype=torch.float64).index_add_(0, g, w * v)
        dS = 2 * (S - d["T"].double()) / G
        r = dS[g]
        t = r * v * w * (1 - w) / tau
        return {"S": S, "loss": (S - d["T"].double()).square().mean().view(1), "dS": dS, "dv": r * w,
                "dc": t.sum().view(1), "dx": -t if c["dx"] else None}
    if k == "pe":
        n, G, T = c["grids"] * c["tiles"], c["grids"], c["tiles"]
        p, q, dS = d["p"].double(), d["q"].double(), d["dS"].double()
        S = torch.empty((G, c["k1"], c["k2"]), device=DEV, dtype=torch.float64)
        dp, dq = torch.zeros_like(p), torch.empty_like(q)
        pt, qt = p.view(G, T, c["k1"]), q.view(G, T, c["k2"])
        for b in range(c["k2"]):
            S[:, :, b] = (pt * qt[:, :, b:b + 1]).sum(1)
            dp += (dS[:, None, :, b] * qt[:, :, b:b + 1]).view(n, c["k1"])
            dq.view(G, T, c["k2"])[:, :, b] = (pt * dS[:, None, :, b]).sum(2)
        return {"S": S, "dp": dp, "dq": dq}
    if k == "where":
        J = c["conjuncts"]
        xs = [d["day"].double(), d["qty"].double(), d["x"].double()][:J]
        th, sg, tau = (1500.0, 12.0, 0.75), (1.0, -1.0, 1.0), (20.0, 1.0, 0.25)
        zs = [sg[j] * (th[j] - xs[j]) / tau[j] for j in range(J)]
        w = torch.sigmoid(zs[0])
        for z in zs[1:]:
            w = w * torch.sigmoid(z)
        e = d["price"].double() if c["value"] else torch.ones_like(w)
        gid = d["region"].long() * 3 + d["flag"].long()
        S = torch.zeros(75, device=DEV, dtype=torch.float64).index_add_(0, gid, w * e)
        T = d["T"].double()
        t = (2 * (S - T) / 75)[gid] * e * w
        dc = torch.stack([(t * torch.sigmoid(-zs[j])).sum() * sg[j] / tau[j] for j in range(J)])
        dtau = torch.stack([-(t * torch.sigmoid(-zs[j]) * zs[j]).sum() / tau[j] for j in range(J)])
        return {"loss": (S - T).square().mean().view(1), "dc": dc, "dtau": dtau if c["dtau"] else None}
    if k == "llp":
        X, W, b, C, n = d["X"].double(), d["W"].double(), d["b"].double(), c["classes"], c["n"]
        p = torch.softmax(X @ W.t() + b, 1)
        bag = torch.arange(n, device=DEV) // c["bag"]
        T = d["T"].double().view(-1, C)
        S = torch.zeros_like(T).index_add_(0, bag, p)
        dp = (2 * (S - T) / T.numel())[bag]
        dz = p * (dp - (p * dp).sum(1, keepdim=True))
        gW, gb = dz.t() @ X, dz.sum(0)
        lr, eps = float(np.float32(0.05)), float(np.float32(1e-8))
        return {"loss": (S - T).square().mean().view(1), "gW": gW, "gb": gb, "W": W - lr * gW / (gW.abs() + eps),
                "b": b - lr * gb / (gb.abs() + eps)}  # Adam's first step from zero moments
    H, ci, co, B = d["H"], d["ci"], d["co"], c["batch"]
    w = d["w"].double().reshape(co, 9 * ci)
    parts, dw, db = [], torch.zeros_like(w), torch.zeros(co, device=DEV, dtype=torch.float64)
    for lo in range(0, B, 64):
        x = d["x"][lo:lo + 64].double()
        m, o = x.shape[0], H - 2
        col = torch.cat([x[:, i:i + o, j:j + o, :] for i in range(3) for j in range(3)], 3).reshape(m * o * o, 9 * ci)
        if k == "conv_fwd":
            parts.append((col @ w.t() + d["bias"].double()).relu_().view(m, o, o, co))
            continue
        dy = d["dy"][lo:lo + 64].double().reshape(m * o * o, co)
        dw += dy.t() @ col
        db += dy.sum(0)
        dcol = (dy @ w).view(m, o, o, 9, ci)
        dx = torch.zeros_like(x)
        for t in range(9):
            i, j = divmod(t, 3)
            dx[:, i:i + o, j:j + o, :] += dcol[:, :, :, t, :]
        parts.append(torch.where(x > 0, dx, 0.0))
    if k == "conv_fwd":
        return {"y": torch.cat(parts)}
    return {"dx": torch.cat(parts), "dw": dw.view(co, 3, 3, ci), "db": db}
