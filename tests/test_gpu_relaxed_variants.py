"""The relaxed query's and the label-proportion kernels' variants (conjuncts,
column types, key domains, table copies; classes, features, bag sizes)
against the float64 oracle, within 1e-5 of the terms' magnitude."""
import ctypes as C

import numpy as np
import pytest
import torch
from scipy.special import expit

import oracle
from paper_2211_02753_amd import _lib as L
from paper_2211_02753_amd import llp
from paper_2211_02753_amd import query as Q
from paper_2211_02753_amd import trainable as TR
from paper_2211_02753_amd.soft import soft_workspace

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
I8, I32, I64, F32 = np.int8, np.int32, np.int64, np.float32


def t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


# conjunct types, key types and lower bounds (32-bit keys at both ends of their range, a bound past it), value type,
# rows (tails of 1 to 3, one and several workgroups), groups (copies per lane, per wave, one)
@pytest.mark.parametrize("preds,keys,value,n,card", [
    ([], [(I8, -3)], None, 5, 3), ([F32], [(I32, -2**31)], None, 4098, 7), ([I32], [(I32, 2**31 - 1 - 65537), (I8, 0)], F32, 40_003, 9),
    ([I32], [(I32, 2**31 - 65536)], I32, 9_001, 40), ([I8, F32], [(I8, -128), (I8, -1)], I8, 70_001, 5),
    ([I32, I32], [(I32, 5)], None, 270_005, 1000), ([I32, I8, F32], [(I8, 0), (I32, 100)], I32, 33_333, 25),
    ([F32, I32, I8, I32], [(I32, 0)], F32, 100_001, 2000), ([I64, F32], [(I32, 0)], None, 50_003, 30),
    ([F32], [(I64, 2**40), (I8, 0)], I64, 50_001, 6), ([I32], [(I32, 0)], I64, 20_002, 12)])
def test_soft_query_variants(preds, keys, value, n, card):
    rng = np.random.default_rng(n + len(preds))
    khost = [(rng.integers(lo, min(lo + card, np.iinfo(dt).max + 1), n).astype(dt), lo, card) for dt, lo in keys]
    xs = [rng.standard_normal(n).astype(F32) if dt == F32 else rng.integers(-100, 100, n).astype(dt) for dt in preds]
    ops = ["<", ">=", "<=", ">"][:len(preds)]
    c = [0.25 if dt == F32 else 10.5 for dt in preds]
    taus = [0.5 if dt == F32 else 12.0 for dt in preds]
    v = None if value is None else (rng.standard_normal(n).astype(F32) if value == F32
                                    else rng.integers(-100, 100, n).astype(value))
    print("soft query", [p.__name__ for p in preds], keys, value, n, card, flush=True)
    q = TR.TrainableQuery(n, [Q.Key(t(k), lo, card) for k, lo, card in khost],
                          [TR.Where(t(x), o, th) for x, o, th in zip(xs, ops, c)], value=None if v is None else t(v),
                          tau=taus if preds else 1.0)
    gid = oracle.group_ids(khost)
    plan = q.compile(trainable=True)
    S = plan().cpu().numpy().astype(np.float64)
    w = np.ones(n)
    zs = [(1.0 if o in ("<", "<=") else -1.0) * (th - x.astype(np.float64)) / ta for x, o, th, ta in zip(xs, ops, c, taus)]
    for z in zs:
        w = w * expit(z)
    e = np.ones(n) if v is None else v.astype(np.float64)
    want = oracle.soft_where(xs, ops, c, taus, v, gid, q.G) if preds else np.bincount(gid, e, q.G)
    scale = np.bincount(gid, np.abs(w * e), q.G)
    assert np.all(np.abs(S - want) <= 1e-5 * np.max(scale))
    dS = rng.standard_normal(q.G).astype(F32)
    J = len(preds)
    out = [torch.zeros(max(J, 1), dtype=torch.float32, device=DEV) for _ in range(3)]
    de = torch.empty(n, dtype=torch.float32, device=DEV)
    ws, dSd, s = soft_workspace(DEV), t(dS), L.stream_handle(torch.device(DEV))
    args = (C.byref(plan.desc), L.ptr(q.c) if J else None, L.ptr(q.tau) if J else None, L.ptr(dSd))
    lib = L.load()
    L.check("bwd", lib.tdp_soft_query_bwd(*args, L.ptr(out[0]), L.ptr(out[1]), L.ptr(de), L.ptr(ws), ws.numel(), s))
    L.check("bwd", lib.tdp_soft_query_bwd(*args, L.ptr(out[2]), None, None, L.ptr(ws), ws.numel(), s))
    base = dS.astype(np.float64)[gid]
    assert np.max(np.abs(de.cpu().numpy() - base * w)) <= 1e-5 * np.max(np.abs(base * w))
    if not J:
        return
    wdc, wdt, _ = oracle.soft_where_bwd(xs, ops, c, taus, v, gid, dS.astype(np.float64))
    got = [o.cpu().numpy() for o in out]
    for j in range(J):
        b = np.abs(base * e * w) * expit(-zs[j]) / taus[j]
        assert abs(got[0][j] - wdc[j]) <= 1e-5 * b.sum() + 1e-30
        assert abs(got[1][j] - wdt[j]) <= 1e-5 * (b * np.abs(zs[j])).sum() + 1e-30
        assert got[2][j] == got[0][j]  # without the temperatures' gradient


# int64 columns beside each other type, one to four conjuncts, tails of 1 to 3 rows, groups beyond the LDS tables
@pytest.mark.parametrize("preds,keys,value,n,card", [
    ([], [(I64, -2**62)], I64, 4099, 7), ([I64], [(I8, 0)], F32, 9_002, 5), ([I64, I8], [(I64, 2**62)], I32, 30_001, 11),
    ([I64, F32, I32], [(I32, 3)], I8, 50_003, 25), ([I8, I64, I32, F32], [(I64, 0), (I8, -3)], None, 33_333, 6),
    ([I32, F32], [(I32, 0), (I64, -5)], I64, 70_001, 200), ([I64, I64, F32], [(I32, 0), (I32, 7)], F32, 20_002, 200)])
def test_soft_query_wide_columns(preds, keys, value, n, card):
    test_soft_query_variants(preds, keys, value, n, card)


# every class count and both feature builds, each kind of bag (one row, folds of units alone, of classes too, a whole
# wave, several rows a lane), with last bags and last waves that are short
@pytest.mark.parametrize("bag", [1, 2, 4, 16, 32, 64, 128, 256])
@pytest.mark.parametrize("n,F,classes", [(63, 1, 2), (16_449, 8, 2), (16_385, 9, 3), (33_001, 16, 4), (70_003, 6, 4)])
def test_llp_variants(n, F, classes, bag):
    rng = np.random.default_rng(n + bag)
    X = rng.standard_normal((n, F)).astype(F32)
    W = (rng.standard_normal((classes, F)) * 0.7).astype(F32)
    b = (rng.standard_normal(classes) * 0.3).astype(F32)
    print("llp", n, F, classes, bag, flush=True)
    m = llp.LinearLLP(t(W), t(b))
    want = oracle.llp_forward(X, W.astype(np.float64), b.astype(np.float64), bag)
    T = (want + rng.standard_normal(want.shape)).astype(F32)
    S, dS = torch.empty(want.size, device=DEV), torch.empty(want.size, device=DEV)
    m.bag_counts(t(X), bag, S, t(T.reshape(-1)), dS)
    assert np.max(np.abs(S.cpu().numpy().reshape(want.shape) - want)) <= 1e-5 * np.max(want)
    Sf = S.cpu().numpy().astype(np.float64).reshape(want.shape)  # the loss and its gradient follow the counts given out
    wl = np.mean((Sf - T) ** 2)
    assert abs(m.loss.item() - wl) <= 1e-6 * wl
    assert np.max(np.abs(dS.cpu().numpy().reshape(want.shape) - 2 * (Sf - T) / want.size)) <= 1e-6 * np.max(np.abs(Sf - T)) / want.size
    g = rng.standard_normal(want.shape).astype(F32)
    gW, gb = m.bag_counts_bwd(t(X), bag, t(g.reshape(-1)))
    wW, wb = oracle.llp_backward(X, W.astype(np.float64), b.astype(np.float64), bag, g.astype(np.float64))
    p = oracle.llp_forward(X, W.astype(np.float64), b.astype(np.float64), 1)
    dp = np.repeat(g.astype(np.float64), bag, axis=0)[:n]
    dz = np.abs(p * (dp - (p * dp).sum(1, keepdims=True)))
    assert np.all(np.abs(gW.cpu().numpy() - wW) <= 1e-5 * (dz.T @ np.abs(X.astype(np.float64))) + 1e-30)
    assert np.all(np.abs(gb.cpu().numpy() - wb) <= 1e-5 * dz.sum(0) + 1e-30)


# workgroups of the segmented probability counts: one group per wave, groups looped over at the least and the most
# workgroups and between
@pytest.mark.parametrize("groups,rows", [(16_383, 1), (16_385, 3), (150_001, 11), (131_073, 65)])
def test_segmented_counts_over_many_groups(groups, rows):
    from paper_2211_02753_amd import soft
    rng = np.random.default_rng(groups)
    lens = rng.integers(max(rows - 1, 1), rows + 2, groups)
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(I64)
    n = int(seg[-1])
    p, q = rng.random((n, 2), dtype=F32), rng.random((n, 1), dtype=F32)
    d = rng.standard_normal((groups, 2)).astype(F32)
    print("segmented counts", groups, n, flush=True)
    st = torch.zeros(1, dtype=torch.int32, device=DEV)
    S = soft.soft_pe_groupby(t(p), t(q), t(seg), groups, status=st).cpu().numpy().reshape(groups, 2)
    assert int(st.item()) == 0
    want = np.add.reduceat(p.astype(np.float64) * q, seg[:-1], axis=0)
    assert np.all(np.abs(S - want) <= 1e-5 * want + 1e-30)
    dp, dq = soft.soft_pe_groupby_bwd(t(p), t(q), t(seg), t(d.reshape(groups, 2, 1)))
    dr = np.repeat(d.astype(np.float64), lens, axis=0)
    assert np.all(np.abs(dp.cpu().numpy() - dr * q) <= 1e-6 * np.abs(dr * q))
    assert np.all(np.abs(dq.cpu().numpy()[:, 0] - (dr * p).sum(1)) <= 1e-6 * np.abs(dr * p).sum(1))


# one group per wave with 64 rows a wave at least (ten and two probabilities), backward only, waves that loop over the
# groups (the wide kernels), and many small groups
@pytest.mark.parametrize("groups,rows,k1,k2", [(40_001, 50, 10, 2), (40_001, 50, 6, 1), (20_003, 40, 5, 4),
                                               (70_001, 20, 3, 2)])
def test_segmented_counts_grids(groups, rows, k1, k2):
    from paper_2211_02753_amd import soft
    rng = np.random.default_rng(groups + k1)
    lens = rng.integers(rows - 3, rows + 4, groups)
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(I64)
    n = int(seg[-1])
    p, q = rng.random((n, k1), dtype=F32), rng.random((n, k2), dtype=F32)
    d = rng.random((groups, k1, k2), dtype=F32)
    print("segmented grids", groups, rows, k1, k2, flush=True)
    st = torch.zeros(1, dtype=torch.int32, device=DEV)
    S = soft.soft_pe_groupby(t(p), t(q), t(seg), groups, status=st).cpu().numpy()
    assert int(st.item()) == 0
    dp, dq = (x.cpu().numpy() for x in soft.soft_pe_groupby_bwd(t(p), t(q), t(seg), t(d)))
    p, q, d = p.astype(np.float64), q.astype(np.float64), d.astype(np.float64)
    for a in range(k1):
        for b in range(k2):
            want = np.add.reduceat(p[:, a] * q[:, b], seg[:-1])
            assert np.all(np.abs(S[:, a, b] - want) <= 1e-6 * want)
    dr = np.repeat(d, lens, axis=0)
    want = np.matmul(dr, q[:, :, None])[:, :, 0]
    assert np.all(np.abs(dp - want) <= 1e-6 * want)
    want = np.matmul(p[:, None, :], dr)[:, 0]
    assert np.all(np.abs(dq - want) <= 2e-6 * want)
