"""Hash tables of small build sides built block by block in LDS, tables that
keep a build-side column's values, and the partial rows of the fused
group-by, bit-exact against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2211_02753_amd import _lib as L
from paper_2211_02753_amd import query as Q

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def _same(got, want, n_keys):
    for k in (["k0", "k1"][:n_keys] + ["sum", "count", "avg"]):
        assert np.array_equal(got[k].cpu().numpy(), want[k]), k


# register rows, one-workgroup totals (up to 256 groups) and the two-kernel totals; one row, one workgroup less a
# row, every CU with small workgroups, every CU with large ones, and a second step
@pytest.mark.parametrize("G", [1, 8, 9, 64, 65, 256, 257, 2048])
@pytest.mark.parametrize("n", [1, 1023, 262_143, 262_145, 1_100_003])
def test_partial_rows(G, n):
    rng = np.random.default_rng(G * 31 + n)
    k = rng.integers(0, G, n).astype(np.int32)
    v = rng.integers(-2**62, 2**62, n)  # sums wrap
    print("partial rows", G, n, flush=True)
    got = Q.GroupbyQuery(n, [Q.Key(dev(k), 0, G)], expr=L.EXPR_COL, a=Q.Operand(dev(v)))
    want = oracle.query(n, keys=[(k, 0)], expr=oracle.EXPR_COL, a=(v, 0))
    _same(got(), want, 1)
    _same(got(), want, 1)  # a second call on the same workspace
    top = Q.GroupbyQuery(n, [Q.Key(dev(k), 0, G)], expr=L.EXPR_COL, a=Q.Operand(dev(v)), topk=5)()
    order = np.lexsort((want["k0"], -want["sum"].astype(object)))[:5]
    assert np.array_equal(top["k0"].cpu().numpy(), want["k0"][order])
    assert np.array_equal(top["sum"].cpu().numpy(), want["sum"][order])


# tables added to the dense one and partial rows on both sides of the lines between them, few and many cells
@pytest.mark.parametrize("n", [3001, (128 << 10) - 1, 128 << 10, 192 << 10, (256 << 10) - 1, 256 << 10])
@pytest.mark.parametrize("G", [9, 192, 193, 256, 300])
@pytest.mark.parametrize("join", [False, True])
def test_partial_rows_or_atomics(n, G, join):
    rng = np.random.default_rng(n + G)
    k, v = rng.integers(0, G, n).astype(np.int32), rng.integers(-2**62, 2**62, n)
    bk, pk = rng.permutation(np.arange(5000, dtype=np.int32)), rng.integers(-50, 5050, n).astype(np.int32)
    print("partial rows or atomics", n, G, join, flush=True)
    want = oracle.query(n, keys=[(k, 0)], expr=oracle.EXPR_COL, a=(v, 0), join=(pk, bk) if join else None)
    order = np.lexsort((want["k0"], -want["sum"].astype(object)))[:5]
    dk, dv = dev(k), dev(v)
    for topk in (0, 5):
        q = Q.GroupbyQuery(n, [Q.Key(dk, 0, G)], expr=L.EXPR_COL, a=Q.Operand(dv), topk=topk,
                           join=(dev(bk), dev(pk), True) if join else None)
        for _ in range(2):  # the workspace is left ready
            got = q()
            if topk:
                assert np.array_equal(got["k0"].cpu().numpy(), want["k0"][order])
                assert np.array_equal(got["sum"].cpu().numpy(), want["sum"][order])
            else:
                _same(got, want, 1)


# one row, one probing block, several, the last direct build and the first bucketed one
@pytest.mark.parametrize("nb", [1, 2047, 2049, 10_000, 65_535, 65_536])
@pytest.mark.parametrize("mode", ["keys", "i8", "i32", "value", "i64", "two", "agg", "aggcount"])
def test_small_build_sides(nb, mode):
    rng = np.random.default_rng(nb + len(mode))
    n = 50_001
    pool = rng.permutation(np.concatenate([[-2**31, 2**31 - 1, 0], rng.integers(-2**31, 2**31, 2 * nb + 10)]))
    pool = np.unique(pool)
    pool = rng.permutation(pool)
    uniq = pool[:nb].astype(np.int32)
    if -2**31 not in uniq:
        uniq[0] = -2**31
    bk = uniq if not mode.startswith("agg") else uniq[rng.integers(0, max(1, nb // 3), nb)]
    pk = np.where(rng.random(n) < 0.8, uniq[rng.integers(0, nb, n)], pool[rng.integers(0, len(pool), n)]).astype(np.int32)
    g = rng.integers(0, 30, n).astype(np.int32)
    v = rng.integers(-2**40, 2**40, n)
    b8, b32 = rng.integers(0, 25, nb).astype(np.int8), rng.integers(0, 25, nb).astype(np.int32)
    bv = rng.integers(-2**31, 2**31, nb).astype(np.int32)  # every 32-bit value
    b64 = rng.integers(-2**40, 2**40, nb)
    col, none = oracle.EXPR_COL, oracle.EXPR_NONE
    P, B = 0, 1
    keys, expr, a = {"keys": ([(g, P, 30)], col, (v, P)), "i8": ([(b8, B, 25), (g, P, 30)], col, (v, P)),
                     "i32": ([(g, P, 30), (b32, B, 25)], none, None), "value": ([(g, P, 30)], col, (bv, B)),
                     "i64": ([(g, P, 30)], col, (b64, B)), "two": ([(b8, B, 25), (b32, B, 25)], col, (v, P)),
                     "agg": ([(g, P, 30)], col, (b64, B)), "aggcount": ([(g, P, 30)], none, None)}[mode]
    unique = not mode.startswith("agg")
    print("small build", nb, mode, flush=True)
    d = {id(x): dev(x) for x in (g, v, b8, b32, bv, b64)}
    for load in (0, 90):
        got = Q.GroupbyQuery(n, [Q.Key(d[id(c)], 0, card, L.BUILD if s else L.PROBE) for c, s, card in keys],
                             expr=L.EXPR_COL if expr == col else L.EXPR_NONE,
                             a=None if a is None else Q.Operand(d[id(a[0])], L.BUILD if a[1] else L.PROBE),
                             join=(dev(bk), dev(pk), unique, load))()
        want = oracle.query(n, keys=[(c, s) for c, s, _ in keys], expr=expr, a=a, join=(pk, bk))
        _same(got, want, len(keys))


# the last direct and the first memory build of each kind, by rows and by slots (load), the longest key list; distinct
# keys, keys held by many rows, and many rows of the key kept outside the blocks
@pytest.mark.parametrize("nb", [8192, 8193, 16_385, 65_535])
@pytest.mark.parametrize("load", [0, 90])
@pytest.mark.parametrize("mode", ["keys", "value", "agg", "hot", "empty", "count"])
def test_small_build_forms(nb, load, mode):
    rng = np.random.default_rng(nb + load)
    n = 30_011
    pool = np.unique(np.concatenate([[-2**31], rng.integers(-2**31, 2**31, 2 * nb)])).astype(np.int32)
    uniq = rng.permutation(pool)[:nb]
    if mode in ("keys", "value"):
        bk = uniq
    else:
        bk = uniq[rng.integers(0, nb // 5, nb)]
        if mode != "agg":
            bk[rng.random(nb) < 0.5] = -2**31 if mode == "empty" else uniq[0]
    pk = np.where(rng.random(n) < 0.9, bk[rng.integers(0, nb, n)], pool[rng.integers(0, len(pool), n)]).astype(np.int32)
    g, v = rng.integers(0, 30, n).astype(np.int32), rng.integers(-2**40, 2**40, n)
    b32 = rng.integers(-2**31, 2**31, nb).astype(np.int32)
    print("build form", nb, load, mode, flush=True)
    a = {"keys": (v, 0), "count": None}.get(mode, (b32, 1))
    q = Q.GroupbyQuery(n, [Q.Key(dev(g), 0, 30)], expr=L.EXPR_NONE if a is None else L.EXPR_COL,
                       a=None if a is None else Q.Operand(dev(a[0]), L.BUILD if a[1] else L.PROBE),
                       join=(dev(bk), dev(pk), mode in ("keys", "value"), load))
    want = oracle.query(n, keys=[(g, 0)], expr=oracle.EXPR_NONE if a is None else oracle.EXPR_COL, a=a, join=(pk, bk))
    _same(q(), want, 1)
    _same(q(), want, 1)


# the largest table that keeps a column's values and the next one, which keeps row ids
@pytest.mark.parametrize("nb", [(1 << 23) - 1, (1 << 23) + 1])
@pytest.mark.parametrize("dtype", [torch.int8, torch.int32])
def test_values_in_large_tables(nb, dtype):
    n = 300_001
    pk = torch.randperm(nb, device=DEV)
    value = torch.randint(0, 100, (nb,), device=DEV).to(dtype)
    key, amount = torch.randint(0, nb + 1000, (n,), device=DEV), torch.randint(-2**40, 2**40, (n,), device=DEV)
    print("values in large tables", nb, dtype, flush=True)
    got = Q.GroupbyQuery(n, [Q.Key(value, 0, 100, L.BUILD)], expr=L.EXPR_COL, a=Q.Operand(amount),
                         join=(pk.to(torch.int32), key.to(torch.int32), True))()
    row = torch.empty_like(pk)
    row[pk] = torch.arange(nb, device=DEV)
    on = key < nb
    g = value[row[key[on]]].long()
    count = torch.zeros(100, dtype=torch.int64, device=DEV).index_add_(0, g, torch.ones_like(g))
    total = torch.zeros(100, dtype=torch.int64, device=DEV).index_add_(0, g, amount[on])
    assert torch.equal(got["count"], count) and torch.equal(got["sum"], total)


def test_small_build_flags():
    n = 1000
    pk = dev(np.arange(n, dtype=np.int32))
    g = dev(np.zeros(n, np.int32))
    dup = np.arange(5000, dtype=np.int32)
    dup[4999] = 17
    with pytest.raises(L.TdpError, match="DUP_BUILD"):
        Q.GroupbyQuery(n, [Q.Key(g, 0, 1)], join=(dev(dup), pk, True))()
    twice = np.arange(5000, dtype=np.int32)
    twice[[3, 4]] = -2**31  # the key kept outside the blocks
    with pytest.raises(L.TdpError, match="DUP_BUILD"):
        Q.GroupbyQuery(n, [Q.Key(g, 0, 1)], join=(dev(twice), pk, True))()
    with pytest.raises(L.TdpError, match="TABLE_FULL"):  # 30,000 distinct keys against a bound of 1000
        Q.GroupbyQuery(n, [Q.Key(g, 0, 1)], join=(dev(np.arange(30_000, dtype=np.int32)), pk, False, 0, 1000))()
    # an empty build side, then a full one on a fresh plan
    r = Q.GroupbyQuery(n, [Q.Key(g, 0, 1)], join=(dev(np.zeros(0, np.int32)), pk, True))()
    assert r["k0"].numel() == 0


# one tile a workgroup, the first second tile, a workgroup whose last tile is one row
@pytest.mark.parametrize("n", [1 << 20, (512 << 12) + 1, (512 << 12) + 4097])
@pytest.mark.parametrize("G", [2049, 4097, 1_000_000])
def test_partitioned_aggregation_tiles(n, G):
    rng = np.random.default_rng(n + G)
    k = rng.integers(-5, G - 5, n).astype(np.int32)
    v = rng.integers(-2**62, 2**62, n)
    day = rng.integers(0, 100, n).astype(np.int32)
    print("partitioned aggregation", n, G, flush=True)
    got = Q.GroupbyQuery(n, [Q.Key(dev(k), -5, G)], expr=L.EXPR_COL, a=Q.Operand(dev(v)), pred=(dev(day), "<", 37))
    want = oracle.query(n, keys=[(k, 0)], expr=oracle.EXPR_COL, a=(v, 0), pred=(day, "<", 37))
    _same(got(), want, 1)
    _same(got(), want, 1)


# whole tiles of one partition, runs of tiles that differ by one between workgroups, a join whose rows partly miss
@pytest.mark.parametrize("tiles", [511, 513, 700])
def test_partitioned_aggregation_sorted_groups(tiles):
    n, G = (tiles << 12) - 5, 70_001
    rng = np.random.default_rng(tiles)
    k = np.sort(rng.integers(0, G, n)).astype(np.int32)
    bk = np.repeat(np.arange(0, 3000, dtype=np.int32), 3)
    bv, pk = rng.integers(-2**40, 2**40, len(bk)), rng.integers(0, 4000, n).astype(np.int32)
    v = rng.integers(-2**20, 2**20, n)
    print("partitioned aggregation, sorted groups", tiles, flush=True)
    got = Q.GroupbyQuery(n, [Q.Key(dev(k), 0, G)], expr=L.EXPR_MUL, a=Q.Operand(dev(v)),
                         b=Q.Operand(dev(bv), L.BUILD), join=(dev(bk), dev(pk), False))
    want = oracle.query(n, keys=[(k, 0)], expr=oracle.EXPR_MUL, a=(v, 0), b=(bv, 1), join=(pk, bk))
    _same(got(), want, 1)
    _same(got(), want, 1)


# every comparison with literals at, beside and beyond the ends of the column's type, outputs that start at each
# position of a 16-byte unit, tiles that end inside a lane's group of rows
@pytest.mark.parametrize("dtype", [np.int8, np.int32, np.int64])
@pytest.mark.parametrize("n", [3, 1023, 16_383, 49_153, 200_003])
def test_filter_literals_and_alignment(dtype, n):
    import ctypes as C
    rng = np.random.default_rng(n)
    info = np.iinfo(dtype)
    col = rng.integers(info.min, info.max, n, dtype=dtype, endpoint=True)
    col[rng.integers(0, n, 5)] = info.min
    col[rng.integers(0, n, 5)] = info.max
    d = dev(col)
    lib, s = L.load(), L.stream_handle(torch.device(DEV))
    ws = L.workspace(lib.tdp_filter_workspace_size(n), DEV)
    tail = torch.zeros(2, dtype=torch.int64, device=DEV)
    lits = [info.min, info.min + 1, 0, int(col[0]), info.max - 1, info.max]
    if dtype != np.int64:
        lits += [info.min - 1, info.max + 1, -2**63, 2**63 - 1]
    print("filter", dtype.__name__, n, flush=True)
    for k, op in enumerate(["<", "<=", ">", ">=", "==", "!="]):
        for i, lit in enumerate(lits):
            out = torch.full((n + 8,), -7, dtype=torch.int32, device=DEV)
            dst = out[(k + i) % 4:]
            c = L.col(d)
            L.check("filter", lib.tdp_filter(C.byref(c), L.CMP[op], int(lit), None, 0, L.ptr(dst), n, L.ptr(tail),
                                             L.ptr(tail[1:]), L.ptr(ws), ws.numel(), s))
            m = int(tail[0])
            x = col.astype(object)
            want = np.nonzero({"<": x < lit, "<=": x <= lit, ">": x > lit, ">=": x >= lit, "==": x == lit,
                               "!=": x != lit}[op].astype(bool))[0]
            got = out.cpu().numpy()
            at = (k + i) % 4
            assert m == len(want) and np.array_equal(got[at:at + m], want), (op, lit)
            assert np.all(got[:at] == -7) and np.all(got[at + m:] == -7), (op, lit)  # nothing beside the survivors
