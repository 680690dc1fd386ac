"""The records of the partitioned probe against the oracle, bit-exact, where
their 32-bit forms end: literals at and beyond the predicate column's range,
key domains at the ends of int32, products and factors that leave int32,
columns of other types (the general kernel), and keys outside their domain."""
import numpy as np
import pytest
import torch

import oracle
from paper_2211_02753_amd import _lib as L
from paper_2211_02753_amd import query as Q

pytestmark = pytest.mark.gpu
I32 = np.iinfo(np.int32)


def t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _cmp(got, want):
    for k in ("k0", "k1", "sum", "count"):
        if k in want:
            assert np.array_equal(got[k].cpu().numpy(), want[k]), k


@pytest.mark.parametrize("n", [3, 4096, 70_001])
@pytest.mark.parametrize("cmp", ["<", "<=", ">", ">=", "==", "!="])
@pytest.mark.parametrize("lit", [-2**40, I32.min, -1, 7, I32.max, 2**40])
def test_static_columns_literals_and_wide_values(n, cmp, lit):
    rng = np.random.default_rng(n)
    pk = rng.permutation(np.arange(-2500, 2500, dtype=np.int32))
    fk = rng.integers(-2600, 2600, n).astype(np.int32)
    p = rng.choice(np.array([I32.min, I32.min + 1, -1, 0, 7, 8, I32.max - 1, I32.max], np.int32), n)
    k0 = rng.integers(-128, -125, n).astype(np.int8)
    k1 = rng.integers(126, 128, n).astype(np.int8)
    a = rng.integers(-2**31, 2**31, n)
    a[n // 2:n // 2 + 300] = rng.integers(-2**40, 2**40, len(a[n // 2:n // 2 + 300]))  # these waves multiply in 64 bits
    b = rng.integers(-3, 4, n)
    b[:2] = [-2**62, 2**62]
    got = Q.GroupbyQuery(n, [Q.Key(t(k0), -128, 3), Q.Key(t(k1), 126, 2)], expr=L.EXPR_MUL_CONST_SUB, a=Q.Operand(t(a)),
                         b=Q.Operand(t(b)), k=100, pred=(t(p), cmp, lit), join=(t(pk), t(fk), True),
                         strategy=L.PROBE_PARTITIONED)()
    want = oracle.query(n, keys=[(k0, 0), (k1, 0)], expr=oracle.EXPR_MUL_CONST_SUB, a=(a, 0), b=(b, 0), K=100,
                        pred=(p, cmp, lit), join=(fk, pk))
    _cmp(got, want)


@pytest.mark.parametrize("lo", [I32.min, -3, I32.max - 6, I32.max - 3])
@pytest.mark.parametrize("wide_key", [False, True])
def test_key_domains_at_the_ends_of_int32(lo, wide_key):
    # the last domain reaches beyond int32, so its keys take the 64-bit form
    n, card = 50_003, 7
    rng = np.random.default_rng(5)
    pk = np.arange(3000, dtype=np.int32)
    fk = rng.integers(0, 4000, n).astype(np.int32)
    key = rng.integers(lo, min(lo + card, I32.max + 1), n).astype(np.int64 if wide_key else np.int32)
    val = rng.integers(-2**33, 2**33, n)
    q = lambda k: Q.GroupbyQuery(n, [Q.Key(t(k), lo, card)], expr=L.EXPR_COL, a=Q.Operand(t(val)),
                                 join=(t(pk), t(fk), True), strategy=L.PROBE_PARTITIONED)
    _cmp(q(key)(), oracle.query(n, keys=[(key, 0)], expr=oracle.EXPR_COL, a=(val, 0), join=(fk, pk)))
    out = key.copy()
    out[n // 3] = I32.max if lo < 0 else I32.min  # outside the domain, also modulo 2**32
    with pytest.raises(Exception, match="KEY_DOMAIN"):
        q(out)()


@pytest.mark.parametrize("lo", [2**63 - 7, 2**63 - 100, -2**63])
@pytest.mark.parametrize("second", [False, True])
def test_key_domains_at_the_ends_of_int64(lo, second):
    """A domain next to the end of int64 holds no int32 key, whatever its
    bounds are modulo 2^32 or 2^64."""
    n, card = 20_003, 7
    rng = np.random.default_rng(6)
    pk = np.arange(3000, dtype=np.int32)
    fk = rng.integers(0, 3000, n).astype(np.int32)
    low = lo & 0xFFFFFFFF  # the domain's first key modulo 2^32
    key = np.full(n, low - (1 << 32) if low >> 31 else low, np.int64).astype(np.int32)
    key += rng.integers(0, card, n).astype(np.int32) if lo < 0 or lo == 2**63 - 7 else 0
    keys = [Q.Key(t(key), lo, card)]
    if second:
        keys = [Q.Key(t(np.zeros(n, np.int8)), 0, 1)] + keys
    q = Q.GroupbyQuery(n, keys, expr=L.EXPR_COL, a=Q.Operand(t(fk.astype(np.int64))), join=(t(pk), t(fk), True),
                       strategy=L.PROBE_PARTITIONED)
    with pytest.raises(Exception, match="KEY_DOMAIN"):
        q()
