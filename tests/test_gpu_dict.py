"""Dictionary-encoded string columns on the GPU: the dictionary and the codes
bit-exact against the oracle, lookup and decode, and the codes as keys of
the exact filter, join and group-by against the oracle's query over the
oracle's codes."""
import numpy as np
import pytest
import torch

import oracle
import tdp_datagen as gen
from paper_2211_02753_amd import _lib as L
from paper_2211_02753_amd import dictenc
from paper_2211_02753_amd import query as Q

pytestmark = pytest.mark.gpu
DEV = "cuda"


def t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


@pytest.mark.parametrize("n,nd,width", [(1, 1, 4), (1000, 37, 8), (1_000_003, 50_000, 16), (300_001, 150_000, 32)])
def test_dictionary_build_matches_oracle(n, nd, width):
    rows, _ = gen.string_column(n, nd, width)
    print(f"dictionary n={n} distinct={nd} width={width}", flush=True)
    d, codes = dictenc.encode(t(rows), max_distinct=nd)
    wd, wc = oracle.dict_build(rows)
    assert np.array_equal(d.cpu().numpy(), wd)
    assert np.array_equal(codes.cpu().numpy(), wc)
    assert np.array_equal(dictenc.decode(d, codes).cpu().numpy(), rows)


def test_dictionary_edges_lookup_and_capacity_flag():
    # empty strings, full-width strings, a single distinct string
    words = [b"", b"abcdefgh", b"", b"abcdefgh", b"abcdefg", b"b"]
    rows = dictenc.pad(words, 8).numpy()
    d, codes = dictenc.encode(t(rows))
    wd, wc = oracle.dict_build(rows)
    assert np.array_equal(d.cpu().numpy(), wd) and np.array_equal(codes.cpu().numpy(), wc)
    same = dictenc.pad([b"same"] * 5000, 4).numpy()
    d1, c1 = dictenc.encode(t(same), max_distinct=1)
    assert d1.shape[0] == 1 and int(c1.max()) == 0
    # lookup of present and absent strings
    probe = dictenc.pad([b"", b"a", b"abcdefg", b"abcdefgh", b"abcdefgi", b"zzzz"], 8).numpy()
    pos, found = dictenc.lookup(d, t(probe))
    wp, wf = oracle.dict_lookup(wd, probe)
    assert np.array_equal(pos.cpu().numpy(), wp) and np.array_equal(found.cpu().numpy(), wf)
    # more distinct strings than the bound: the flag
    rows2, _ = gen.string_column(20_000, 5000, 8)
    with pytest.raises(L.TdpError, match="TABLE_FULL"):
        dictenc.encode(t(rows2), max_distinct=1000)


def test_codes_as_keys_of_filter_join_and_groupby():
    """SELECT city, SUM(amount), COUNT(*) FROM sales JOIN stores ON sales.store = stores.store
    WHERE city >= 'm' GROUP BY city, with city and store names dictionary-encoded."""
    rng = np.random.default_rng(4)
    n = 400_003
    store_names, _ = gen.string_column(3000, 3000, 12, seed=gen.SEED_STR + 1)
    store_names = np.unique(store_names.view("S12").ravel()).view(np.uint8).reshape(-1, 12)
    cities, _ = gen.string_column(len(store_names), 120, 8, seed=gen.SEED_STR + 2)
    pick = rng.integers(0, len(store_names) + 200, n)   # some sales name stores that do not exist
    others, _ = gen.string_column(200, 200, 12, seed=gen.SEED_STR + 3)
    sale_store = np.where(pick[:, None] < len(store_names), store_names[np.minimum(pick, len(store_names) - 1)],
                          others[np.maximum(pick - len(store_names), 0) % len(others)])
    amount = rng.integers(1, 10_000, n).astype(np.int64)
    # encode: store names through the stores' dictionary, sales looked up in it
    sd, scode = dictenc.encode(t(store_names))
    spos, sfound = dictenc.lookup(sd, t(sale_store))
    sale_code = torch.where(sfound.bool(), spos, torch.full_like(spos, -1)).contiguous()
    cd, ccode = dictenc.encode(t(cities))
    op, lit = dictenc.literal_predicate(cd, ">=", b"m")
    # city per sale comes from the store (build side), so the filter applies after the join:
    # express it as a filter on the build side's city codes, then the join and group-by
    keep = Q.filter(ccode, op, lit)
    build_keys = scode[keep.long()].contiguous()
    build_city = ccode[keep.long()].contiguous()
    got = Q.GroupbyQuery(n, [Q.Key(build_city, 0, cd.shape[0], L.BUILD)], expr=L.EXPR_COL, a=Q.Operand(t(amount)),
                         join=(build_keys, sale_code, True))()
    # oracle: the same query over the oracle's codes, then keys decoded to strings
    od_s, oc_s = oracle.dict_build(store_names)
    od_c, oc_c = oracle.dict_build(cities)
    opos, ofound = oracle.dict_lookup(od_s, sale_store)
    osale = np.where(ofound == 1, opos, -1).astype(np.int32)
    city_str = [bytes(r).rstrip(b"\0") for r in cities]
    kept = np.array([i for i, c in enumerate(city_str) if c >= b"m"], np.int32)
    want = oracle.query(n, keys=[(oc_c[kept], 1)], expr=oracle.EXPR_COL, a=(amount, 0),
                        join=(osale, oc_s[kept].astype(np.int32)))
    assert np.array_equal(got["k0"].cpu().numpy(), want["k0"])
    assert np.array_equal(got["sum"].cpu().numpy(), want["sum"])
    assert np.array_equal(got["count"].cpu().numpy(), want["count"])
    names = dictenc.decode(cd, got["k0"].to(torch.int32).contiguous()).cpu().numpy()
    assert all(bytes(r).rstrip(b"\0") >= b"m" for r in names)
    assert np.array_equal(names, od_c[want["k0"]])


def _distinct_words(rng, nd, width, prefix):
    """nd distinct zero-padded strings (the empty one first) whose first `prefix` bytes are alike."""
    rows = np.full((nd, width), ord("p"), np.uint8)
    ids = rng.permutation(nd)
    for k in range(prefix, width):  # base-25 digits of a distinct number, then nothing
        rows[:, k] = ord("a") + ids % 25 if 25 ** (k - prefix) < 4 * nd else 0
        ids = ids // 25
    rows[0] = 0
    return rows


# tile and merge edges of the sort (tiles of 1024, 16 runs a merge), strings that differ only behind the first
# 8 bytes, rows that repeat at least 8 times (string copies by slot) and rows that do not
@pytest.mark.parametrize("nd,n,width,prefix", [(1023, 1023, 4, 0), (1024, 2000, 8, 4), (1025, 9000, 12, 8),
                                                (16384, 140_001, 16, 9), (16385, 20_000, 20, 8),
                                                (17_000, 136_000, 24, 12), (33_000, 300_007, 32, 24)])
@pytest.mark.parametrize("shift", [0, 4])  # a column that starts 4 bytes past a 16-byte boundary
def test_dictionary_build_sort_and_repeat_edges(nd, n, width, prefix, shift):
    rng = np.random.default_rng(nd + width)
    words = _distinct_words(rng, nd, width, prefix)
    rows = words[rng.permutation(np.arange(n) % nd)]
    print(f"dictionary n={n} distinct={nd} width={width} prefix={prefix} shift={shift}", flush=True)
    buf = torch.zeros(n * width + shift, dtype=torch.uint8, device=DEV)
    col = buf[shift:].view(n, width)
    col.copy_(t(rows))
    d, codes = dictenc.encode(col, max_distinct=nd)
    wd, wc = oracle.dict_build(rows)
    assert np.array_equal(d.cpu().numpy(), wd)
    assert np.array_equal(codes.cpu().numpy(), wc)


def test_dictionary_over_its_bound_with_repeated_rows_raises_the_flag():
    words = _distinct_words(np.random.default_rng(9), 40_000, 16, 4)
    rows = words[np.random.default_rng(10).integers(0, 40_000, 200_000)]
    with pytest.raises(L.TdpError, match="TABLE_FULL"):
        dictenc.encode(t(rows), max_distinct=5000)


def _base26(v, width, prefix):
    """Rows of `prefix` letters 'q' and then v in `width - prefix` base-26 letters: they order as v does."""
    out = torch.full((len(v), width), ord("q"), dtype=torch.uint8, device=DEV)
    for k in range(width - 1, prefix - 1, -1):
        out[:, k] = (v % 26 + ord("a")).to(torch.uint8)
        v = v // 26
    return out


# three levels of merges with strings at every one, and more strings than one step of the merge's workgroups takes;
# strings that differ in their first, second and last word pair
@pytest.mark.parametrize("n,width,prefix", [(300_001, 8, 0), (300_001, 12, 6), (2_200_003, 16, 8), (2_200_003, 32, 25)])
def test_dictionary_of_many_strings(n, width, prefix):
    v = torch.randperm(n, device=DEV)
    strs = _base26(v, width, prefix)
    print("many strings", n, width, flush=True)
    d, codes = dictenc.encode(strs)
    assert d.shape[0] == n and torch.equal(codes.long(), v)
    assert torch.equal(d, _base26(torch.arange(n, device=DEV), width, prefix))


def test_dictionary_of_a_bound_above_2_to_the_30():
    """A column of more than 2^30 rows without a bound of its own: the table's slots stay int32, the merge's grid
    within a launch's limit."""
    n, nd = (1 << 30) + 1001, 250
    if torch.cuda.mem_get_info()[0] < 170 << 30:
        pytest.skip("needs 170 GiB of device memory")
    words = _base26(torch.arange(nd, device=DEV), 4, 1)
    pick = torch.randint(0, nd, (n,), dtype=torch.uint8, device=DEV)
    strs = torch.empty((n, 4), dtype=torch.uint8, device=DEV)
    for i in range(0, n, 1 << 27):
        strs[i:i + (1 << 27)] = words[pick[i:i + (1 << 27)].long()]
    print("bound above 2^30", flush=True)
    d, codes = dictenc.encode(strs)
    assert torch.equal(d, words)
    assert all(torch.equal(codes[i:i + (1 << 27)], pick[i:i + (1 << 27)].int()) for i in range(0, n, 1 << 27))
    del strs, codes, pick, d
    torch.cuda.empty_cache()


# no merge before the last, one and two of them; buffers that start 4 bytes off a 16-byte unit, odd word counts
@pytest.mark.parametrize("n,bound", [(900, 0), (20_000, 0), (20_000, 16_385), (300_007, 290_000)])
@pytest.mark.parametrize("width", [4, 12, 20, 28, 32])
def test_dictionary_buffer_beyond_the_strings(n, bound, width):
    """The rows of the dictionary's buffer behind the last string stay as they were."""
    nd = min(n // 2, 14_000, 26 ** 3 - 1) if width == 4 else n // 2 if bound != 16_385 else 16_000
    v = torch.randint(0, nd, (n,), device=DEV)
    v[:nd] = torch.randperm(nd, device=DEV)
    strs = _base26(v, width, 1)
    md = bound or n
    lib, s = L.load(), L.stream_handle(torch.device("cuda:0"))
    buf = torch.full((4 + md * width + 4,), 0xEE, dtype=torch.uint8, device=DEV)
    dic, codes = buf[4:], torch.empty(n, dtype=torch.int32, device=DEV)
    cnt, st = torch.zeros(1, dtype=torch.int64, device=DEV), torch.zeros(1, dtype=torch.int32, device=DEV)
    ws = L.workspace(lib.tdp_dict_build_workspace_size(n, bound), DEV)
    print("dictionary buffer", n, bound, width, flush=True)
    L.check("dict", lib.tdp_dict_build(L.ptr(strs), n, width, bound, L.ptr(dic), L.ptr(cnt), L.ptr(codes), L.ptr(st),
                                       L.ptr(ws), ws.numel(), s))
    assert int(cnt) == nd and int(st) == 0
    assert torch.equal(codes.long(), v)
    assert torch.equal(dic[:nd * width].view(nd, width), _base26(torch.arange(nd, device=DEV), width, 1))
    assert bool((buf[:4] == 0xEE).all()) and bool((dic[nd * width:] == 0xEE).all())


# columns whose rows are copied from a sample: sizes at the ends of its units and groups, strings that only one row
# holds, orders that show the sample one string, half of them, all of them, runs of them, or the same rows again
@pytest.mark.parametrize("n", [1 << 17, (1 << 17) + 1, (1 << 17) + 127, (1 << 17) + 129, 200_003])
@pytest.mark.parametrize("order", ["sorted", "one", "halves", "cycle", "random"])
def test_dictionary_of_repeating_rows(n, order):
    nd, width = 4096, 12
    at = torch.arange(n, device=DEV)
    rnd = torch.randint(0, nd - 2, (n,), device=DEV)
    v = {"sorted": at * (nd - 2) // n, "one": torch.where(at < n // 2, 0, rnd), "cycle": at % 2048, "random": rnd,
         "halves": torch.where(at < n // 2, rnd // 2, rnd // 2 + nd // 2 - 2)}[order]
    v[-1], v[n // 3] = nd - 1, nd - 2  # one row each, the last one among them
    want, codes_want = torch.unique(v, return_inverse=True)
    print("repeating rows", n, order, flush=True)
    d, codes = dictenc.encode(_base26(v, width, 5), max_distinct=nd)
    assert torch.equal(d, _base26(want, width, 5))
    assert torch.equal(codes.long(), codes_want)
