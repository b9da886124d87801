"""The sizes at which a kernel changes its shape: edges of tiles and units,
remainders, and both sides of each rule that picks a variant.  Integers are
compared with the CPU oracle bit for bit, averages within 1e-12 relative."""
import numpy as np
import pytest
import torch

import oracle
import paper_2506_09226_amd as gq

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = gq.Context(0)
    yield c
    c.close()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# 512-row units up to 2^17 rows; 1024-row units above, of 1..16 steps per wave
@pytest.mark.parametrize("n", [255, 257, 131_072, 131_073, 1_048_575, 2 * 1024 * 512 + 1, 17 * 1024 * 512 + 777])
@pytest.mark.parametrize("lf", [0.5, 0.9])
def test_ordered_probe_units(ctx, n, lf):
    r = np.random.default_rng(n)
    m = 57_000
    bkey = r.integers(-(1 << 62), 1 << 62, size=m)
    bpay = r.integers(-(1 << 31), 1 << 31, size=m).astype(np.int32)
    fk = np.where(r.random(n) < 0.7, bkey[r.integers(0, m, size=n)], r.integers(-(1 << 62), 1 << 62, size=n))
    fk[r.random(n) < 0.01] = np.iinfo(np.int64).min            # the empty-slot marker matches nothing
    sel = np.flatnonzero(r.random(n) < 0.6).astype(np.int32)
    table = gq.gq_join_build(ctx, dev(bkey), dev(bpay), load_factor=lf)
    fk_d, sel_d = dev(fk), dev(sel)
    half = torch.tensor([len(sel) // 2], dtype=torch.int64, device="cuda")
    for s, n_dev, used in ((None, None, None), (sel_d, None, sel), (sel_d, half, sel[:len(sel) // 2])):
        ep, ey = oracle.join(bkey, bpay, fk, used)
        prow, pay, cnt = gq.gq_join_probe(ctx, table, fk_d, sel=s, n_dev=n_dev)
        assert ctx.status() == gq.GQ_OK
        k = int(cnt.item())
        assert k == len(ep)
        assert np.array_equal(prow[:k].cpu().numpy(), ep) and np.array_equal(pay[:k].cpu().numpy(), ey)


def check_groups(res, exp, key):
    g = res.host()
    o = np.argsort(g[key], kind="stable")
    for f in (key, "count", "sum_qty", "sum_rev_lo", "sum_rev_hi"):
        assert np.array_equal(g[f][o], exp[f]), f
    for f in ("avg_qty", "avg_rev"):
        np.testing.assert_allclose(g[f][o], exp[f], rtol=1e-12, atol=0)


# few groups: 32 have copies of their sums; up to 512 bounds stay on this path
@pytest.mark.parametrize("n", [1, 1023, 8193, 300_007])
@pytest.mark.parametrize("groups", [1, 32, 33, 512])
@pytest.mark.parametrize("kind", ["code", "disc"])
def test_small_groupby_copies(ctx, n, groups, kind):
    r = np.random.default_rng(n + groups)
    qty = r.integers(-50, 50, size=n)
    price = r.integers(0, 10_000_000, size=n)
    disc = r.integers(0, 11, size=n)
    wide = r.random(n) < 0.02                                  # factors past 32 bits, revenues past 64
    price[wide] = r.integers(-(1 << 62), 1 << 62, size=int(wide.sum()))
    date = r.integers(0, 100, size=n).astype(np.int32)
    q, p, d, t = dev(qty), dev(price), dev(disc), dev(date)
    if kind == "code":                                         # keys beside the row ids, with a device count
        rows = np.flatnonzero(date < 60).astype(np.int32)
        key = r.integers(0, groups, size=max(n, 1)).astype(np.int32)[:len(rows)]
        if len(key) and groups < 512:
            key[0] = np.iinfo(np.int32).min                    # the empty marker of the LDS table is a key too
        cnt = torch.tensor([len(rows)], dtype=torch.int64, device="cuda")
        pad = np.zeros(n, dtype=np.int32)
        pad[:len(rows)] = rows
        kpad = np.zeros(n, dtype=np.int32)
        kpad[:len(rows)] = key
        res = gq.gq_groupby_agg(ctx, q, p, d, n=n, n_dev=cnt, rowid=dev(pad), key32=dev(kpad), max_groups=min(groups + 1, 512))
        exp = oracle.groupby(len(rows), qty, price, disc, rowid=rows, key32=key)
        assert ctx.status() == gq.GQ_OK
        check_groups(res, exp, "key32")
    else:                                                      # a value column as key, filtered rows
        key = r.integers(0, groups, size=n) * (1 << 33) - (1 << 40)
        res = gq.gq_groupby_agg(ctx, q, p, d, n=n, key64=dev(key), max_groups=groups, filter_col=t, filter_lo=10,
                                filter_hi=70)
        rows = np.flatnonzero((date >= 10) & (date < 70)).astype(np.int32)
        exp = oracle.groupby(len(rows), qty, price, disc, rowid=rows, key64=key[rows])
        assert ctx.status() == gq.GQ_OK
        check_groups(res, exp, "key64")


def test_small_groupby_more_groups_than_the_bound(ctx):
    """More distinct keys than twice the bound are refused, with room in the outputs or without."""
    n = 50_000
    key = dev((np.arange(n) % 300).astype(np.int32))
    one = dev(np.ones(n, dtype=np.int64))
    out = gq.alloc_groups(ctx, 400, False, True)
    gq.gq_groupby_agg(ctx, one, one, one, key32=key, max_groups=64, out=out)
    assert ctx.status() == gq.GQ_ERR_CAPACITY


# one list, one merge, two merge levels (more than 32768 candidates); rows in
# order (all of the best in one list), ties, and values that share all or none
# of their leading digits
@pytest.mark.parametrize("n,k", [(1, 1), (8192, 2048), (8193, 5), (300_000, 2048), (2_000_003, 64), (2_000_003, 2048)])
@pytest.mark.parametrize("kind", ["cents", "sorted", "ties", "signed", "equal"])
def test_topk_lists_and_merges(ctx, n, k, kind):
    r = np.random.default_rng(n + k)
    val = {"cents": lambda: r.integers(100, 10_000_000, size=n), "sorted": lambda: np.arange(n) * 7 - 1000,
           "ties": lambda: r.integers(0, 3, size=n),
           "signed": lambda: r.integers(-(1 << 63), (1 << 63) - 1, size=n, endpoint=True),
           "equal": lambda: np.full(n, -5)}[kind]().astype(np.int64)
    sel = np.flatnonzero(r.random(n) < 0.7).astype(np.int32)
    for desc in (True, False):
        for s in (None, sel):
            ev, er = oracle.topk(val, k, sel=s, descending=desc)
            v, row, cnt = gq.gq_topk(ctx, dev(val), k, sel=None if s is None else dev(s), descending=desc)
            c = int(cnt.item())
            assert c == len(ev)
            assert np.array_equal(v[:c].cpu().numpy(), ev) and np.array_equal(row[:c].cpu().numpy(), er)


# batches of 1..40 groups per instance around the 32 groups with copies, with
# tiles cut finer than asked for, and instances built in LDS and by device CAS
@pytest.mark.parametrize("groups,tile", [(1, 8192), (32, 131_072), (33, 4096), (60, 524_288)])
def test_batch_tiles_and_group_copies(ctx, groups, tile):
    r = np.random.default_rng(groups)
    specs, exp = [], []
    for m, n in [(1, 5), (700, 4095), (3000, 4097), (20_000, 150_001), (60_000, 333_333)]:
        key = r.permutation(np.arange(m) * 7919 - 12345).astype(np.int64)
        attr = r.integers(-groups, 0, size=m).astype(np.int32)
        fk = np.where(r.random(n) < 0.9, key[r.integers(0, m, size=n)], -5)
        date = r.integers(0, 100, size=n).astype(np.int32)
        qty, disc = r.integers(-9, 50, size=n), r.integers(0, 11, size=n)
        price = r.integers(0, 10_000_000, size=n)
        price[r.random(n) < 0.01] = 1 << 58                    # revenues past 32 bits and past 64
        sel = np.flatnonzero((date >= 0) & (date < 60)).astype(np.int32)
        prow, pay = oracle.join(key, attr, fk, sel)
        exp.append(oracle.groupby(len(prow), qty, price, disc, rowid=prow, key32=pay))
        specs.append({"dim_key": dev(key), "dim_attr": dev(attr), "fk": dev(fk), "date": dev(date), "qty": dev(qty),
                      "price": dev(price), "disc": dev(disc), "date_lo": 0, "date_hi": 60,
                      "out": gq.alloc_groups(ctx, 64, False, True)})
    inst = gq.make_instances(specs)
    t = gq.gq_default_tuning()
    t.probe_tile, t.load_factor = tile, 0.6
    for _ in range(2):
        gq.gq_batch_join_agg(ctx, inst, t)
        assert ctx.status() == gq.GQ_OK
        for sp, e in zip(specs, exp):
            check_groups(sp["out"], e, "key32")


# one launch up to 2^16 rows (2^15 with a selection), units of 1..32 steps above;
# ranges that take every value of the type, one value, or none
@pytest.mark.parametrize("n", [1, 1023, 1025, 32_768, 32_769, 65_536, 65_537, 262_143, 262_144, 4_194_305])
@pytest.mark.parametrize("dtype", [np.int32, np.int64])
def test_filter_units_and_ranges(ctx, n, dtype):
    r = np.random.default_rng(n)
    ii = np.iinfo(dtype)
    col = r.integers(ii.min, ii.max, size=n, dtype=dtype, endpoint=True)
    col[r.random(n) < 0.5] = r.integers(-3, 4)
    col[0], col[-1] = ii.min, ii.max
    sel = np.flatnonzero(r.random(n) < 0.8).astype(np.int32)
    half = torch.tensor([len(sel) // 2], dtype=torch.int64, device="cuda")
    c, s = dev(col), dev(sel)
    x = int(col[n // 2])
    i64 = np.iinfo(np.int64)
    for lo, hi in [(i64.min, i64.max), (int(ii.min), int(ii.max)), (x, x + 1) if x < i64.max else (x, x), (5, 5), (9, -9),
                   (-4, 4), (int(ii.max), i64.max), (i64.min, int(ii.min))]:
        keep = (col >= lo) & (col < hi)
        for sd, nd, used in ((None, None, np.arange(n, dtype=np.int32)), (s, None, sel), (s, half, sel[:len(sel) // 2])):
            exp = used[keep[used]]
            out, cnt = gq.gq_filter(ctx, c, lo, hi, sel_in=sd, n_dev=nd)
            k = int(cnt.item())
            assert k == len(exp) and np.array_equal(out[:k].cpu().numpy(), exp)


# the large path around its bucket rules: fewer rows than one bucket per CU
# needs, just enough, and a chunk size of one to several scatter tiles
@pytest.mark.parametrize("n", [4097, 100_001, 1_048_577, 5_000_011])
@pytest.mark.parametrize("groups", [513, 20_000])
@pytest.mark.parametrize("kind", ["code", "composite"])
def test_large_groupby_buckets(ctx, n, groups, kind):
    r = np.random.default_rng(n + groups)
    qty, disc = r.integers(-50, 50, size=n), r.integers(0, 11, size=n)
    price = r.integers(0, 10_000_000, size=n)
    date = r.integers(0, 100, size=n).astype(np.int32)
    rows = np.flatnonzero(date < 60).astype(np.int32)
    code = r.integers(0, groups // 2, size=n).astype(np.int32)
    args = dict(n=n, max_groups=groups, filter_col=dev(date), filter_lo=20, filter_hi=100)
    used = rows[date[rows] >= 20]
    pad = np.zeros(n, dtype=np.int32)
    pad[:len(rows)] = rows
    args.update(rowid=dev(pad), n_dev=torch.tensor([len(rows)], dtype=torch.int64, device="cuda"))
    q, p, d = dev(qty), dev(price), dev(disc)
    if kind == "code":
        res = gq.gq_groupby_agg(ctx, q, p, d, key32=dev(code), key32_by_rowid=True, **args)
        exp = oracle.groupby(len(used), qty, price, disc, rowid=used, key32=code[used])
        assert ctx.status() == gq.GQ_OK
        check_groups(res, exp, "key32")
    else:
        k64 = (code.astype(np.int64) // 2) * (1 << 40) - 7
        k32 = (code % 2).astype(np.int32)
        res = gq.gq_groupby_agg(ctx, q, p, d, key64=dev(k64), key64_by_rowid=True, key32=dev(k32), key32_by_rowid=True,
                                **args)
        exp = oracle.groupby(len(used), qty, price, disc, rowid=used, key64=k64[used], key32=k32[used])
        assert ctx.status() == gq.GQ_OK
        g = res.host()
        o = np.lexsort((g["key32"], g["key64"]))
        for f in ("key64", "key32", "count", "sum_qty", "sum_rev_lo", "sum_rev_hi"):
            assert np.array_equal(g[f][o], exp[f]), f


# tables built in LDS (up to 8192 slots) and just above, with a selection and a
# device count, keys that wrap past the last slot, and the error cases
@pytest.mark.parametrize("m,lf", [(1, 0.5), (57, 0.9), (4096, 0.5), (7372, 0.9), (7373, 0.9), (9000, 0.5)])
def test_lds_build(ctx, m, lf):
    r = np.random.default_rng(m)
    key = r.permutation(np.arange(2 * m) - m).astype(np.int64)
    pay = r.integers(-(1 << 31), 1 << 31, size=2 * m).astype(np.int32)
    sel = np.sort(r.choice(2 * m, size=m, replace=False)).astype(np.int32)
    cnt = max(1, m - 3)
    fk = r.integers(-2 * m, 2 * m, size=20_011)
    fk[5] = np.iinfo(np.int64).min
    k, p, f, s = dev(key), dev(pay), dev(fk), dev(sel)
    n_dev = torch.tensor([cnt], dtype=torch.int64, device="cuda")
    whole = (k[:m].contiguous(), p[:m].contiguous())
    for table, bk, bp in (
            (gq.gq_join_build(ctx, *whole, load_factor=lf), key[:m], pay[:m]),
            (gq.gq_join_build(ctx, k, p, sel=s, load_factor=lf), key[sel], pay[sel]),
            (gq.gq_join_build(ctx, k, p, sel=s, n_dev=n_dev, load_factor=lf), key[sel[:cnt]], pay[sel[:cnt]])):
        assert ctx.status() == gq.GQ_OK
        ep, ey = oracle.join(bk, bp, fk, None)
        prow, out, c = gq.gq_join_probe(ctx, table, f)
        c = int(c.item())
        assert c == len(ep)
        assert np.array_equal(prow[:c].cpu().numpy(), ep) and np.array_equal(out[:c].cpu().numpy(), ey)
    if m > 1:
        bad = key[:m].copy()
        bad[-1] = bad[0]
        gq.gq_join_build(ctx, dev(bad), whole[1], load_factor=lf)
        assert ctx.status() == gq.GQ_ERR_DUPLICATE_KEY
        bad[-1] = np.iinfo(np.int64).min
        gq.gq_join_build(ctx, dev(bad), whole[1], load_factor=lf)
        assert ctx.status() == gq.GQ_ERR_INVALID_KEY


def test_filter_of_a_misaligned_column(ctx):
    """A column that does not start on 16 bytes takes the scalar loads."""
    r = np.random.default_rng(5)
    for dtype in (np.int32, np.int64):
        col = r.integers(0, 100, size=50_001).astype(dtype)
        d = dev(col)
        for o in range(1, 4):
            out, cnt = gq.gq_filter(ctx, d[o:], 20, 70)
            exp = np.flatnonzero((col[o:] >= 20) & (col[o:] < 70)).astype(np.int32)
            k = int(cnt.item())
            assert k == len(exp) and np.array_equal(out[:k].cpu().numpy(), exp)


# partition tiles of 2048 rows below 2^21 rows, of 4096 from there on; a wave's
# and a workgroup's remainder in the last tile
@pytest.mark.parametrize("n", [63, 2047, 2049, 33 * 2048 + 1025, (1 << 21) - 1, 1 << 21])
@pytest.mark.parametrize("log2p", [2, 8])
def test_partition_tiles(ctx, n, log2p):
    r = np.random.default_rng(n + log2p)
    key = r.integers(-(1 << 62), 1 << 62, size=n)
    key[r.random(n) < 0.3] = 7                                 # one heavy bucket
    cols = [r.integers(0, 1 << 31, size=n).astype(np.int32), r.integers(-(1 << 62), 1 << 62, size=n)]
    ek, ec, erow, eoff = oracle.partition(key, log2p, cols)
    for rowid in (True, False):
        k, c, row, off = gq.gq_radix_partition(ctx, dev(key), log2p, [dev(x) for x in cols], rowid=rowid)
        assert ctx.status() == gq.GQ_OK
        assert np.array_equal(off.cpu().numpy(), eoff) and np.array_equal(k.cpu().numpy(), ek)
        assert all(np.array_equal(x.cpu().numpy(), e) for x, e in zip(c, ec))
        assert (row is None) if not rowid else np.array_equal(row.cpu().numpy(), erow)


# run offsets: one chunk of tiles and several, shares that are loaded once and
# in batches (tiles of 2048 rows; 32 tiles a chunk, so 32 and 33, and 64 a chunk)
@pytest.mark.parametrize("n", [32 * 2048, 32 * 2048 + 1, 100 * 2048 + 5])
@pytest.mark.parametrize("log2p", [0, 5, 7])
def test_partition_offsets(ctx, n, log2p):
    r = np.random.default_rng(n)
    key = r.integers(0, 1 << 20, size=n)
    ek, _, erow, eoff = oracle.partition(key, log2p)
    k, _, row, off = gq.gq_radix_partition(ctx, dev(key), log2p)
    assert ctx.status() == gq.GQ_OK
    assert np.array_equal(off.cpu().numpy(), eoff) and np.array_equal(row.cpu().numpy(), erow)
    assert np.array_equal(k.cpu().numpy(), ek)


# more tiles than 192 chunks of 32 (shares longer than one load): the invariants of a partition
def test_partition_offsets_many_tiles(ctx):
    n = 6200 * 4096 + 3
    key = torch.randint(0, 1 << 40, (n,), dtype=torch.int64, device="cuda", generator=torch.Generator("cuda").manual_seed(3))
    for log2p in (1, 8):
        k, _, row, off = gq.gq_radix_partition(ctx, key, log2p)
        assert ctx.status() == gq.GQ_OK
        assert torch.equal(k, key[row.long()])
        off = off.cpu().numpy()
        assert off[0] == 0 and off[-1] == n
        b = np.repeat(np.arange(1 << log2p), np.diff(off))
        h = k.cpu().numpy().view(np.uint64)                    # fmix64 of the keys
        for mul in (0xff51afd7ed558ccd, 0xc4ceb9fe1a85ec53):
            h = (h ^ (h >> np.uint64(33))) * np.uint64(mul)
        h = (h ^ (h >> np.uint64(33))) >> np.uint64(64 - log2p)
        assert np.array_equal(h.astype(np.int64), b)
        d = torch.diff(row.long())
        edges = torch.zeros(n - 1, dtype=torch.bool, device="cuda")
        edges[torch.from_numpy(off[1:-1] - 1).cuda()] = True
        assert bool(((d > 0) | edges).all())                   # stable inside each bucket


# answers that are ranked by counting (up to 256 keys) and sorted (more), from
# scans of one step, two and many workgroups
@pytest.mark.parametrize("n", [1, 255, 4096, 4097, 300_001])
@pytest.mark.parametrize("k", [1, 255, 256, 257])
def test_topk_ranked(ctx, n, k):
    r = np.random.default_rng(n + k)
    val = r.integers(-50, 50, size=n).astype(np.int64)             # ties go to the smaller row id
    for desc in (True, False):
        v, row, cnt = gq.gq_topk(ctx, dev(val), k, descending=desc)
        c = int(cnt.item())
        exp = np.lexsort((np.arange(n), -val if desc else val))[:k]
        assert c == len(exp)
        assert np.array_equal(row[:c].cpu().numpy(), exp) and np.array_equal(v[:c].cpu().numpy(), val[exp])


# keys that walk far from their home slot: one cluster at load factor 0.9, past
# the table's end, and a second copy of a key at the end of the walk
def test_insert_walks(ctx):
    slots = 1 << 14
    def unmix(h):                                                  # the inverse of fmix64
        h = h ^ (h >> np.uint64(33))
        h = h * np.uint64(0x9cb4b2f8129337db)
        h = h ^ (h >> np.uint64(33))
        h = h * np.uint64(0x4f74430c22a54005)
        return h ^ (h >> np.uint64(33))
    home = np.concatenate([np.full(200, slots - 20), np.full(57, 77), np.arange(1000, 9000)]).astype(np.uint64)
    h = (home << np.uint64(64 - 14)) | np.arange(len(home), dtype=np.uint64)
    key = unmix(h).view(np.int64)
    assert len(np.unique(key)) == len(key)
    pay = np.arange(len(key), dtype=np.int32)
    fk = np.concatenate([key, key + 1])
    table = torch.empty(256 + slots * 16, dtype=torch.uint8, device="cuda")
    gq.gq_join_build(ctx, dev(key), dev(pay), table=table)
    assert ctx.status() == gq.GQ_OK
    prow, out, cnt = gq.gq_join_probe(ctx, table, dev(fk))
    ep, ey = oracle.join(key, pay, fk, None)
    c = int(cnt.item())
    assert c == len(ep) and np.array_equal(prow[:c].cpu().numpy(), ep) and np.array_equal(out[:c].cpu().numpy(), ey)
    gq.gq_join_build(ctx, dev(np.append(key, key[199])), dev(np.append(pay, 0).astype(np.int32)), table=table)
    assert ctx.status() == gq.GQ_ERR_DUPLICATE_KEY


# two scatter levels (1280 buckets): key64 records carry their sub-bucket in a
# byte, key32 records do not; ragged last tiles, and a filter that drops rows
@pytest.mark.parametrize("n", [1, 2047, 2049, 200_003])
@pytest.mark.parametrize("kind", ["key64", "both", "key32"])
def test_two_level_groupby(ctx, n, kind):
    r = np.random.default_rng(n)
    domain = 50_000
    qty, price, disc = (r.integers(lo, hi, size=n).astype(np.int64) for lo, hi in ((1, 51), (100, 10_000_001), (0, 11)))
    key64 = r.integers(-(1 << 62), 1 << 62, size=domain)[r.integers(0, domain, size=n)] if kind != "key32" else None
    key32 = r.integers(0, 2 if kind == "both" else domain, size=n).astype(np.int32) if kind != "key64" else None
    used = np.flatnonzero(disc < 7)
    cap = 1_400_000 if kind != "key32" else 2_000_000
    sub = lambda x: None if x is None else x[used]
    exp = oracle.groupby(len(used), qty[used], price[used], disc[used], key64=sub(key64), key32=sub(key32))
    d = lambda x: None if x is None else dev(x)
    res = gq.gq_groupby_agg(ctx, dev(qty), dev(price), dev(disc), key64=d(key64), key32=d(key32), max_groups=cap,
                            filter_col=dev(disc.astype(np.int32)), filter_lo=0, filter_hi=7)
    assert ctx.status() == gq.GQ_OK
    g = res.host()
    o = np.lexsort((g["key32"] if key32 is not None else np.zeros(len(g["count"])),
                    g["key64"] if key64 is not None else np.zeros(len(g["count"]))))
    for f in ("key64", "key32", "count", "sum_qty", "sum_rev_lo", "sum_rev_hi"):
        if g[f] is not None:
            assert np.array_equal(g[f][o], exp[f]), f


# tables built by regions of 8192 slots (2^15 slots and more, here at load
# factor 0.5) beside one that is not: a bin that overflows, walks past a region
# and past the table's end, keys that repeat inside a bin and across the
# overflow list, the marker as a key, and errors kept to their own instance
def test_batch_region_builds(ctx):
    r = np.random.default_rng(11)

    def unmix(h):                                                  # the inverse of fmix64
        h = h ^ (h >> np.uint64(33))
        h = h * np.uint64(0x9cb4b2f8129337db)
        h = h ^ (h >> np.uint64(33))
        h = h * np.uint64(0x4f74430c22a54005)
        return h ^ (h >> np.uint64(33))

    def keys(home, bits):                                          # distinct keys with these home slots
        return unmix((home.astype(np.uint64) << np.uint64(64 - bits)) | np.arange(len(home), dtype=np.uint64)).view(np.int64)

    spread = r.integers(-(1 << 62), 1 << 62, size=140_001)
    crowd = keys(np.concatenate([r.integers(8192, 16384, size=12_000), np.full(2000, 16383)]), 15)
    ends = keys(np.concatenate([np.full(300, 32767), r.integers(0, 32768, size=14_000)]), 15)
    dup, marker = spread[:15_000].copy(), spread[:15_000].copy()
    dup[-1] = dup[3]
    marker[77] = np.iinfo(np.int64).min
    crowd_dup = np.append(crowd, [crowd[5], crowd[13_999]])
    good = [spread, spread[:8192], spread[:8193], crowd, ends, spread[:50_000]]
    bad = {6: (dup, gq.GQ_ERR_DUPLICATE_KEY), 7: (marker, gq.GQ_ERR_INVALID_KEY), 8: (crowd_dup, gq.GQ_ERR_DUPLICATE_KEY)}
    specs, exp = [], []
    for key in good + [k for k, _ in bad.values()]:
        m, n = len(key), 60_000
        attr = r.integers(0, 20, size=m).astype(np.int32)
        fk = np.where(r.random(n) < 0.8, key[r.integers(0, m, size=n)], r.integers(-(1 << 62), 1 << 62, size=n))
        date = r.integers(0, 100, size=n).astype(np.int32)
        qty, price, disc = r.integers(1, 51, size=n), r.integers(100, 10_000_001, size=n), r.integers(0, 11, size=n)
        if len(exp) < len(good):
            prow, pay = oracle.join(key, attr, fk, np.flatnonzero(date < 60).astype(np.int32))
            exp.append(oracle.groupby(len(prow), qty, price, disc, rowid=prow, key32=pay))
        specs.append({"dim_key": dev(key), "dim_attr": dev(attr), "fk": dev(fk), "date": dev(date), "qty": dev(qty),
                      "price": dev(price), "disc": dev(disc), "date_lo": 0, "date_hi": 60,
                      "out": gq.alloc_groups(ctx, 64, False, True)})
    for count in (len(good), len(specs)):
        status = torch.full((count,), -1, dtype=torch.int32, device="cuda")
        gq.gq_batch_join_agg(ctx, gq.make_instances(specs[:count]), inst_status=status)
        word = ctx.status()
        assert (word == gq.GQ_OK) == (count == len(good))
        assert status.tolist() == [gq.GQ_OK] * len(good) + [c for _, c in bad.values()][:count - len(good)]
        for sp, e in zip(specs, exp):
            check_groups(sp["out"], e, "key32")


# a filter over few groups: the waves' spans of 512 rows, lists that fill a
# batch exactly, nearly and never, and rows kept by value and by position
@pytest.mark.parametrize("n", [1, 511, 513, 8193, 2_200_003])
@pytest.mark.parametrize("keep", [0.0, 0.01, 0.5, 1.0])
def test_small_groupby_filter_lists(ctx, n, keep):
    r = np.random.default_rng(n)
    qty, price, disc = (r.integers(lo, hi, size=n).astype(np.int64) for lo, hi in ((-9, 51), (100, 10_000_001), (0, 11)))
    price[r.random(n) < 0.01] = 1 << 58                            # revenues past 32 bits and past 64
    key32 = r.integers(0, 40, size=n).astype(np.int32)             # some past the 32 groups that have copies
    col = np.where(r.random(n) < keep, r.integers(-5, 5, size=n), 100).astype(np.int32)
    used = np.flatnonzero((col >= -5) & (col < 5))
    for k64 in (None, disc):
        exp = oracle.groupby(len(used), qty[used], price[used], disc[used], key32=key32[used],
                             key64=None if k64 is None else k64[used])
        res = gq.gq_groupby_agg(ctx, dev(qty), dev(price), dev(disc), key32=dev(key32),
                                key64=None if k64 is None else dev(k64), max_groups=512, filter_col=dev(col),
                                filter_lo=-5, filter_hi=5)
        assert ctx.status() == gq.GQ_OK
        g = res.host()
        o = np.lexsort((g["key32"], np.zeros(len(g["count"])) if k64 is None else g["key64"]))
        for f in ("key64", "key32", "count", "sum_qty", "sum_rev_lo", "sum_rev_hi"):
            if g[f] is not None:
                assert np.array_equal(g[f][o], exp[f]), f


# probes on both sides of the unit rules (2^18, 2^20, 2^21 rows) over a table
# with long walks, some past its end
@pytest.mark.parametrize("n", [(1 << 18) - 1, 1 << 18, (1 << 20) + 1, (1 << 21) - 1])
def test_probe_walks(ctx, n):
    r = np.random.default_rng(n)
    m, slots = 14_700, 1 << 14                                     # load factor 0.897
    key = r.permutation(np.arange(3 * m))[:m].astype(np.int64) * 1_000_003
    pay = r.integers(-(1 << 31), 1 << 31, size=m).astype(np.int32)
    fk = np.where(r.random(n) < 0.5, key[r.integers(0, m, size=n)], r.integers(0, 3 * m, size=n) * 1_000_003 + 1)
    table = torch.empty(256 + slots * 16, dtype=torch.uint8, device="cuda")
    gq.gq_join_build(ctx, dev(key), dev(pay), table=table)
    prow, out, cnt = gq.gq_join_probe(ctx, table, dev(fk))
    assert ctx.status() == gq.GQ_OK
    ep, ey = oracle.join(key, pay, fk, None)
    c = int(cnt.item())
    assert c == len(ep) and np.array_equal(prow[:c].cpu().numpy(), ep) and np.array_equal(out[:c].cpu().numpy(), ey)
