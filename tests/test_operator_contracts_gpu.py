"""What the operators promise beyond the plain call: selections that name a row
more than once, outputs that are also inputs, and empty inputs.  Everything is
whole numbers, compared with the CPU oracle bit for bit."""
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


def guarded(k, dtype, mark):
    """An output of k entries between two borders of 4096 entries that no call may touch."""
    t = torch.full((k + 8192,), mark, dtype=dtype, device="cuda")
    return t, t[4096:4096 + k]


# a selection with repeats: inside the answer, across the k-th place and over
# the whole buffer (4096 candidates); answers ranked (k <= 256) and sorted; one
# list, one merge and two merge levels
@pytest.mark.parametrize("n", [6, 5000, 70_001, 2_000_003])
@pytest.mark.parametrize("k", [1, 10, 256, 257, 1000, 2048])
@pytest.mark.parametrize("rows", ["one", "few", "pairs", "any"])
def test_topk_of_repeated_rows(ctx, n, k, rows):
    r = np.random.default_rng(n + k)
    sel = {"one": lambda: np.full(n, 3), "few": lambda: r.integers(0, 7, size=n),
           "pairs": lambda: r.permutation(np.arange(n) // 2), "any": lambda: r.integers(0, n, size=n)}[rows]()
    sel = sel.astype(np.int32)
    val = r.integers(0, 1000 if rows == "any" else 1 << 40, size=max(n, 8)).astype(np.int64)
    for desc in (True, False):
        vall, v = guarded(k, torch.int64, -77)
        rall, row = guarded(k, torch.int32, -77)
        ev, er = oracle.topk(val, k, sel=sel, descending=desc)
        _, _, cnt = gq.gq_topk(ctx, dev(val), k, sel=dev(sel), descending=desc, val_out=v, rowid_out=row)
        c = int(cnt.item())
        assert c == len(ev) == min(n, k)
        assert np.array_equal(v[:c].cpu().numpy(), ev) and np.array_equal(row[:c].cpu().numpy(), er)
        for t in (vall, rall):
            assert bool((t[:4096] == -77).all()) and bool((t[4096 + c:] == -77).all())


# a device count narrowed in place: n_out_dev is n_dev.  Few rows pass, so a
# workgroup that read the new count would drop matches.
@pytest.mark.parametrize("n", [0, 1, 1025, 32_768, 32_769, 200_000])
@pytest.mark.parametrize("with_sel", [False, True])
def test_filter_narrows_its_count_in_place(ctx, n, with_sel):
    r = np.random.default_rng(n)
    col = r.integers(0, 1000, size=n + 100).astype(np.int32)
    sel = r.permutation(n + 100)[:n].astype(np.int32) if with_sel else None
    sel_d = None if sel is None else dev(sel)
    used = n - n // 50
    exp = oracle.filter(col[:used] if sel is None else col, 0, 20, sel_in=None if sel is None else sel[:used])
    col_d = dev(col[:n] if sel is None else col)
    for f in (gq.gq_filter, gq.gq_filter_noalloc):
        for _ in range(20):
            cnt = torch.tensor([used if n else 5], dtype=torch.int64, device="cuda")
            out = torch.full((max(n, 1),), -1, dtype=torch.int32, device="cuda")
            f(ctx, col_d, 0, 20, sel_in=sel_d, n=n, n_dev=cnt, out=out, n_out=cnt)
            assert int(cnt.item()) == len(exp)
            assert np.array_equal(out[:len(exp)].cpu().numpy(), exp)


# a selection narrowed in place (sel_out is sel_in), alone and with its count;
# units of 1024 rows, of several steps and of 32 (the most row ids held)
@pytest.mark.parametrize("n", [1, 65, 1025, 32_768, 32_769, 262_145, 4_194_304 + 77, 9_000_001])
@pytest.mark.parametrize("dtype", [np.int32, np.int64])
@pytest.mark.parametrize("hi", [20, 900])
def test_filter_narrows_a_selection_in_place(ctx, n, dtype, hi):
    r = np.random.default_rng(n)
    col = r.integers(0, 1000, size=n + 100).astype(dtype)
    sel = r.permutation(n + 100)[:n].astype(np.int32)
    col_d = dev(col)
    for f, used in ((gq.gq_filter, n), (gq.gq_filter, n - n // 50), (gq.gq_filter_noalloc, n - n // 3)):
        exp = oracle.filter(col, 0, hi, sel_in=sel[:used])
        s = dev(sel)
        if used == n:
            cnt = torch.zeros(1, dtype=torch.int64, device="cuda")
            f(ctx, col_d, 0, hi, sel_in=s, out=s, n_out=cnt)
        else:
            cnt = torch.tensor([used], dtype=torch.int64, device="cuda")
            f(ctx, col_d, 0, hi, sel_in=s, n_dev=cnt, out=s, n_out=cnt)
        assert int(cnt.item()) == len(exp)
        assert np.array_equal(s[:len(exp)].cpu().numpy(), exp)
        assert np.array_equal(s[len(exp):].cpu().numpy(), sel[len(exp):])      # nothing past the answer is touched


# a probe that narrows its selection in place (prow_out is sel), with its count:
# units of 512 rows, of 1024 rows and of 16 steps
@pytest.mark.parametrize("n", [1, 65, 513, 131_072, 131_073, 2_000_003, (1 << 25) + 5])
@pytest.mark.parametrize("hits", [0.02, 0.9])
def test_probe_narrows_a_selection_in_place(ctx, n, hits):
    r = np.random.default_rng(n)
    m = 5000
    key = r.permutation(m * 4)[:m].astype(np.int64) * 7919
    pay = r.integers(-(1 << 31), 1 << 31, size=m).astype(np.int32)
    rows = min(n, 500_000) + 100
    fk = np.where(r.random(rows) < hits, key[r.integers(0, m, size=rows)], -1)
    sel = r.integers(0, rows, size=n).astype(np.int32)
    table = gq.gq_join_build(ctx, dev(key), dev(pay))
    fk_d = dev(fk)
    for f, used in ((gq.gq_join_probe, n), (gq.gq_join_probe_partitioned, n - n // 3)):
        ep, ey = oracle.join(key, pay, fk, sel[:used])
        s = dev(sel)
        cnt = torch.tensor([used], dtype=torch.int64, device="cuda")
        _, got, _ = f(ctx, table, fk_d, sel=s, n_dev=cnt, prow=s, n_out=cnt)
        assert ctx.status() == gq.GQ_OK
        assert int(cnt.item()) == len(ep)
        assert np.array_equal(s[:len(ep)].cpu().numpy(), ep) and np.array_equal(got[:len(ep)].cpu().numpy(), ey)
        assert np.array_equal(s[len(ep):].cpu().numpy(), sel[len(ep):])        # nothing past the answer is touched


# few groups whose keys are structured: sums of the key's words that agree, and
# strides at which a plain product puts neighbours side by side
@pytest.mark.parametrize("n", [513, 100_003])
@pytest.mark.parametrize("kind", ["anti-diagonal", "grid", "key64 stride", "key32 stride"])
def test_small_groupby_of_structured_keys(ctx, n, kind):
    r = np.random.default_rng(n)
    i = r.integers(0, 512, size=n)
    k64, k32 = {"anti-diagonal": (i, 511 - i), "grid": (i % 22, i // 22 % 23), "key64 stride": (i * 10_946, None),
                "key32 stride": (None, i * -1597)}[kind]
    k32 = None if k32 is None else k32.astype(np.int32)
    qty, price, disc = r.integers(-50, 50, size=n), r.integers(0, 10_000_000, size=n), r.integers(0, 11, size=n)
    exp = oracle.groupby(n, qty, price, disc, key64=k64, key32=k32)
    res = gq.gq_groupby_agg(ctx, dev(qty), dev(price), dev(disc), key64=None if k64 is None else dev(k64),
                            key32=None if k32 is None else dev(k32), max_groups=512)
    assert ctx.status() == gq.GQ_OK
    g = res.host()
    order = np.lexsort([g[f] for f in ("key32", "key64") if g[f] is not None])
    for f in ("key64", "key32", "count", "sum_qty", "sum_rev_lo", "sum_rev_hi"):
        if g[f] is not None:
            assert np.array_equal(g[f][order], exp[f]), f


# no rows, on every path (few groups, buckets, two levels), in a workspace that
# holds anything
@pytest.mark.parametrize("max_groups", [64, 5000, 2_000_000])
@pytest.mark.parametrize("kind", ["key32", "key64", "both", "none"])
@pytest.mark.parametrize("counted", [False, True])
def test_groupby_of_no_rows(ctx, max_groups, kind, counted):
    n = 1000 if counted else 0
    e = torch.zeros(1000, dtype=torch.int64, device="cuda")
    k64 = e if kind in ("key64", "both") else None
    k32 = e.int() if kind in ("key32", "both") else None
    has64, has32 = kind in ("key64", "both"), kind in ("key32", "both")
    out = gq.alloc_groups(ctx, max_groups, has64, has32)
    out.n_groups.fill_(7)
    need = gq.lib().gq_groupby_workspace_bytes(n, max_groups, int(has64), int(has32))
    ws = torch.full((need,), 0x5A, dtype=torch.uint8, device="cuda")
    zero = torch.zeros(1, dtype=torch.int64, device="cuda") if counted else None
    gq.gq_groupby_agg(ctx, e, e, e, n=n, n_dev=zero, key64=k64, key32=k32, max_groups=max_groups, out=out, ws=ws)
    assert ctx.status() == gq.GQ_OK
    assert int(out.n_groups.item()) == 0


# both sides of the line between the filter's one-launch and look-back forms
@pytest.mark.parametrize("dtype,n,with_sel", [(np.int32, 131_072, False), (np.int32, 131_073, False),
                                              (np.int64, 65_536, False), (np.int64, 65_537, False),
                                              (np.int32, 16_384, True), (np.int64, 16_385, True)])
def test_filter_forms_meet(ctx, dtype, n, with_sel):
    r = np.random.default_rng(n)
    col = r.integers(-50, 50, size=n).astype(dtype)
    sel = r.permutation(n).astype(np.int32) if with_sel else None
    exp = oracle.filter(col, -20, 30, sel_in=sel)
    out, cnt = gq.gq_filter(ctx, dev(col), -20, 30, sel_in=None if sel is None else dev(sel))
    assert int(cnt.item()) == len(exp) and np.array_equal(out[:len(exp)].cpu().numpy(), exp)


def batch_of(r, sizes):
    specs = []
    for m, n in sizes:
        key = r.permutation(np.arange(m) * 7919).astype(np.int64)
        specs.append({"dim_key": dev(key), "dim_attr": dev(r.integers(0, 20, size=m).astype(np.int32)),
                      "fk": dev(key[r.integers(0, m, size=n)]), "date": dev(r.integers(0, 100, size=n).astype(np.int32)),
                      "qty": dev(r.integers(1, 50, size=n)), "price": dev(r.integers(0, 10_000_000, size=n)),
                      "disc": dev(r.integers(0, 11, size=n)), "date_lo": 0, "date_hi": 60})
    return specs


def test_autotune_leaves_what_changes_nothing(ctx):
    """Tables that are built by regions at every load factor leave no builds in
    the queue: lag and build tile stay at the search's starting point."""
    specs = [dict(s, out=gq.alloc_groups(ctx, 64, False, True))
             for s in batch_of(np.random.default_rng(1), [(40_000, 60_000), (50_000, 40_001)])]
    best, ms = gq.gq_batch_autotune(ctx, gq.make_instances(specs))
    assert ctx.status() == gq.GQ_OK
    assert ms > 0 and (best.lag, best.build_tile) == (4, gq.gq_default_tuning().build_tile)


# the library's scratch after a larger call: both later ones use it too
@pytest.mark.parametrize("dtype", [np.int32, np.int64])
def test_noalloc_clears_its_scratch(ctx, dtype):
    r = np.random.default_rng(17)
    for n in (3_000_001, 200_001, 140_000, 3_000_001):
        col = r.integers(0, 2557, size=n).astype(dtype)
        out = torch.empty(n, dtype=torch.int32, device="cuda")
        cnt = torch.zeros(1, dtype=torch.int64, device="cuda")
        gq.gq_filter_noalloc(ctx, dev(col), 100, 900, out, cnt)
        exp = oracle.filter(col, 100, 900)
        assert int(cnt.item()) == len(exp) and np.array_equal(out[:len(exp)].cpu().numpy(), exp)


# waves whose matches go through the stage in one round and in two (up to half
# and three quarters of their rows), and waves that write step by step; units
# of 8, 16 and 32 steps; densities that change within a unit
@pytest.mark.parametrize("n", [1_048_576, 2_097_152 + 77, 4_194_304 + 31 * 1024 + 5])
@pytest.mark.parametrize("dtype", [np.int32, np.int64])
@pytest.mark.parametrize("keep", [0.002, 0.25, 0.5, 0.74, 0.76, 1.0, None])
def test_filter_stage(ctx, n, dtype, keep):
    r = np.random.default_rng(n)
    col = r.integers(0, 1000, size=n).astype(dtype)
    if keep is None:                                           # another density every 512 rows
        thr = np.repeat(r.integers(0, 1001, size=n // 512 + 1), 512)[:n]
        col = np.where(col < thr, 0, 999).astype(dtype)
    hi = 500 if keep is None else int(keep * 1000)
    sel = r.permutation(n).astype(np.int32)[:n - 3] if keep in (0.25, 0.74) else None
    exp = oracle.filter(col, 0, hi, sel_in=sel)
    out = torch.full((n + 4096,), -1, dtype=torch.int32, device="cuda")
    _, cnt = gq.gq_filter(ctx, dev(col), 0, hi, sel_in=None if sel is None else dev(sel), out=out)
    assert int(cnt.item()) == len(exp) and np.array_equal(out[:len(exp)].cpu().numpy(), exp)
    assert bool((out[len(exp):] == -1).all())


# both sides of the probe's shape rule: 1 to 4 steps with a unit per CU, then the
# fewest steps that keep the rounds (4, 5; 16 and, a round more, 9)
@pytest.mark.parametrize("n", [262_145, 524_289, 786_433, 1_048_577, 2_097_153, 8_388_608, 8_388_609])
def test_probe_rounds(ctx, n):
    r = np.random.default_rng(n)
    m = 3000
    key = r.permutation(m * 3)[:m].astype(np.int64) * 7919
    pay = r.integers(-(1 << 31), 1 << 31, size=m).astype(np.int32)
    fk = np.where(r.random(n) < 0.6, key[r.integers(0, m, size=n)], -1)
    ep, ey = oracle.join(key, pay, fk, None)
    table = gq.gq_join_build(ctx, dev(key), dev(pay))
    prow, got, cnt = gq.gq_join_probe(ctx, table, dev(fk))
    assert ctx.status() == gq.GQ_OK
    assert int(cnt.item()) == len(ep)
    assert np.array_equal(prow[:len(ep)].cpu().numpy(), ep) and np.array_equal(got[:len(ep)].cpu().numpy(), ey)
