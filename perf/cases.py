"""The work whose speed this library is measured by: its public entry points
over the sizes and options that its users run.

A case is a dict of plain values; `op` names the entry point or driver.  Inputs
have the column shapes of the workloads in `synth` (unique int64 dimension
keys, foreign keys into them, dates in [0, 2557), quantities, prices in cents,
discounts); their sizes come from the bench, the smoke run and the tests, or
are odd sizes between those.  What a query program holds from one call to the
next (tables, workspaces, output buffers, instance lists, a running server) is
made by prepare(); run() is one pass through the library.

Group-by results come out of the library in no particular order, so a pass
that aggregates ends, as such a query does, with ORDER BY its group key.  The
buffers are as long as the group bound; the keys past the last group hold the
type's largest value, so they sort to the end.
"""
from __future__ import annotations

import math

import torch

import paper_2506_09226_amd as gq
import synth
from paper_2506_09226_amd.pipeline import PlainPipeline
from paper_2506_09226_amd.serve import QuerySpec, Server

DEVICE = "cuda"
I32_MAX, I64_MAX = (1 << 31) - 1, (1 << 63) - 1
DATE_HI = 1500                          # the workloads' usual predicate: 58.7% of the rows
SEL_FRAC = DATE_HI / synth.DATE_RANGE
STATS = ("count", "sum_qty", "sum_rev_lo", "sum_rev_hi", "avg_qty", "avg_rev")


# --------------------------------------------------------------------- cases
def listed():
    return [
        # The smallest call in use: one filter over a smoke-sized column.
        {"name": "filter_64k", "op": "filter", "n": 65_536, "dtype": "i32", "sel": False, "keep": SEL_FRAC},
        # A dimension look-up join of a few thousand keys: build and probe, latency bound.
        {"name": "join_small", "op": "join", "m": 4_096, "n": 65_536, "hit": 1.0},
        # A join whose table is larger than the caches, with a fifth of the probes unmatched.
        {"name": "join_large", "op": "join", "m": 6_000_000, "n": 50_000_021, "hit": 0.8},
        # The local half of a wide shuffle: 256 buckets, mixed column widths, a ragged row count.
        {"name": "partition_256", "op": "partition", "n": 20_000_003, "log2p": 8, "w4": 1, "w8": 2, "rowid": True},
        # ORDER BY price LIMIT 1000 over a selection.
        {"name": "topk_1000", "op": "topk", "n": 50_000_017, "k": 1000, "desc": False, "sel": True},
        # A report with few groups: filter and group by a low-cardinality column, one scan.
        {"name": "groupby_disc", "op": "groupby", "kind": "disc", "n": 60_000_007, "groups": 11},
        # Group by the attribute that a join returned: a middling number of groups.
        {"name": "groupby_codes", "op": "groupby", "kind": "code", "n": 5_000_011, "groups": 100_000},
        # A skewed composite key (Zipf foreign key, small second key): heavy keys and millions of groups.
        {"name": "groupby_zipf", "op": "groupby", "kind": "zipf", "n": 50_000_000, "groups": 2_000_000},
        # The small workload: the whole chain over a million rows, 25 groups.
        {"name": "pipeline_small", "op": "pipeline", "n": 1_048_576, "m": 65_536, "groups": 25, "log2p": 6,
         "topk": 100, "date_hi": DATE_HI, "streams": 1},
        # One GPU's share: the bench's default step, 200M x 25M rows and 1.5M groups.
        {"name": "pipeline_share", "op": "pipeline", "n": 200_000_000, "m": 25_000_000, "groups": 1_500_000,
         "log2p": 6, "topk": 100, "date_hi": DATE_HI, "streams": 1},
        # Independent join + aggregate instances in one launch, drawn as in the batched workload.
        {"name": "batch_64", "op": "batch", "count": 64, "lo": 1e3, "hi": 2e6, "tuned": True},
        # A burst of served queries, two of each template, over resident tables.
        {"name": "serve_burst", "op": "serve", "n": 40_000_000, "m": 2_000_000, "codes": 100_000, "queries": 8},
    ]


def _log(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    op = rng.choice(["filter", "join", "partition", "topk", "disc", "code", "zipf", "pipeline", "pipeline", "batch",
                     "serve"])
    if op == "filter":
        return {"op": op, "n": _log(rng, 1_000, 200_000_000), "dtype": rng.choice(["i32", "i64"]),
                "sel": rng.random() < 0.4, "keep": round(rng.uniform(0.01, 0.99), 3)}
    if op == "join":
        m = _log(rng, 1_000, 12_000_000)
        return {"op": op, "m": m, "n": min(int(m * rng.uniform(1, 16)), 80_000_000),
                "hit": rng.choice([1.0, 0.9, 0.5])}
    if op == "partition":
        return {"op": op, "n": _log(rng, 10_000, 60_000_000), "log2p": rng.randint(1, 8), "w4": rng.randint(0, 2),
                "w8": rng.randint(0, 3), "rowid": rng.random() < 0.7}
    if op == "topk":
        return {"op": op, "n": _log(rng, 10_000, 150_000_000), "k": _log(rng, 1, 2_048),
                "desc": rng.random() < 0.5, "sel": rng.random() < 0.6}
    if op == "disc":
        return {"op": "groupby", "kind": op, "n": _log(rng, 20_000, 120_000_000), "groups": 11}
    if op == "code":
        n = _log(rng, 20_000, 60_000_000)
        return {"op": "groupby", "kind": op, "n": n, "groups": _log(rng, 20, max(40, min(n // 4, 1_500_000)))}
    if op == "zipf":
        n = _log(rng, 200_000, 50_000_000)
        return {"op": "groupby", "kind": op, "n": n, "groups": max(2_000, int(n * rng.uniform(0.01, 0.04)))}
    if op == "pipeline":
        m = _log(rng, 4_096, 6_000_000)
        return {"op": op, "n": int(m * rng.uniform(8, 16)), "m": m, "groups": _log(rng, 20, max(25, m // 16)),
                "log2p": rng.choice([0, 4, 6, 6, 8]), "topk": rng.choice([0, 10, 100]),
                "date_hi": rng.choice([128, 700, DATE_HI, 2_400]), "streams": rng.choice([1, 1, 2])}
    if op == "batch":
        return {"op": op, "count": rng.randint(4, 96), "lo": 1e3, "hi": _log(rng, 2_000, 1_500_000),
                "tuned": rng.random() < 0.5}
    m = _log(rng, 20_000, 2_000_000)
    return {"op": "serve", "n": int(m * rng.uniform(8, 20)), "m": m, "codes": _log(rng, 1_000, max(2_000, m // 16)),
            "queries": 4 * rng.randint(1, 3)}


# -------------------------------------------------------------------- inputs
def _rows(n):
    return torch.arange(n, dtype=torch.int64, device=DEVICE)


def _fact(case, seed, **kw):
    return synth.fact_table(synth.FactSpec(case["n"], kw.pop("m"), seed, **kw), device=DEVICE)


def _columns(n, seed, names):
    """Fact columns without foreign keys, made in chunks."""
    out = {}
    for name in names:
        dt = torch.int32 if name == "date" else torch.int64
        out[name] = torch.empty(n, dtype=dt, device=DEVICE)
    lim = {"date": (synth.S_DATE, 0, synth.DATE_RANGE - 1), "qty": (synth.S_QTY, synth.QTY_LO, synth.QTY_HI),
           "price": (synth.S_PRICE, synth.PRICE_LO, synth.PRICE_HI),
           "disc": (synth.S_DISC, synth.DISC_LO, synth.DISC_HI)}
    for a in range(0, n, 1 << 26):
        b = min(n, a + (1 << 26))
        rows = torch.arange(a, b, dtype=torch.int64, device=DEVICE)
        for name in names:
            stream, lo, hi = lim[name]
            out[name][a:b] = synth.uniform_int(seed, stream, rows, lo, hi).to(out[name].dtype)
    return out


def _selection(date, hi):
    """(row ids padded to the column's length, their number), as a filter leaves them."""
    rows = torch.nonzero(date < hi).reshape(-1).to(torch.int32)
    sel = torch.zeros(date.numel(), dtype=torch.int32, device=DEVICE)
    sel[:rows.numel()] = rows
    return sel, torch.tensor([rows.numel()], dtype=torch.int64, device=DEVICE)


def _zeros(n, dtype):
    return torch.zeros(max(n, 1), dtype=dtype, device=DEVICE)


class _Groups:
    """Output buffers of `rows` group-bys (a leading axis when rows is given)."""

    def __init__(self, cap, key64, key32, rows=None):
        shape = (cap,) if rows is None else (rows, cap)
        self.key64 = torch.full(shape, I64_MAX, dtype=torch.int64, device=DEVICE) if key64 else None
        self.key32 = torch.full(shape, 0 if key64 else I32_MAX, dtype=torch.int32, device=DEVICE) if key32 else None
        self.vals = torch.zeros((6,) + shape, dtype=torch.int64, device=DEVICE)
        self.n = torch.zeros(1 if rows is None else rows, dtype=torch.int64, device=DEVICE)

    def result(self, r=None):
        at = (lambda t: t) if r is None else (lambda t: None if t is None else t[r])
        v = [at(self.vals[i]) for i in range(6)]
        return gq.GroupResult(at(self.key64), at(self.key32), v[0], v[1], v[2], v[3], v[4].view(torch.float64),
                              v[5].view(torch.float64), self.n if r is None else self.n[r:r + 1])

    def ordered(self):
        """ORDER BY the group key (a composite key's second part is 0 or 1, and
        the first is a 64-bit random key: key64 ^ key32 orders the pairs)."""
        out = {}
        if self.key64 is not None and self.key32 is not None:
            order = torch.argsort(self.key64 ^ self.key32)
            out["key64"], out["key32"] = self.key64[order], self.key32[order]
        elif self.key64 is not None:
            out["key64"], order = torch.sort(self.key64, dim=-1)
        else:
            out["key32"], order = torch.sort(self.key32, dim=-1)
        if order.dim() == 1:
            vals = self.vals.index_select(1, order)
        else:
            vals = self.vals.gather(2, order.expand_as(self.vals))
        for i, f in enumerate(STATS):
            out[f] = vals[i].view(torch.float64) if f.startswith("avg") else vals[i]
        out["n_groups"] = self.n
        return out


# ------------------------------------------------------------------- prepare
def prepare(case, seed):
    ctx = gq.Context(torch.cuda.current_device())
    st = {"case": case, "ctx": ctx}
    _PREPARE[case["op"]](st, case, seed, gq.lib())
    return st


def _filter_inputs(case, seed):
    n = case["n"]
    if case["dtype"] == "i32":
        col, span = _columns(n, seed, ["date"])["date"], synth.DATE_RANGE
        lo = 0
    else:
        col, span = _columns(n, seed, ["price"])["price"], synth.PRICE_HI - synth.PRICE_LO + 1
        lo = synth.PRICE_LO
    hi = lo + int(round(case["keep"] * span))
    sel = _selection(_columns(n, seed + 1, ["date"])["date"], DATE_HI) if case["sel"] else (None, None)
    return col, lo, hi, sel


def _p_filter(st, case, seed, L):
    n = case["n"]
    st["col"], st["lo"], st["hi"], (st["sel"], st["n_sel"]) = _filter_inputs(case, seed)
    st["out"], st["n_out"] = _zeros(n, torch.int32), _zeros(1, torch.int64)
    st["ws"] = st["ctx"].workspace(L.gq_filter_workspace_bytes(n))


def _p_join(st, case, seed, L):
    m, n = case["m"], case["n"]
    keys = int(math.ceil(m / case["hit"]))          # foreign keys reach past the build side: the rest finds no match
    st["fk"] = synth.dim_key(seed, synth.uniform_int(seed, synth.S_FK_ROW, _rows(n), 0, keys - 1))
    st["dim"] = synth.dim_table(m, seed, 1000, device=DEVICE)
    st["table"] = torch.empty(gq.gq_join_table_bytes(m, 0.5), dtype=torch.uint8, device=DEVICE)
    st["ws_build"] = st["ctx"].workspace(L.gq_join_build_workspace_bytes(m, st["table"].numel()))
    st["ws_probe"] = st["ctx"].workspace(L.gq_join_probe_workspace_bytes(n))
    st["prow"], st["pay"], st["n_out"] = _zeros(n, torch.int32), _zeros(n, torch.int32), _zeros(1, torch.int64)


def _p_partition(st, case, seed, L):
    n = case["n"]
    st["key"] = synth.dim_key(seed, synth.uniform_int(seed, synth.S_FK_ROW, _rows(n), 0, max(1, n // 8)))
    cols = [_columns(n, seed + i, ["date"])["date"] for i in range(case["w4"])]
    cols += [_columns(n, seed + i, ["price"])["price"] for i in range(case["w8"])]
    st["cols"] = cols
    st["outs"] = (torch.zeros_like(st["key"]), [torch.zeros_like(c) for c in cols],
                  _zeros(n, torch.int32) if case["rowid"] else None, _zeros((1 << case["log2p"]) + 1, torch.int64))
    st["ws"] = st["ctx"].workspace(L.gq_radix_partition_workspace_bytes(n, case["log2p"]))


def _p_topk(st, case, seed, L):
    n, k = case["n"], case["k"]
    cols = _columns(n, seed, ["price", "date"])
    st["val"] = cols["price"]
    st["sel"], st["n_sel"] = _selection(cols["date"], DATE_HI) if case["sel"] else (None, None)
    st["vo"], st["ro"], st["no"] = _zeros(k, torch.int64), _zeros(k, torch.int32), _zeros(1, torch.int64)
    st["ws"] = st["ctx"].workspace(L.gq_topk_workspace_bytes(n, k))


def _groupby_inputs(case, seed):
    """Keyword arguments of gq_groupby_agg, and which key parts there are."""
    n, kind = case["n"], case["kind"]
    f = _columns(n, seed, ["qty", "price", "disc"] + ([] if kind == "zipf" else ["date"]))
    args = {"qty": f["qty"], "price": f["price"], "disc": f["disc"], "n": n}
    if kind == "disc":
        args.update(key64=f["disc"], key64_by_rowid=True, filter_col=f["date"], filter_lo=0, filter_hi=DATE_HI)
        return args, True, False
    if kind == "code":
        sel, cnt = _selection(f["date"], DATE_HI)
        code = synth.uniform_int(seed, synth.S_DIM_ATTR, _rows(n), 0, case["groups"] - 1).to(torch.int32)
        args.update(rowid=sel, n_dev=cnt, key32=code)
        return args, False, True
    fk = torch.empty(n, dtype=torch.int64, device=DEVICE)
    for a in range(0, n, 1 << 25):
        rows = torch.arange(a, min(n, a + (1 << 25)), dtype=torch.int64, device=DEVICE)
        fk[a:a + rows.numel()] = synth.dim_key(seed, synth.zipf_row(seed, synth.S_FK_ROW, rows, case["groups"]))
    g32 = synth.uniform_int(seed, synth.S_G32, _rows(n), 0, 1).to(torch.int32)
    args.update(key64=fk, key32=g32)
    return args, True, True


def _group_bound(case):
    """The bound a program gives: the known domain (a few groups get some room)."""
    if case["kind"] == "zipf":
        return 2 * case["groups"]
    return max(64, case["groups"])


def _p_groupby(st, case, seed, L):
    args, k64, k32 = _groupby_inputs(case, seed)
    cap = _group_bound(case)
    st["groups"] = _Groups(cap, k64, k32)
    ws = st["ctx"].workspace(L.gq_groupby_workspace_bytes(case["n"], cap, int(k64), int(k32)))
    st["args"] = dict(args, max_groups=cap, out=st["groups"].result(), ws=ws)


def _pipeline_inputs(case, seed):
    return (_fact(case, seed, m=case["m"]), synth.dim_table(case["m"], seed, case["groups"], device=DEVICE))


def _p_pipeline(st, case, seed, L):
    fact, dim = _pipeline_inputs(case, seed)
    cap = max(64, case["groups"])
    pl = PlainPipeline(st["ctx"], fact, dim, case["date_hi"], max_groups=cap, log2_fanout=case["log2p"] or 6,
                       topk=case["topk"], partition=case["log2p"] > 0, streams=case["streams"])
    for t in (pl.sel, pl.prow, pl.pay):
        t.zero_()
    if case["topk"]:
        pl.tk_val.zero_(), pl.tk_row.zero_()
    st["groups"] = _Groups(cap, False, True)
    pl.groups = st["groups"].result()
    st["pl"] = pl


def _p_batch(st, case, seed, L):
    # the instances' sizes are the case's own: only their contents follow the seed
    cols, layout = _batch_tables(case, seed)
    groups = _Groups(64, False, True, rows=len(layout))
    specs = [{"dim_key": cols["dim_key"][mo:mo + m], "dim_attr": cols["dim_attr"][mo:mo + m],
              "fk": cols["fk"][no:no + n], "date": cols["date"][no:no + n], "qty": cols["qty"][no:no + n],
              "price": cols["price"][no:no + n], "disc": cols["disc"][no:no + n], "date_lo": -(1 << 31),
              "date_hi": DATE_HI, "out": groups.result(i)} for i, (mo, m, no, n) in enumerate(layout)]
    st["instances"] = gq.make_instances(specs)
    st["cols"], st["groups"] = cols, groups
    st["tuning"] = None
    if case["tuned"]:                               # as the autotuner leaves it for the batched workload
        t = gq.gq_default_tuning()
        t.load_factor, t.probe_tile, t.build_tile, t.lag, t.fanout = 0.4, 131_072, 16_384, 64, 1
        st["tuning"] = t
    st["status"] = _zeros(len(layout), torch.int32)
    tp = gq.C.byref(st["tuning"]) if st["tuning"] is not None else None
    st["ws"] = st["ctx"].workspace(L.gq_batch_workspace_bytes(st["instances"], len(layout), tp))


def _batch_sizes(case):
    return synth.batch_sizes(synth.BatchSpec(count=case["count"], build_lo=case["lo"], build_hi=case["hi"]))


def _batch_tables(case, seed):
    sizes = _batch_sizes(case)
    M, N = sum(m for m, _ in sizes), sum(n for _, n in sizes)
    cols = {"dim_key": torch.empty(M, dtype=torch.int64, device=DEVICE), "dim_attr": _zeros(M, torch.int32),
            "date": _zeros(N, torch.int32)}
    cols.update({c: torch.empty(N, dtype=torch.int64, device=DEVICE) for c in ("fk", "qty", "price", "disc")})
    layout, mo, no = [], 0, 0
    for i, (m, n) in enumerate(sizes):
        s = seed + 1 + i
        d, f = synth.dim_table(m, s, 25, device=DEVICE), synth.fact_table(synth.FactSpec(n, m, s), device=DEVICE)
        cols["dim_key"][mo:mo + m], cols["dim_attr"][mo:mo + m] = d["key"], d["attr"]
        for c in ("fk", "date", "qty", "price", "disc"):
            cols[c][no:no + n] = f[c]
        layout.append((mo, m, no, n))
        mo, no = mo + m, no + n
    return cols, layout


KINDS = (gq.GQ_QUERY_FILTER_AGG, gq.GQ_QUERY_JOIN_AGG, gq.GQ_QUERY_JOIN2_AGG, gq.GQ_QUERY_FILTER_TOPK)


def _serve_queries(case):
    """(template, date_hi) of the burst: the templates in turn, selectivities spread over 1% to 60%."""
    q = case["queries"]
    return [(KINDS[i % 4], int(round((0.01 + 0.59 * ((i * 5 + 2) % q) / max(1, q - 1)) * synth.DATE_RANGE)))
            for i in range(q)]


def _serve_inputs(case, seed):
    spec = synth.ServeSpec(n=case["n"], m=case["m"], seed=seed, code_range=case["codes"])
    return synth.serve_tables(spec, device=DEVICE)


def _p_serve(st, case, seed, L):
    ctx = st["ctx"]
    fact, dim1, dim2 = _serve_inputs(case, seed)
    t1, t2 = gq.gq_join_build(ctx, dim1["key"], dim1["attr"]), gq.gq_join_build(ctx, dim2["key"], dim2["attr"])
    ctx.raise_status()
    pool = torch.empty(((case["n"] * 100 + (256 << 20)) // 256) * 256, dtype=torch.uint8, device=DEVICE)
    st["server"] = Server(ctx, fact, t1, t2, pool, streams=2, max_batch=16)
    per = case["queries"] // 4
    st["agg"], st["join"], st["join2"] = (_Groups(64, True, False, per), _Groups(case["codes"], False, True, per),
                                          _Groups(64, False, True, per))
    st["tk_val"], st["tk_row"] = _zeros(per * 100, torch.int64).view(per, 100), _zeros(per * 100, torch.int32).view(per, 100)
    st["tk_n"] = _zeros(per, torch.int64)
    st["queries"] = []
    for i, (kind, hi) in enumerate(_serve_queries(case)):
        r = i // 4
        if kind == gq.GQ_QUERY_FILTER_TOPK:
            out, spec = (st["tk_val"][r], st["tk_row"][r], st["tk_n"][r:r + 1]), QuerySpec(kind, hi, k=100)
        else:
            g = {KINDS[0]: st["agg"], KINDS[1]: st["join"], KINDS[2]: st["join2"]}[kind]
            out, spec = g.result(r), QuerySpec(kind, hi, max_groups=g.vals.shape[-1])
        st["queries"].append((spec, out))


_PREPARE = {"filter": _p_filter, "join": _p_join, "partition": _p_partition, "topk": _p_topk,
            "groupby": _p_groupby, "pipeline": _p_pipeline, "batch": _p_batch, "serve": _p_serve}


# ----------------------------------------------------------------------- run
def run(st):
    return _RUN[st["case"]["op"]](st)


def _r_filter(st):
    out, n = gq.gq_filter(st["ctx"], st["col"], st["lo"], st["hi"], sel_in=st["sel"], n_dev=st["n_sel"],
                          out=st["out"], n_out=st["n_out"], ws=st["ws"])
    return {"sel": out, "n": n}


def _r_join(st):
    table = gq.gq_join_build(st["ctx"], st["dim"]["key"], st["dim"]["attr"], table=st["table"], ws=st["ws_build"])
    prow, pay, n = gq.gq_join_probe(st["ctx"], table, st["fk"], prow=st["prow"], payload=st["pay"],
                                    n_out=st["n_out"], ws=st["ws_probe"])
    return {"prow": prow, "payload": pay, "n": n}


def _r_partition(st):
    key, cols, rowid, off = gq.gq_radix_partition(st["ctx"], st["key"], st["case"]["log2p"], st["cols"],
                                                  rowid=st["case"]["rowid"], outs=st["outs"], ws=st["ws"])
    return {"key": key, "cols": cols, "rowid": rowid, "offsets": off}


def _r_topk(st):
    v, r, n = gq.gq_topk(st["ctx"], st["val"], st["case"]["k"], sel=st["sel"], n=st["case"]["n"], n_dev=st["n_sel"],
                         descending=st["case"]["desc"], val_out=st["vo"], rowid_out=st["ro"], n_out=st["no"],
                         ws=st["ws"])
    return {"val": v, "row": r, "n": n}


def _r_groupby(st):
    gq.gq_groupby_agg(st["ctx"], **st["args"])
    return st["groups"].ordered()


def _r_pipeline(st):
    pl = st["pl"]
    pl.step()
    out = {"groups": st["groups"].ordered(), "sel": pl.sel, "n_sel": pl.n_sel, "prow": pl.prow, "payload": pl.pay,
           "n_join": pl.n_join}
    if pl.partition:
        out.update(key=pl.p_key, cols=pl.p_cols, rowid=pl.p_rowid, offsets=pl.p_off)
    if pl.k:
        out.update(tk_val=pl.tk_val, tk_row=pl.tk_row, tk_n=pl.tk_n)
    return out


def _r_batch(st):
    gq.gq_batch_join_agg(st["ctx"], st["instances"], st["tuning"], ws=st["ws"], inst_status=st["status"])
    return dict(st["groups"].ordered(), status=st["status"])


def _r_serve(st):
    srv = st["server"]
    subs = [srv.submit(spec, out=out) for spec, out in st["queries"]]
    for s in subs:
        srv.wait(s)
    return {"status": [s.status for s in subs], "agg": st["agg"].ordered(), "join": st["join"].ordered(),
            "join2": st["join2"].ordered(), "topk": {"val": st["tk_val"], "row": st["tk_row"], "n": st["tk_n"]}}


_RUN = {"filter": _r_filter, "join": _r_join, "partition": _r_partition, "topk": _r_topk, "groupby": _r_groupby,
        "pipeline": _r_pipeline, "batch": _r_batch, "serve": _r_serve}


# ---------------------------------------------------------------------- work
def _expected_groups(case):
    """Groups that come out: about all of a small domain, about 0.9 of the Zipf ranks' pairs."""
    return case["groups"] * (1.3 if case.get("kind") == "zipf" else 1.0)


def work(case):
    """Bytes of the inputs that are read and of the outputs that are written, each once; integer work only."""
    op, n = case["op"], case.get("n", 0)
    if op == "filter":
        rows = n * (SEL_FRAC if case["sel"] else 1.0)
        b = rows * ((4 if case["dtype"] == "i32" else 8) + (4 if case["sel"] else 0)) + 4 * rows * case["keep"]
    elif op == "join":
        b = 12 * case["m"] + 8 * n + 8 * n * case["hit"]
    elif op == "partition":
        row = 8 + 4 * case["w4"] + 8 * case["w8"]
        b = n * (2 * row + (4 if case["rowid"] else 0))
    elif op == "topk":
        b = n * SEL_FRAC * 12 if case["sel"] else n * 8
    elif op == "groupby":
        rows, key = {"disc": (n * SEL_FRAC, 0), "code": (n * SEL_FRAC, 8), "zipf": (n, 12)}[case["kind"]]
        b = rows * (24 + key) + (4 * n if case["kind"] == "disc" else 0) + 60 * _expected_groups(case)
    elif op == "pipeline":
        s = n * case["date_hi"] / synth.DATE_RANGE
        b = 12 * case["m"] + 36 * n + 4 * s + 8 * s + 52 * min(case["groups"], s)
        b += 40 * n if case["log2p"] else 0
    elif op == "batch":
        b = sum(12 * m + 4 * r + 32 * r * SEL_FRAC for m, r in _batch_sizes(case))
    else:
        b = 44 * n + 16 * 2 * case["m"] + 52 * case["codes"] * case["queries"] / 4
    return {"bytes": float(b), "flops": 0.0}


# --------------------------------------------------------------------- exact
def _agg(idx, cnt_groups, qty, rev):
    z = lambda: torch.zeros(cnt_groups, dtype=torch.int64, device=DEVICE)  # noqa: E731
    c = z().index_add_(0, idx, torch.ones_like(idx))
    return c, z().index_add_(0, idx, qty), z().index_add_(0, idx, rev)


def _averages(c, q, r, cap):
    """The averages of the groups that exist, in key order, as the buffers hold them."""
    have = c > 0
    out = {}
    for name, s in (("avg_qty", q), ("avg_rev", r)):
        v = torch.zeros(cap, dtype=torch.float64, device=DEVICE)
        v[:int(have.sum())] = (s[have].to(torch.float64) / c[have].to(torch.float64))[:cap]
        out[name] = v
    return out


def _lookup(dim, fk):
    """The attribute of each foreign key, by binary search over the sorted keys."""
    keys, order = torch.sort(dim["key"])
    at = torch.searchsorted(keys, fk).clamp_(max=keys.numel() - 1)
    return dim["attr"][order[at]].to(torch.int64)


def exact(case, seed):
    op = case["op"]
    if op == "groupby":
        a, _, _ = _groupby_inputs(case, seed)
        cap = _group_bound(case)
        if case["kind"] == "zipf":
            _, idx = torch.unique(a["key64"] ^ a["key32"], return_inverse=True)
            rows = slice(None)
        elif case["kind"] == "disc":
            rows = torch.nonzero(a["filter_col"] < DATE_HI).reshape(-1)
            idx = a["key64"][rows]
        else:
            rows = a["rowid"][:int(a["n_dev"])].long()
            idx = a["key32"][:rows.numel()].long()
        rev = (a["price"] * (100 - a["disc"]))[rows]
        return _averages(*_agg(idx, max(int(idx.max()) + 1, cap), a["qty"][rows], rev), cap)
    if op == "pipeline":
        f, d = _pipeline_inputs(case, seed)
        rows = torch.nonzero(f["date"] < case["date_hi"]).reshape(-1)
        idx = _lookup(d, f["fk"][rows])
        cap = max(64, case["groups"])
        rev = (f["price"] * (100 - f["disc"]))[rows]
        return {"groups": _averages(*_agg(idx, cap, f["qty"][rows], rev), cap)}
    if op == "batch":
        cols, layout = _batch_tables(case, seed)
        got = {"avg_qty": [], "avg_rev": []}
        for mo, m, no, n in layout:
            rows = torch.nonzero(cols["date"][no:no + n] < DATE_HI).reshape(-1) + no
            idx = _lookup({"key": cols["dim_key"][mo:mo + m], "attr": cols["dim_attr"][mo:mo + m]}, cols["fk"][rows])
            v = _averages(*_agg(idx, 64, cols["qty"][rows], cols["price"][rows] * (100 - cols["disc"][rows])), 64)
            for k in got:
                got[k].append(v[k])
        return {k: torch.stack(v) for k, v in got.items()}
    if op == "serve":
        f, d1, d2 = _serve_inputs(case, seed)
        rev = f["price"] * (100 - f["disc"])
        ids = {KINDS[0]: f["disc"], KINDS[1]: _lookup(d1, f["fk"]), KINDS[2]: _lookup(d2, f["fk2"])}
        names = {KINDS[0]: "agg", KINDS[1]: "join", KINDS[2]: "join2"}
        got = {name: {"avg_qty": [], "avg_rev": []} for name in names.values()}
        for kind, hi in _serve_queries(case):
            if kind in names:
                cap = case["codes"] if kind == KINDS[1] else 64
                rows = torch.nonzero(f["date"] < hi).reshape(-1)
                v = _averages(*_agg(ids[kind][rows], cap, f["qty"][rows], rev[rows]), cap)
                for k in v:
                    got[names[kind]][k].append(v[k])
        return {name: {k: torch.stack(x) for k, x in v.items()} for name, v in got.items()}
    return None                                     # the other operators return whole numbers only
