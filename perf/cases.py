"""The work this library is used for, as cases that can be timed one by one.

Each case is one pass through the public entry points: a star query with its
dimension builds, the Q1.1-shaped scan, a shared-scan batch, a served burst,
selection (in input order, and unordered followed by ORDER BY), projection, a
hash join with its build, the dense group-by, and radix sort and partition.
Sizes are those of the benchmark's workloads and of smaller tables of the same
shapes; odd row counts are among them because real tables have them.

Inputs are drawn on the GPU from the seed alone, with the distributions of
``paper_2003_01178_amd.datagen`` (uniform keys, measures and constants; the
dimension tables come from that module itself).
"""
import math
import time
from types import SimpleNamespace

import numpy as np
import torch

from paper_2003_01178_amd import crystal as cx
from paper_2003_01178_amd import datagen, queries

DEV = "cuda"
LINE = 32          # int32 values of a 128-byte memory line
SEGMENTS = 8       # clock steps a served table is cut into


def listed():
    return [
        # the benchmark's default workload: four filtered dimension builds, then one fused kernel over 120M rows
        {"name": "star_120m", "kind": "star", "rows": 120_000_000, "template": "q2", "columns": "int32"},
        # the same query over a small table with compressed columns (a day's load): launches and latency count
        {"name": "star_packed_1m", "kind": "star", "rows": 1_000_003, "template": "q2", "columns": "packed"},
        # the Q1.1-shaped scan at scale factor 1: a short scalar query, run over and over
        {"name": "q11_6m", "kind": "q11", "rows": 6_000_000, "flight": 1},
        # one clock segment of the served 600M-row table: 16 star queries answered in one pass, with their mask builds
        {"name": "scan_star_75m", "kind": "scan", "rows": 75_000_000, "template": "star", "queries": 16},
        # a burst of mixed queries submitted to the server at once and awaited
        {"name": "serve_burst_60m", "kind": "serve", "rows": 60_000_000, "queries": 32},
        # selection in input order from a ragged column, half of it qualifying
        {"name": "select_stable_64m", "kind": "select", "rows": 64_000_003, "percent": 50},
        # SELECT y WHERE y < v ORDER BY y: unordered selection, then a sort of the tenth that qualifies
        {"name": "order_by_32m", "kind": "order_by", "rows": 1 << 25, "percent": 10},
        # projection over two large columns
        {"name": "project_256m", "kind": "project", "rows": 1 << 28, "sigmoid": False},
        # hash join of 2^27 rows with a million-row dimension, build included (linear probing, table beyond an L2)
        {"name": "join_1m_128m", "kind": "join", "dim": 1 << 20, "rows": 1 << 27, "table": "linear", "payload": False},
        # dense group-by into the star query's 7,000 groups
        {"name": "groupby_7k_64m", "kind": "groupby", "rows": 1 << 26, "groups": 7000},
        # the benchmark's sort: 2^28 key/value pairs, most significant digit first
        {"name": "sort_msb_256m", "kind": "radix", "op": "sort_msb", "rows": 1 << 28, "values": True, "key_bits": 32},
        # a small sort, such as the result of a query, with the default entry point
        {"name": "sort_lsb_100k", "kind": "radix", "op": "sort", "rows": 100_003, "values": True, "key_bits": 32},
    ]


def _log_int(rng, lo, hi):
    """A whole number between lo and hi, uniform in its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["star", "star", "q11", "scan", "serve", "select", "order_by", "project", "join", "join",
                       "groupby", "radix", "radix"])
    if kind == "star":
        return {"kind": kind, "rows": _log_int(rng, 300_000, 120_000_000),
                "template": rng.choice(["q2", "q2", "q3", "q4"]),
                "columns": rng.choice(["int32", "int32", "packed", "narrow"])}
    if kind == "q11":
        return {"kind": kind, "rows": _log_int(rng, 300_000, 120_000_000), "flight": rng.randint(1, 3)}
    if kind == "scan":
        return {"kind": kind, "rows": _log_int(rng, 1_000_000, 75_000_000), "template": rng.choice(["star", "q11"]),
                "queries": rng.randint(1, 16)}
    if kind == "serve":
        return {"kind": kind, "rows": _log_int(rng, 8_000_000, 60_000_000), "queries": rng.randint(4, 32)}
    if kind == "select":
        return {"kind": kind, "rows": _log_int(rng, 100_000, 1 << 28), "percent": rng.randint(0, 100)}
    if kind == "order_by":
        return {"kind": kind, "rows": _log_int(rng, 100_000, 1 << 26), "percent": rng.randint(1, 50)}
    if kind == "project":
        return {"kind": kind, "rows": _log_int(rng, 100_000, 1 << 28), "sigmoid": rng.random() < 0.5}
    if kind == "join":
        return {"kind": kind, "dim": _log_int(rng, 1 << 10, 1 << 23), "rows": _log_int(rng, 1 << 18, 1 << 27),
                "table": rng.choice(["linear", "linear", "direct"]), "payload": rng.random() < 0.3}
    if kind == "groupby":
        return {"kind": kind, "rows": _log_int(rng, 100_000, 1 << 28), "groups": _log_int(rng, 7, 200_000)}
    return {"kind": kind, "op": rng.choice(["sort", "sort_msb", "partition"]), "rows": _log_int(rng, 30_000, 1 << 27),
            "values": rng.random() < 0.75, "key_bits": rng.choice([32, 32, 20])}


# ------------------------------------------------------------------ inputs --
class _Draws:
    """Columns drawn on the GPU, one generator per case."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(seed)
        self.host = np.random.default_rng(seed)

    def ints(self, lo, hi, n):
        """n int32 values uniform on [lo, hi]."""
        return torch.randint(lo, hi + 1, (n,), generator=self.g, device=DEV, dtype=torch.int32)

    def floats(self, n):
        return torch.rand(n, generator=self.g, device=DEV, dtype=torch.float32)

    def words(self, bits, n):
        """n unsigned `bits`-bit words, as int32 bit patterns."""
        if bits < 32:
            return self.ints(0, (1 << bits) - 1, n)
        return torch.randint(-(1 << 31), 1 << 31, (n,), generator=self.g, device=DEV, dtype=torch.int32)


def _schema(n, seed, d, served=False):
    """A star schema with its dimension tables, and n fact rows drawn on the GPU."""
    dims, consts = datagen.star_dims(seed)
    none = np.zeros(0, np.int32)
    s = queries.StarSchema(datagen.StarTables(fk=[none] * 4, m1=none, m2=none, dims=dims, consts=consts), device=DEV)
    days = torch.from_numpy(datagen.day_keys()[0]).to(DEV)
    s.n = n
    s.day = d.ints(0, datagen.N_DAYS - 1, n)
    s.fk = [days[s.day]] + [d.ints(0, rows - 1, n) for rows in datagen.DIM_ROWS[1:]]
    s.m1, s.m2 = d.ints(1, 1_000_000, n), d.ints(1, 1_000_000, n)
    if served:
        s.extra = {"discount": d.ints(0, 10, n), "quantity": d.ints(1, 50, n), "price": d.ints(90_000, 10_000_000, n)}
        s.col_range = {"datekey": (int(days.min()), int(days.max())), "discount": (0, 10), "quantity": (1, 50),
                       "price": (90_000, 10_000_000)}
    return s


def _star(case, seed, d):
    s = _schema(case["rows"], seed, d)
    if case["template"] == "q2":
        items, plan = s.build_items(), s.plan()
    else:   # flights 3 and 4 probe tables that are built once, with payload filters
        f = queries.FlightTemplates(s)
        items = []
        plan = (f.q3 if case["template"] == "q3" else f.q4)(s.consts[1] % 23, s.consts[3] % 21)
    cols, joins = list(plan.cols), [dict(j) for j in plan.joins]
    if case["columns"] == "narrow":
        cols[1], _ = cx.pack_column(s.fk[1], 0, 2)
    elif case["columns"] == "packed":
        # dates as 12-bit day codes, with the date table keyed by the code; fk1 in 16 bits
        cols[0], _ = cx.pack_column_bits(s.day, 0, 12)
        cols[1], _ = cx.pack_column_bits(s.fk[1], 0, 16)
        d0 = s.dims[0]
        codes = torch.from_numpy(datagen.day_codes(d0["key"].cpu().numpy())).to(DEV)
        table = cx.HashTable(cx.HT_DIRECT, d0["n"], 0, datagen.N_DAYS - 1, has_payload=True)
        if items:
            items[0] = (table, codes, *items[0][2:])
        else:
            table.build(codes, payload=d0["packed"], status=s.status)
        joins = [dict(j, table=table) if j["fk_col"] == 0 else j for j in joins]
    plan = cx.StarQuery(cols, n_groups=plan.n_groups, joins=joins, agg=plan.c.agg,
                        agg_cols=(plan.c.agg_col0, plan.c.agg_col1))
    return dict(items=items, plan=plan, keep=s, out=torch.zeros(plan.n_groups, dtype=torch.int64, device=DEV),
                status=cx.new_status())


def _q11(case, seed, d):
    n = case["rows"]
    days = torch.from_numpy(datagen.day_keys()[0]).to(DEV)
    cols = (days[d.ints(0, datagen.N_DAYS - 1, n)], d.ints(0, 10, n), d.ints(1, 50, n), d.ints(90_000, 10_000_000, n))
    year = datagen.FIRST_YEAR + int(d.host.integers(0, 7))
    return dict(plan=queries.q1x_plan(cols, case["flight"], year=year),
                out=torch.zeros(1, dtype=torch.int64, device=DEV), status=cx.new_status())


def _scan(case, seed, d):
    sv = queries.ServingTemplates(_schema(case["rows"], seed, d, served=True))
    k = case["queries"]
    star = case["template"] == "star"
    consts = [datagen.random_star_constants(d.host) if star else datagen.random_q11_constants(d.host)
              for _ in range(k)]
    out = torch.zeros((k, queries.STAR_GROUPS if star else 1), dtype=torch.int64, device=DEV)
    return dict(sv=sv, consts=consts, out=out, outs=list(out), star=star, status=cx.new_status())


def _serve(case, seed, d):
    sv = queries.ServingTemplates(_schema(case["rows"], seed, d, served=True))
    torch.cuda.synchronize()
    seg = (case["rows"] // SEGMENTS + 3) // 4 * 4
    srv = cx.Server(sv.server_templates(), slots=16, segment_rows=seg, max_queue=1 << 16, inflight=2)
    asked = [(0, sv.star_request(datagen.random_star_constants(d.host))) if k % 2 == 0 else
             (1, sv.q11_request(*datagen.random_q11_constants(d.host))) for k in range(case["queries"])]
    return dict(server=srv, asked=asked, keep=sv)


def _select(case, seed, d):
    n = case["rows"]
    lo, hi = datagen.select_threshold_range(case["percent"] / 100)
    scratch = torch.empty(cx.load().crystal_select_stable_scratch_bytes(n), dtype=torch.uint8, device=DEV)
    return dict(x=d.ints(0, 2 ** 31 - 2, n), lo=lo, hi=hi, out=torch.zeros(n, dtype=torch.int32, device=DEV),
                count=torch.zeros(1, dtype=torch.int64, device=DEV), scratch=scratch)


def _order_by(case, seed, d):
    st = _select(case, seed, d)
    n = case["rows"]
    st["scratch"] = torch.empty(cx.load().crystal_sort_pairs_scratch_bytes(n, 0), dtype=torch.uint8, device=DEV)
    st["sorted"] = torch.zeros(n, dtype=torch.int32, device=DEV)
    return st


def _project(case, seed, d):
    n = case["rows"]
    a, b = (float(np.float32(v)) for v in d.host.uniform(-4.0, 4.0, 2))
    return dict(x1=d.floats(n), x2=d.floats(n), a=a, b=b, sigmoid=case["sigmoid"],
                out=torch.empty(n, dtype=torch.float32, device=DEV))


def _join(case, seed, d):
    dim, n = case["dim"], case["rows"]
    key = torch.randperm(dim, generator=d.g, device=DEV).to(torch.int32)
    kind = cx.HT_LINEAR if case["table"] == "linear" else cx.HT_DIRECT
    return dict(table=cx.HashTable(kind, dim, 0, dim - 1, has_payload=True), key=key, val=d.ints(0, 2 ** 31 - 2, dim),
                fk=d.ints(0, dim - 1, n), payload=d.ints(0, 1_000_000, n) if case["payload"] else None,
                status=cx.new_status(), out=torch.zeros(2, dtype=torch.int64, device=DEV))


def _groupby(case, seed, d):
    n, groups = case["rows"], case["groups"]
    return dict(group=d.ints(0, groups - 1, n), value=d.ints(1, 1_000_000, n), groups=groups,
                out=torch.zeros(groups, dtype=torch.int64, device=DEV), status=cx.new_status())


def _radix(case, seed, d):
    n, vals = case["rows"], case["values"]
    lib = cx.load()
    nbytes = {"partition": lambda: lib.crystal_radix_partition_scratch_bytes(n),
              "sort": lambda: lib.crystal_sort_pairs_scratch_bytes(n, int(vals)),
              "sort_msb": lambda: lib.crystal_sort_pairs_msb_scratch_bytes(n, int(vals))}[case["op"]]()
    return dict(op=case["op"], keys=d.words(case["key_bits"], n), vals=d.words(32, n) if vals else None,
                shift=case["key_bits"] - 8, out_keys=torch.zeros(n, dtype=torch.int32, device=DEV),
                out_vals=torch.zeros(n, dtype=torch.int32, device=DEV) if vals else None,
                parts=torch.zeros(257, dtype=torch.int32, device=DEV),
                scratch=torch.empty(max(256, nbytes), dtype=torch.uint8, device=DEV))


_PREPARE = {"star": _star, "q11": _q11, "scan": _scan, "serve": _serve, "select": _select, "order_by": _order_by,
            "project": _project, "join": _join, "groupby": _groupby, "radix": _radix}


def prepare(case, seed):
    return SimpleNamespace(kind=case["kind"], **_PREPARE[case["kind"]](case, seed, _Draws(seed)))


# --------------------------------------------------------------------- run --
def run(s):
    return _RUN[s.kind](s)


def _run_star(s):
    if s.items:
        cx.build_tables(s.items, status=s.status)
    s.plan.run(out=s.out, status=s.status)
    return {"groups": s.out, "status": s.status}


def _run_q11(s):
    s.plan.run(out=s.out, status=s.status)
    return {"sum": s.out, "status": s.status}


def _run_scan(s):
    s.out.zero_()       # a pass accumulates
    if s.star:
        s.sv.build_star_masks(s.consts)
        s.sv.run_star_batch(s.outs, status=s.status)
    else:
        s.sv.run_q11_batch(s.consts, s.outs, status=s.status)
    return {"out": s.out, "status": s.status}


def _run_serve(s):
    tickets = [s.server.submit(t, **request) for t, request in s.asked]
    got = []
    for tk in tickets:
        while True:
            done, out, _ = s.server.poll(tk)
            if done:
                break
            time.sleep(5e-5)
        got.append(out)
    return {"star": np.stack(got[0::2]), "q11": np.stack(got[1::2])}


def _run_select(s):
    cx.select(s.x, s.lo, s.hi, out=s.out, count=s.count, stable=True, scratch=s.scratch)
    return {"out": s.out, "count": s.count}


def _run_order_by(s):
    cx.select(s.x, s.lo, s.hi, out=s.out, count=s.count)
    n = int(s.count.item())     # the sort's size is a host argument
    cx.sort_pairs(s.out[:n], out_keys=s.sorted, scratch=s.scratch)
    return {"sorted": s.sorted, "count": n}


def _run_project(s):
    return cx.project(s.x1, s.x2, s.a, s.b, out=s.out, sigmoid=s.sigmoid)


def _run_join(s):
    s.table.build(s.key, payload=s.val, status=s.status)
    s.table.probe(s.fk, probe_payload=s.payload, out=s.out)
    return {"sum_and_matches": s.out, "status": s.status}


def _run_groupby(s):
    cx.groupby_agg(s.group, s.value, s.groups, out=s.out, status=s.status)
    return {"sums": s.out, "status": s.status}


def _run_radix(s):
    if s.op == "partition":
        cx.radix_partition(s.keys, s.shift, 8, vals=s.vals, out_keys=s.out_keys, out_vals=s.out_vals,
                           part_offsets=s.parts, scratch=s.scratch)
        return {"keys": s.out_keys, "values": s.out_vals, "parts": s.parts}
    cx.sort_pairs(s.keys, s.vals, out_keys=s.out_keys, out_vals=s.out_vals, scratch=s.scratch, msb=s.op == "sort_msb")
    return {"keys": s.out_keys, "values": s.out_vals}


_RUN = {"star": _run_star, "q11": _run_q11, "scan": _run_scan, "serve": _run_serve, "select": _run_select,
        "order_by": _run_order_by, "project": _run_project, "join": _run_join, "groupby": _run_groupby,
        "radix": _run_radix}


# -------------------------------------------------------------------- work --
def _line(p):
    """Bytes per row of an int32 column read only where a row is alive, each alive with probability p: a row's
    share of the 128-byte lines that hold one."""
    return 4 * (1 - (1 - p) ** LINE)


def work(case):
    kind, n = case["kind"], case["rows"]
    if kind == "star":
        first = {"int32": (4, 4), "narrow": (4, 2), "packed": (1.5, 2)}[case["columns"]]
        dims = sum(datagen.DIM_ROWS)
        # probability that a row is alive after each join in plan order, and the columns read with it
        alive = {"q2": (1 / 25, 1 / 25 ** 2, 1 / 25 ** 3, 1 / 25 ** 4),
                 "q3": (1 / 25, 5 / 25 ** 2, 6 / 7 * 5 / 25 ** 2, 6 / 7 * 5 / 25 ** 2),
                 "q4": (3 / 25, 2 / 7 * 3 / 25, 2 / 7 * 3 / 25 ** 2, 2 / 7 * 3 / 25 ** 2 * 13 / 25)}[case["template"]]
        measures = 2 if case["template"] == "q4" else 1
        per_row = first[1] + sum(_line(p) for p in alive[:3]) + measures * _line(alive[3])
        if case["columns"] == "packed" and case["template"] != "q3":
            per_row += (first[0] / 4 - 1) * _line(alive[0])     # the date column follows the first join
        groups = {"q2": 7000, "q3": 56_000, "q4": 112}[case["template"]]
        # the builds read every dimension's key and filter, and a group attribute of two of them
        builds = 8 * dims if case["template"] == "q2" else 0
        return {"bytes": n * per_row + builds + 8 * groups, "flops": n}
    if kind == "q11":
        p = {1: (1 / 7, 1 / 7 * 3 / 11, 1 / 7 * 3 / 11 * 24 / 50),
             2: (1 / 84, 1 / 84 * 3 / 11, 1 / 84 * 3 / 11 / 5),
             3: (1 / 365, 1 / 365 * 3 / 11, 1 / 365 * 3 / 11 / 5)}[case["flight"]]
        return {"bytes": n * (4 + sum(_line(x) for x in p)) + 8, "flops": n}
    if kind in ("scan", "serve"):
        def some(p, k):
            return 1 - (1 - p) ** k

        def star(k):
            return 4 + sum(_line(some(1 / 25 ** i, k)) for i in (1, 2, 3, 4))

        def q11(k):
            return 4 + sum(_line(some(p, k)) for p in (1 / 7, 1 / 7 * 3 / 11, 1 / 7 * 3 / 11 / 2))

        k = case["queries"]
        if kind == "scan":
            per_row, out = (star(k), 8 * 7000 * k) if case["template"] == "star" else (q11(k), 8 * k)
        else:
            per_row, out = star(min(16, (k + 1) // 2)) + q11(min(16, max(1, k // 2))), 8 * 7000 * ((k + 1) // 2)
        return {"bytes": n * per_row + out, "flops": n}
    if kind == "select":
        return {"bytes": n * 4 * (1 + case["percent"] / 100), "flops": n}
    if kind == "order_by":
        return {"bytes": n * 4 * (1 + case["percent"] / 100), "flops": n}
    if kind == "project":
        return {"bytes": 12 * n, "flops": 3 * n}
    if kind == "join":
        return {"bytes": n * (8 if case["payload"] else 4) + 16 * case["dim"], "flops": n}
    if kind == "groupby":
        return {"bytes": 8 * n + 8 * case["groups"], "flops": n}
    return {"bytes": n * (16 if case["values"] else 8), "flops": n}


def exact(case, seed):
    """The projection's value in 64 bits; every other output is a whole number."""
    if case["kind"] != "project":
        return None
    s = prepare(case, seed)
    t = s.a * s.x1.double() + s.b * s.x2.double()
    return 1 / (1 + torch.exp(-t)) if s.sigmoid else t
