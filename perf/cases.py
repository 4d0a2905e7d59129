"""Performance cases of the library: the queries a program built on it runs, through the public calls of the binding.

Four kinds of work, told apart by a case's "kind":

  predict  star join fused with a linear operator or ReLU MLP (lq_project_dims, lq_fused_join_predict), or the non-fused
           pipeline of the same query (lq_materialized_join_predict)
  group    filtered star join with GROUP BY and SUM / COUNT (lq_masked_groupby_sum); from raw key values where "keys" says
           so (lq_keymap*_lookup first, lq_order_groups on the result)
  agg      the wider aggregate: fact range predicates, computed measures, SUM / COUNT / MIN / MAX (lq_groupby_agg)
  tree     star join fused with a decision tree (lq_tree_*, lq_fused_join_tree, lq_fused_join_tree_masks)

Sizes are those of the repository's own configurations and of the benchmark schemas they follow: fact tables from a
serving batch of a few thousand rows to 1e8, dimensions of 50 to 1e6 rows, joined widths of 16 to 2,048 columns.
"refresh" says whether the dimension side is new in every pass (the pre-fused tables are then built in the pass) or
unchanged since earlier queries (a program keeps the tables, and so does the state).
"""
import math

import numpy as np
import torch

import paper_2306_08367_amd as lq

DEV = "cuda"


def _predict(name, n, c_f, rows, cols, layers, **more):
    case = {"kind": "predict", "n": n, "c_f": c_f, "rows": rows, "cols": cols, "layers": layers, "dtype": "f32", "bias": False,
            "fk": "uniform", "refresh": True, "fused": True}
    if name:
        case["name"] = name
    case.update(more)
    return case


def _group(name, n, sf, **more):
    """n fact rows over the four dimensions of a benchmark schema at scale factor sf; g_*: values of the grouping
    attribute of a dimension (0: does not group), s_*: share of its rows that its predicate keeps (1: no predicate)."""
    case = {"kind": "group", "n": n, "sf": sf, "g_date": 7, "g_cust": 0, "g_supp": 0, "g_part": 0, "s_date": 1.0, "s_cust": 1.0,
            "s_supp": 1.0, "s_part": 1.0, "measures": 1, "fact_mask": False, "keys": "rows", "refresh": False}
    if name:
        case["name"] = name
    case.update(more)
    return case


def _agg(name, n, joins, op, **more):
    case = {"kind": "agg", "n": n, "joins": joins, "op": op, "preds": 2, "group": 0, "min_max": False}
    if name:
        case["name"] = name
    case.update(more)
    return case


def _tree(name, n, rows, columns, leaves, **more):
    case = {"kind": "tree", "n": n, "rows": rows, "columns": columns, "leaves": leaves, "c_f": 0, "form": "masks", "onehot": False,
            "refresh": False}
    if name:
        case["name"] = name
    case.update(more)
    return case


def listed():
    return [
        # Linear regression over a tiny star, table refresh and scoring: nothing but calls and launches.
        _predict("tiny_linear", 10_000, 4, "100,50", "8,8", "1"),
        # Online scoring: one batch of 4,099 requests against tables that are kept, a three-layer model with biases.
        _predict("serving_batch", 4_099, 5, "1000,10000,2556", "32,32,32", "64,32,1", bias=True, refresh=False),
        # The headline: a two-layer MLP over ten million fact rows.
        _predict("mlp_1e7", 10_000_000, 4, "1000,10000,100000", "32,32,32", "64,1"),
        # Skewed keys into two dimensions of a million rows each, four linear outputs, 1e8 fact rows.
        _predict("linear_skewed_1e8", 100_000_000, 8, "1000000,1000000", "128,128", "4", fk="zipf"),
        # The wide bf16 model: 1,024 joined columns, 256 hidden units, 16 outputs, 5e7 rows. The largest.
        _predict("wide_bf16_5e7", 50_000_000, 0, "10000,10000,10000,10000", "256,256,256,256", "256,16", dtype="bf16"),
        # A wide linear operator over small tables, where refreshing the pre-fused tables is most of the query.
        _predict("wide_operator", 12_000, 0, "6000,8000,2555", "683,683,682", "2048"),
        # A narrow star under a wide operator: the query for which the non-fused pipeline is the advised one.
        _predict("non_fused", 600_000, 0, "20000,2000,2555", "6,5,5", "128", fused=False, refresh=False),
        # Four joins, two predicates, GROUP BY year x nation at scale factor 1.
        _group("group_by_sf1", 6_000_000, 1, g_cust=25, s_supp=0.2, s_part=0.12),
        # GROUP BY year x nation x brand at scale factor 4: 175,000 groups, a fifth of the rows survive, two measures.
        _group("group_by_many_sf4", 24_000_000, 4, g_cust=25, g_part=1000, s_supp=0.2, measures=2),
        # The same schema from raw key values: four key columns mapped through kept domains, group-by, ORDER BY.
        _group("keyed_query_sf1", 6_000_000, 1, g_part=1000, s_supp=0.2, s_part=0.04, keys="sparse"),
        # One join, two range predicates on the fact table, SUM(a * b).
        _agg("agg_one_join", 6_000_000, 1, "mul"),
        # Decision tree of 64 leaves over 128 joined columns, an odd number of fact rows, tables kept as leaf masks.
        _tree("tree_64_leaves", 4_799_999, "80000,16000,2555", 128, 64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["linear", "mlp", "mlp", "bf16", "operator", "non_fused", "group", "group", "keyed", "agg", "tree", "tree"])
    if kind == "linear":
        K = rng.randint(1, 4)
        return _predict(None, _log_int(rng, 1e4, 5e7), rng.randint(0, 8), ",".join(str(_log_int(rng, 50, 1e6)) for _ in range(K)),
                        ",".join(str(rng.choice([8, 16, 31, 64, 128])) for _ in range(K)), str(rng.choice([1, 1, 2, 4])),
                        bias=rng.random() < 0.5, fk=rng.choice(["uniform", "zipf"]), refresh=rng.random() < 0.5)
    if kind == "mlp":
        K = rng.randint(2, 4)
        hidden = rng.choice([16, 32, 50, 64, 64, 100, 128])
        layers = [hidden] + rng.choice([[1], [1], [4], [16], [32, 1], [64, 1], [hidden, hidden, 1]])
        return _predict(None, _log_int(rng, 4e3, 1e7), rng.randint(0, 12), ",".join(str(_log_int(rng, 100, 1e5)) for _ in range(K)),
                        ",".join(str(rng.choice([8, 17, 32, 64])) for _ in range(K)), ",".join(str(x) for x in layers),
                        bias=rng.random() < 0.5, refresh=rng.random() < 0.5)
    if kind == "bf16":
        K = rng.randint(2, 4)
        layers = [rng.choice([64, 128, 200, 256])] + rng.choice([[1], [16], [16], [64, 16]])
        return _predict(None, _log_int(rng, 4e3, 2e7), rng.choice([0, 0, 4]), ",".join(str(_log_int(rng, 1e3, 2e4)) for _ in range(K)),
                        ",".join(str(rng.choice([64, 128, 256])) for _ in range(K)), ",".join(str(x) for x in layers), dtype="bf16",
                        bias=rng.random() < 0.5, refresh=rng.random() < 0.5)
    if kind == "operator":
        sf, k = rng.randint(1, 4), rng.choice([256, 500, 1024, 2048])
        rows = (2_000 * (1 + int(math.log2(sf))), 2_000 * sf, 2_555)
        return _predict(None, 3_000 * sf + rng.randint(0, 99), 0, ",".join(map(str, rows)), "%d,%d,%d" % (k - 2 * (k // 3), k // 3, k // 3),
                        str(_log_int(rng, 16, k)), refresh=rng.random() < 0.7)
    if kind == "non_fused":
        k = rng.choice([16, 32, 64, 100])
        return _predict(None, _log_int(rng, 1e4, 2.4e6), 0, "%d,%d,2555" % (_log_int(rng, 2e3, 8e4), _log_int(rng, 1e3, 2e4)),
                        "%d,%d,%d" % (k - 2 * (k // 3), k // 3, k // 3), str(_log_int(rng, 16, 128)), fused=False, refresh=False)
    if kind in ("group", "keyed"):
        n = _log_int(rng, 6e4, 4.8e7 if kind == "group" else 1.2e7)
        case = _group(None, n, max(1, min(8, round(n / 6e6))), g_date=rng.choice([0, 7, 7]), g_cust=rng.choice([0, 25, 25, 250]),
                      g_part=rng.choice([0, 0, 25, 1000]), s_cust=rng.choice([1.0, 1.0, 0.2]), s_supp=rng.choice([1.0, 0.2, 0.2]),
                      s_part=rng.choice([1.0, 0.2, 0.12, 0.04]), measures=rng.choice([1, 1, 2]), fact_mask=rng.random() < 0.2)
        if kind == "keyed":
            case.update(keys=rng.choice(["dense", "sparse", "sparse64"]), refresh=rng.random() < 0.3)
        if case["g_date"] + case["g_cust"] + case["g_part"] == 0 and rng.random() < 0.8:
            case["g_supp"] = 25
        return case
    if kind == "agg":
        return _agg(None, _log_int(rng, 6e4, 2.4e7), rng.randint(1, 4), rng.choice(["col", "mul", "sub"]), preds=rng.randint(0, 3),
                    group=rng.choice([0, 7, 7, 25]), min_max=rng.random() < 0.3)
    sf = rng.choice([1, 2, 4, 8])
    small = rng.random() < 0.4
    rows = "%d,%d,2555" % ((2_000 if small else 20_000) * (1 + int(math.log2(sf))), (500 if small else 2_000) * sf)
    onehot = rng.random() < 0.25
    return _tree(None, _log_int(rng, 3e3, 1e6 if onehot else 5e6), rows, rng.choice([16, 32, 64, 128]), _log_int(rng, 4, 600),
                 c_f=rng.choice([0, 0, 0, 4]), form=rng.choice(["masks", "masks", "tables"]), onehot=onehot, refresh=rng.random() < 0.4)


# ------------------------------------------------------------------------------------------------ shapes of a case


def _ints(text):
    return [int(x) for x in text.split(",")]


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _schema(sf):
    """Rows of the date, customer, supplier and part dimensions."""
    return [2_556, 30_000 * sf, 2_000 * sf, 200_000 * (1 + int(math.log2(sf)))]


def _cards(case):
    return [case["g_date"], case["g_cust"], case["g_supp"], case["g_part"]]


def _tree_cols(case):
    K = len(_ints(case["rows"]))
    k = case["columns"] - case["c_f"]
    return [k // K + (j < k % K) for j in range(K)]


# ------------------------------------------------------------------------------------------------ inputs


class _Source:
    def __init__(self, seed):
        self.gen = torch.Generator(device=DEV)
        self.gen.manual_seed(seed)

    def normal(self, shape, dtype, sigma=1.0):
        return (torch.randn(shape, generator=self.gen, device=DEV) * sigma).to(dtype)

    def ints(self, shape, lo, hi, dtype=torch.int32):
        return torch.randint(lo, hi, shape, generator=self.gen, device=DEV, dtype=dtype)

    def zipf(self, n, r, s=1.1):
        """Bounded Zipf(s) ranks, scattered over the rows by a random permutation."""
        cdf = torch.arange(1, r + 1, dtype=torch.float64, device=DEV).pow(-s).cumsum(0)
        cdf /= cdf[-1].clone()
        perm = torch.randperm(r, generator=self.gen, device=DEV).to(torch.int32)
        out = torch.empty(n, dtype=torch.int32, device=DEV)
        for lo in range(0, n, 1 << 24):
            u = torch.rand(min(n - lo, 1 << 24), generator=self.gen, device=DEV, dtype=torch.float64)
            out[lo:lo + u.numel()] = perm[torch.searchsorted(cdf, u).clamp_(max=r - 1)]
        return out

    def fks(self, n, rows, how="uniform"):
        return [self.zipf(n, r) if how == "zipf" else self.ints((n,), 0, r) for r in rows]


def _prepare_predict(case, src):
    n, rows, cols, layers, dt = case["n"], _ints(case["rows"]), _ints(case["cols"]), _ints(case["layers"]), _dtype(case)
    widths = [case["c_f"] + sum(cols)] + layers
    s = {"X": src.normal((n, case["c_f"]), dt) if case["c_f"] else None,
         "dims": [src.normal((r, c), dt) for r, c in zip(rows, cols)],
         "fks": src.fks(n, rows, case["fk"]),
         "W": [src.normal((a, b), dt, a ** -0.5) for a, b in zip(widths, widths[1:])]}
    s["b"] = [src.normal((b,), dt, 0.5) for b in layers] if case["bias"] else None
    s["P"] = None if case["refresh"] or not case["fused"] else lq.lq_project_dims(s["dims"], s["W"][0], case["c_f"])
    return s


def _prepare_group(case, src):
    n, rows, cards = case["n"], _schema(case["sf"]), _cards(case)
    shares = [case["s_date"], case["s_cust"], case["s_supp"], case["s_part"]]
    s = {"rows": rows, "masks": [], "codes": [], "cards": [max(1, c) for c in cards], "maps": None,
         "measures": [src.ints((n,), 1, 100_001) for _ in range(case["measures"])],
         "fact_mask": (src.ints((n,), 0, 10) > 0).to(torch.uint8) if case["fact_mask"] else None}
    for r, card, share in zip(rows, cards, shares):
        # a coarse attribute of 7 or 25 values, which predicates select by, and a finer one inside each of its values
        base = 7 if card == 7 else 25
        coarse = src.ints((r,), 0, base)
        s["masks"].append(None if share == 1.0 else (coarse < max(1, round(base * share))).to(torch.uint8))
        s["codes"].append(None if not card else coarse * (card // base) + src.ints((r,), 0, card // base))
    fks = src.fks(n, rows)
    if case["keys"] == "rows":
        s["fks"] = fks
        return s
    wide = case["keys"] == "sparse64"
    s["build"], s["lookup"] = (lq.lq_keymap64_build, lq.lq_keymap64_lookup) if wide else (lq.lq_keymap_build, lq.lq_keymap_lookup)
    s["dim_keys"] = []
    for r in rows:
        k = torch.randperm(r if case["keys"] == "dense" else 8 * r, generator=src.gen, device=DEV)[:r] + 1
        s["dim_keys"].append((k * 1_000_003 if wide else k.to(torch.int32)).contiguous())
    s["fact_keys"] = [k[f.long()] for k, f in zip(s["dim_keys"], fks)]
    if not case["refresh"]:
        s["maps"] = [s["build"](k) for k in s["dim_keys"]]
    return s


def _prepare_agg(case, src):
    n, rows = case["n"], [2_556, 30_000, 2_000, 200_000][:case["joins"]]
    year = src.ints((rows[0],), 0, 7)
    s = {"fks": src.fks(n, rows), "rows": rows, "cards": [1] * len(rows), "codes": [None] * len(rows),
         "masks": [(year == 1).to(torch.uint8) if case["group"] != 7 else None]}
    s["masks"] += [(src.ints((r,), 0, 5) == 2).to(torch.uint8) for r in rows[1:]]
    if case["group"] == 7:
        s["codes"][0], s["cards"][0] = year, 7
    elif case["group"] == 25:
        s["codes"][-1], s["cards"][-1] = src.ints((rows[-1],), 0, 25), 25
    price, discount, quantity, cost = (src.ints((n,), lo, hi) for lo, hi in ((90_000, 10_000_000), (0, 11), (1, 51), (50_000, 100_000)))
    s["preds"] = [(discount, 1, 3), (quantity, 1, 24), (cost, 60_000, 90_000)][:case["preds"]]
    s["measures"] = [(case["op"], price, {"col": None, "mul": discount, "sub": cost}[case["op"]])]
    s["want"] = ("sum", "min", "max", "count") if case["min_max"] else ("sum", "count")
    return s


def _path_matrix(leaves, columns, seed):
    """Random binary tree in matrix form: tested column and threshold of every node, and H [nodes x leaves] (+1 / -1 where a
    node lies on the path to a leaf on its true / false side)."""
    rng = np.random.default_rng(seed)
    paths = [[]]
    for q in range(leaves - 1):
        at = int(rng.integers(0, len(paths)))
        path = paths[at]
        paths[at:at + 1] = [path + [(q, -1)], path + [(q, 1)]]
    H = np.zeros((leaves - 1, leaves), dtype=np.int8)
    for j, path in enumerate(paths):
        for q, sign in path:
            H[q, j] = sign
    feature = rng.integers(0, columns, leaves - 1).astype(np.int32)
    threshold = (rng.standard_normal(leaves - 1) * 0.7).astype(np.float32)
    return [torch.from_numpy(x).to(DEV) for x in (feature, threshold, H)]


def _tree_tables(case, s):
    tables, target = lq.lq_tree_project_dims(s["dims"], case["c_f"], *s["tree"])
    if case["form"] == "tables":
        return {"tables": tables, "target": target}
    return {"masks": lq.lq_tree_compress_tables(s["dims"], tables, *s["tree"], c_f=case["c_f"]),
            "fact_masks": lq.lq_tree_fact_masks(case["c_f"], *s["tree"]) if case["c_f"] else None}


def _prepare_tree(case, src, seed):
    rows = _ints(case["rows"])
    s = {"dims": [src.normal((r, c), torch.float32) for r, c in zip(rows, _tree_cols(case))],
         "fks": src.fks(case["n"], rows), "tree": _path_matrix(case["leaves"], case["columns"], seed),
         "X": src.normal((case["n"], case["c_f"]), torch.float32) if case["c_f"] else None}
    s["kept"] = None if case["refresh"] else _tree_tables(case, s)
    return s


def prepare(case, seed):
    src = _Source(seed)
    if case["kind"] == "tree":
        s = _prepare_tree(case, src, seed)
    else:
        s = {"predict": _prepare_predict, "group": _prepare_group, "agg": _prepare_agg}[case["kind"]](case, src)
    s["case"] = case
    return s


# ------------------------------------------------------------------------------------------------ one pass


def _run_predict(case, s):
    if not case["fused"]:
        return lq.lq_materialized_join_predict(s["X"], s["dims"], s["fks"], s["W"], s["b"])
    P = s["P"] if s["P"] is not None else lq.lq_project_dims(s["dims"], s["W"][0], case["c_f"])
    Y = lq.lq_fused_join_predict(s["X"], s["fks"], P, s["W"], s["b"])
    return (Y, P) if case["refresh"] else Y


def _run_group(case, s):
    if case["keys"] == "rows":
        return lq.lq_masked_groupby_sum(s["fks"], s["rows"], s["masks"], s["codes"], s["cards"], s["fact_mask"], s["measures"])
    maps = s["maps"] or [s["build"](k) for k in s["dim_keys"]]
    fks = [s["lookup"](m, k) for m, k in zip(maps, s["fact_keys"])]
    sums, counts = lq.lq_masked_groupby_sum(fks, s["rows"], s["masks"], s["codes"], s["cards"], s["fact_mask"], s["measures"])
    if counts.shape[0] > 8192:     # the largest result that the library orders itself
        return fks, sums, counts
    cards = [c for c, code in zip(s["cards"], s["codes"]) if code is not None]
    keys = [(lq.LQ_KEY_GROUP_COLUMN, 0, 0)] if cards else []
    return fks, sums, counts, lq.lq_order_groups(cards, sums, counts, keys + [(lq.LQ_KEY_SUM, 0, 1)])


def _run_agg(case, s):
    return lq.lq_groupby_agg(s["fks"], s["rows"], s["masks"], s["codes"], s["cards"], s["preds"], s["measures"], want=s["want"])


def _run_tree(case, s):
    kept = s["kept"] or _tree_tables(case, s)
    if case["form"] == "tables":
        out = lq.lq_fused_join_tree(s["X"], s["fks"], kept["tables"], kept["target"], *s["tree"], want_onehot=case["onehot"])
    else:
        out = lq.lq_fused_join_tree_masks(s["fks"], kept["masks"], *s["tree"], want_onehot=case["onehot"], X=s["X"],
                                          fact_masks=kept["fact_masks"])
    return (out, kept[case["form"]]) if case["refresh"] else out


def run(state):
    case = state["case"]
    return {"predict": _run_predict, "group": _run_group, "agg": _run_agg, "tree": _run_tree}[case["kind"]](case, state)


# ------------------------------------------------------------------------------------------------ floors and tolerances


def _work_predict(case):
    n, rows, cols, layers = case["n"], _ints(case["rows"]), _ints(case["cols"]), _ints(case["layers"])
    es = 2 if case["dtype"] == "bf16" else 4
    K, l1, k = len(rows), layers[0], case["c_f"] + sum(cols)
    later = 2 * n * sum(a * b for a, b in zip(layers, layers[1:]))
    stream = n * (case["c_f"] * es + 4 * K + layers[-1] * es)
    model = es * sum(a * b for a, b in zip([k] + layers, layers))
    if not case["fused"]:
        return {"bytes": stream + model + es * sum(min(n, r) * c for r, c in zip(rows, cols)), "flops": 2 * n * k * l1 + later}
    refresh = case["refresh"]
    tables = es * sum(r * (l1 + c) if refresh else min(n, r) * l1 for r, c in zip(rows, cols))
    return {"bytes": stream + model + tables,
            "flops": (2 * l1 * sum(r * c for r, c in zip(rows, cols)) if refresh else 0) + n * l1 * (2 * case["c_f"] + K) + later}


def _work_group(case):
    n, rows, cards = case["n"], _schema(case["sf"]), _cards(case)
    shares = [case["s_date"], case["s_cust"], case["s_supp"], case["s_part"]]
    survive, G, side = (0.9 if case["fact_mask"] else 1.0), 1, 0
    for r, card, share in zip(rows, cards, shares):
        survive *= share
        G *= max(1, card)
        side += r * ((4 if card else 0) + (1 if share < 1 else 0))
    # a measure column comes in lines of 32 values: those without a survivor need not be read
    measure = 4 * n * case["measures"] * (1 - (1 - survive) ** 32)
    total = n * (4 * len(rows) + (1 if case["fact_mask"] else 0)) + measure + side + 8 * G * (case["measures"] + 1)
    if case["keys"] != "rows":      # the key columns are read, the mapped ones written (and then read, as above)
        key = 8 if case["keys"] == "sparse64" else 4
        total += n * (key + 4) * len(rows) + sum(rows) * (key + 4) * (2 if case["refresh"] else 1)
    return {"bytes": total, "flops": 0}


def _work_agg(case):
    n, rows = case["n"], [2_556, 30_000, 2_000, 200_000][:case["joins"]]
    survive = (1.0 if case["group"] == 7 else 1 / 7) * 0.2 ** (len(rows) - 1)
    for share in (3 / 11, 24 / 50, 0.6)[:case["preds"]]:
        survive *= share
    columns = (2 if case["op"] != "col" else 1) - (1 if case["op"] == "mul" and case["preds"] else 0)
    measure = 4 * n * columns * (1 - (1 - survive) ** 32)
    return {"bytes": n * 4 * (len(rows) + case["preds"]) + measure + 5 * sum(rows), "flops": 0}


def _work_tree(case):
    n, rows, cols, leaves = case["n"], _ints(case["rows"]), _tree_cols(case), case["leaves"]
    per_leaf = 1 if case["form"] == "tables" else 1 / 8
    total = n * (4 * len(rows) + 4 * case["c_f"] + 4 + (leaves if case["onehot"] else 0)) + (leaves - 1) * (leaves + 8)
    if case["refresh"]:
        total += sum(r * (4 * c + leaves * per_leaf) for r, c in zip(rows, cols))
    else:
        total += sum(min(n, r) * leaves * per_leaf for r in rows)
    return {"bytes": total, "flops": 0}


def work(case):
    return {"predict": _work_predict, "group": _work_group, "agg": _work_agg, "tree": _work_tree}[case["kind"]](case)


def tolerance(case):
    if case["kind"] != "predict":
        return "exact"              # whole numbers
    return {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 1e-5}
