"""The work a user of the epsilon join has it do, as measurable cases through the public entry points.

Every case is a dict of plain values; `kind` says which call it makes:

  count    EJoin.selfjoin_count: neighbours per point (density, outliers, the size of a result before it is fetched)
  graph    EJoin.selfjoin_pairs of a small set, its result written into a weighted adjacency matrix
  pairs    EJoin.selfjoin_pairs, its result put into the order of (j, i): the neighbour list of a data set
  pairs2   EJoin.join_pairs of two sets, ordered the same way
  queries  EJoinSet.join_count: a batch of query points against a point set prepared once (the serving call)
  split    EJoin.selfjoin_count_f32: the higher-accuracy join of FP32 rows
  ingest   EJoin.convert_f32 and EJoin.norms: FP32 rows made ready for the joins
  dense    EJoin.dist2_tile: a block of the distance matrix itself

Sizes follow the five workloads of datagen.py (n = 4,096 ... 5,000,000, d = 128 ... 960, mean selectivity 16 ... 1,024, about
1,000 points a cluster), kept to what runs in well under a second, and go down to sets that a few workgroups cover; d takes
the widths of common descriptors and embeddings too (96, 200, 300, 784), which are no multiples of 64.

A pair list comes in no particular order, so a pass that returns one ends with the sort (or the scatter) that a program needs
before it can look a point up.
"""
import math
import statistics

import torch

import paper_2508_21230_amd as ejoin

POINTS_PER_CLUSTER = 1000
_ctx = None


def _join():
    """The one context of the process, as a program keeps it."""
    global _ctx
    if _ctx is None:
        _ctx = ejoin.EJoin(0)
    return _ctx


# ------------------------------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest calls: one batch of points looked at for its density; launches and latency are what counts
        dict(name="count_1k_d96", kind="count", data="uniform", n=1000, d=96, S=16),
        # the first workload: 4,096 points, d = 128, some 30 neighbours each, as a neighbour graph
        dict(name="graph_4k_d128", kind="graph", data="uniform", n=4096, d=128, S=40),
        # a mid-sized set of wide descriptors (d = 960), n no multiple of anything
        dict(name="pairs_20k_d960", kind="pairs", data="mixture", n=20011, d=960, S=16),
        # the second workload: 100,000 points, d = 128, 64 neighbours each: dense output for its size
        dict(name="pairs_100k_d128", kind="pairs", data="mixture", n=100000, d=128, S=64),
        # the fourth workload's width with many neighbours, counted before they are fetched
        dict(name="count_300k_d384", kind="count", data="mixture", n=300000, d=384, S=256),
        # the fifth workload scaled down: a million points, d = 128, counts only
        dict(name="count_1m_d128", kind="count", data="mixture", n=1000000, d=128, S=64),
        # the third workload scaled down: the widest vectors, the largest call
        dict(name="pairs_600k_d960", kind="pairs", data="mixture", n=600000, d=960, S=16),
        # serving: 500 query points against 200,000 prepared ones
        dict(name="queries_500_of_200k_d384", kind="queries", data="mixture", n=200000, nq=500, d=384, S=32),
        # two sets matched against each other once, ragged in every size
        dict(name="pairs2_30k_7k_d200", kind="pairs2", data="mixture", n=30011, nq=7001, d=200, S=16),
        # near-duplicates among FP32 embeddings of 300 coordinates: more than FP16's accuracy, a tight threshold
        dict(name="split_50k_d300", kind="split", data="mixture", n=50000, d=300, S=1),
        # ingestion: FP32 rows of 200 coordinates centred, scaled and rounded, and their norms
        dict(name="ingest_500k_d200", kind="ingest", data="mixture", n=500000, d=200, S=0),
        # a block of the distance matrix of 20,000 points, off the diagonal and ragged
        dict(name="dense_4000x5000_d384", kind="dense", data="mixture", n=20000, d=384, S=0, rows=4000, cols=5000),
    ]


WIDTHS = (16, 32, 64, 96, 100, 128, 192, 200, 256, 300, 384, 512, 768, 784, 960)


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(("count", "count", "graph", "pairs", "pairs", "pairs2", "queries", "split", "ingest", "dense"))
    d = rng.choice(WIDTHS) if rng.random() < 0.6 else log_int(16, 960)
    S = log_int(4, 64)
    if kind == "count":
        n = log_int(300, min(1000000, int(math.sqrt(3e14 / d))))
        return dict(kind=kind, data="uniform" if n < 8000 else "mixture", n=n, d=d, S=min(log_int(4, 512), n // 8))
    if kind == "graph":
        return dict(kind=kind, data="uniform", n=log_int(500, 5000), d=min(d, 512), S=S)
    if kind == "pairs":
        return dict(kind=kind, data="mixture", n=log_int(8000, min(600000, int(math.sqrt(3e14 / d)))), d=d, S=S)
    if kind == "pairs2":
        return dict(kind=kind, data="mixture", n=log_int(2000, 100000), nq=log_int(500, 20000), d=d, S=S)
    if kind == "queries":
        return dict(kind=kind, data="mixture", n=log_int(20000, 400000), nq=log_int(8, 4000), d=d, S=S)
    if kind == "split":
        return dict(kind=kind, data="mixture", n=log_int(2000, 60000), d=min(d, 400), S=rng.randint(1, 2))
    if kind == "ingest":
        return dict(kind=kind, data="mixture", n=log_int(10000, min(1000000, 200000000 // d)), d=d, S=0)
    return dict(kind=kind, data="mixture", n=log_int(8000, 40000), d=d, S=0, rows=log_int(200, 6000), cols=log_int(200, 6000))


# ------------------------------------------------------------------------------------------ inputs
def _sigma(d):
    """Spread of a cluster: 0.05 at d = 128, 0.03 at 384, 0.02 at 960, as in the workloads."""
    return 0.05 * math.sqrt(128.0 / d)


def _rows(case, n, gen, centres):
    """n FP32 rows: uniform in [0, 1), or around the centres and clipped to [0, 1]."""
    d = case["d"]
    if centres is None:
        return torch.rand((n, d), generator=gen, device="cuda")
    x = torch.randn((n, d), generator=gen, device="cuda")
    x.mul_(_sigma(d))
    ids = torch.randint(centres.shape[0], (n,), generator=gen, device="cuda")
    for r in range(0, n, 65536):
        x[r:r + 65536] += centres[ids[r:r + 65536]]
    return x.clamp_(0.0, 1.0)


def _fp16(x):
    """FP16 rows with a row stride that is a multiple of 64, padded with zeros: what the joins take."""
    n, d = x.shape
    out = torch.zeros((n, (d + 63) // 64 * 64), dtype=torch.float16, device="cuda")
    out[:, :d] = x
    return out


def _eps(case):
    """The distance that gives about S neighbours a point."""
    n, d, S = case["n"], case["d"], case["S"]
    if case["data"] == "uniform":  # squared distance of two points: mean d/6, variance 7d/180
        z = statistics.NormalDist().inv_cdf(S / n)
        return math.sqrt(max(d / 6.0 + z * math.sqrt(7.0 * d / 180.0), d / 60.0))
    # Within a cluster the squared distance is 2 var chi^2_d (quantile: Wilson-Hilferty); clipping a coordinate whose centre is
    # uniform in [0, 1] takes 2 * 0.59 sigma off the variance sigma^2.
    z = statistics.NormalDist().inv_cdf(S * _clusters(n) / n)
    var = _sigma(d) ** 2 * (1.0 - 1.18 * _sigma(d))
    return math.sqrt(2.0 * var * d * (1.0 - 2.0 / (9.0 * d) + z * math.sqrt(2.0 / (9.0 * d))) ** 3)


def _clusters(n):
    return max(1, round(n / POINTS_PER_CLUSTER))


def _capacity(case):
    """Room for the result: half as much again as is expected (few coordinates: twice, neighbouring clusters overlap there)."""
    room = 1.5 if case["d"] >= 64 else 2.0
    if case["kind"] == "pairs2":
        return 8192 + int(room * case["nq"] * case["S"])
    return 8192 + case["n"] + int(room * case["n"] * case["S"] / 2)


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    centres = None
    if case["data"] == "mixture":
        centres = torch.rand((_clusters(case["n"]), case["d"]), generator=gen, device="cuda")
    X = _rows(case, case["n"], gen, centres)
    Q = _rows(case, case["nq"], gen, centres) if "nq" in case else None
    return X, Q


def prepare(case, seed):
    ej, kind = _join(), case["kind"]
    X, Q = _inputs(case, seed)
    state = dict(kind=kind, n=case["n"], d=case["d"])
    if kind in ("split", "ingest"):
        state["X32"] = X
        if kind == "ingest":
            state["center"] = X.mean(dim=0)
        else:
            ej.reserve(2 * case["n"], 3 * state["d"])
    else:
        state["X"] = _fp16(X)
        if Q is not None:
            state["Q"] = _fp16(Q)
        ej.reserve(case["n"] + case.get("nq", 0), case["d"])
    if case["S"]:
        state["eps"] = _eps(case)
    if kind == "queries":
        state["set"] = ej.prepare(state["X"], d=case["d"])
    if kind in ("graph", "pairs", "pairs2"):
        cap = _capacity(case)
        state["capacity"] = cap
        # entries past the end of the result: no pair (the graph: the first point's loop once more)
        state["pairs"] = torch.full((cap, 2), 0 if kind == "graph" else -1, dtype=torch.int32, device="cuda")
        state["dist2"] = torch.zeros(cap, dtype=torch.float32, device="cuda")
        state["n_pairs"] = torch.zeros(1, dtype=torch.int64, device="cuda")
    if kind == "graph":
        state["adjacency"] = torch.full((case["n"], case["n"]), -1.0, dtype=torch.float32, device="cuda")
    if kind == "dense":
        state["block"] = (case["n"] // 7, case["n"] - case["cols"], case["rows"], case["cols"])
    torch.cuda.synchronize()
    return state


# ------------------------------------------------------------------------------------------ a pass
def _ordered(pairs, dist2, n_pairs):
    """The pair list in the order of (j, i), entries past its end first."""
    keys, order = torch.sort(pairs.view(torch.int64).view(-1))
    return {"pairs": keys, "dist2": dist2[order], "n_pairs": n_pairs}


def run(state):
    ej, kind, d = _join(), state["kind"], state["d"]
    if kind == "count":
        counts, total = ej.selfjoin_count(state["X"], state["eps"], d=d)
        return {"counts": counts, "total": total}
    if kind in ("graph", "pairs"):
        pairs, dist2, n_pairs = ej.selfjoin_pairs(state["X"], state["eps"], state["capacity"], d=d, pairs=state["pairs"],
                                                  dist2=state["dist2"], n_pairs=state["n_pairs"])
        if kind == "pairs":
            return _ordered(pairs, dist2, n_pairs)
        state["adjacency"].index_put_((pairs[:, 0], pairs[:, 1]), dist2)
        return {"adjacency": state["adjacency"], "n_pairs": n_pairs}
    if kind == "pairs2":
        return _ordered(*ej.join_pairs(state["X"], state["Q"], state["eps"], state["capacity"], d=d, pairs=state["pairs"],
                                       dist2=state["dist2"], n_pairs=state["n_pairs"]))
    if kind == "queries":
        counts_p, counts_q, total = state["set"].join_count(state["Q"], state["eps"])
        return {"counts_p": counts_p, "counts_q": counts_q, "total": total}
    if kind == "split":
        counts, _ = ej.selfjoin_count_f32(state["X32"], state["eps"])  # (the total is half the counts' sum)
        return {"counts": counts}
    if kind == "ingest":
        X16 = ej.convert_f32(state["X32"], scale=2.0, center=state["center"])
        return {"X16": X16, "norms": ej.norms(X16, d=d)}
    return {"dist2": ej.dist2_tile(state["X"], *state["block"], d=d)}


# ------------------------------------------------------------------------------------------ what a pass cannot do without
def work(case):
    n, d, S, kind = case["n"], case["d"], case["S"], case["kind"]
    nq = case.get("nq", 0)
    if kind in ("count", "split"):
        return {"bytes": (4 if kind == "split" else 2) * n * d + 4 * n, "flops": n * (n + 1.0) * d}
    if kind in ("graph", "pairs"):
        return {"bytes": 2 * n * d + 12 * n * (1 + S / 2), "flops": n * (n + 1.0) * d}
    if kind == "pairs2":
        return {"bytes": 2 * (n + nq) * d + 12 * nq * S, "flops": 2.0 * n * nq * d}
    if kind == "queries":
        return {"bytes": 2 * (n + nq) * d + 4 * (n + nq), "flops": 2.0 * n * nq * d}
    if kind == "ingest":
        return {"bytes": n * (4 * d + 2 * ((d + 63) // 64 * 64) + 4), "flops": 4.0 * n * d}
    return {"bytes": 2 * (case["rows"] + case["cols"]) * d + 4 * case["rows"] * case["cols"], "flops": 2.0 * case["rows"] * case["cols"] * d}


def tolerance(case):
    """The interface defines the arithmetic of the FP16 join to the bit (the order of k, the step that adds the norms), and a
    result set or a count follows from it: those are exact."""
    if case["kind"] == "split":
        # the interface does not fix the order of the sums over the two halves' products, so pairs next to the threshold may
        # fall on either side (against 64 bits 0.4 % of the points are counted differently at one neighbour each)
        return {"rel": 0.0, "differ": 0.01}
    if case["kind"] in ("ingest", "dense"):
        return {"rel": 2e-6, "max": 1.2e-5}  # FP32 sums: four times 4.4e-7 and 2.7e-6, the block's error against 64 bits
    return "exact"


def exact(case, seed):
    """Distances, norms and converted rows in 64 bits.  The values of a pair list have none: one pair next to the threshold
    that falls on the other side moves every entry after it; counts are whole numbers."""
    if case["kind"] not in ("graph", "ingest", "dense"):
        return None
    X, _ = _inputs(case, seed)
    if case["kind"] == "ingest":
        center = X.mean(dim=0)
        y = (X - center) * 2.0  # (the rounded rows are what the norms are taken of)
        X16 = torch.zeros((case["n"], (case["d"] + 63) // 64 * 64), dtype=torch.float64, device="cuda")
        norms = torch.empty(case["n"], dtype=torch.float64, device="cuda")
        for r in range(0, case["n"], 65536):
            h = y[r:r + 65536].half().double()
            norms[r:r + 65536] = (h * h).sum(dim=1)
            X16[r:r + 65536, :case["d"]] = (X[r:r + 65536].double() - center.double()) * 2.0
        return {"X16": X16, "norms": norms}
    X = X.half().double()

    def dist2(a, b):
        return ((a * a).sum(dim=1)[:, None] + (b * b).sum(dim=1)[None, :] - 2.0 * (a @ b.T)).clamp_(min=0.0)

    if case["kind"] == "dense":
        i0, j0 = case["n"] // 7, case["n"] - case["cols"]
        return {"dist2": dist2(X[i0:i0 + case["rows"]], X[j0:j0 + case["cols"]])}
    D = dist2(X, X)
    D.fill_diagonal_(0.0)
    D[~(torch.ones_like(D, dtype=torch.bool).triu() & (D <= _eps(case) ** 2))] = -1.0
    return {"adjacency": D, "n_pairs": None}
