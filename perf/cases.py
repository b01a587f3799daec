"""Performance cases: the work a user of the landscape engine has it do.

A search space is the product of parameter value lists with one measured
runtime per configuration; configurations that violate a constraint hold +inf
and failed ones NaN.  The spaces here are random stand-ins with the structure
of brute-forced kernel-tuning tables: log-normal runtimes with a few dominant
parameters and pairwise interactions, index-sum constraints on the leading
parameters, and a share of failed runs.

``listed()`` names the cases, ``draw()`` gives more of the same ranges,
``prepare()`` builds what a program holds before the call, ``run()`` makes one
pass through the public entry points, ``work()`` states what a pass cannot do
without, and ``exact()`` gives the same outputs in 64 bits from plain torch.
"""
import math
import random

import torch

from paper_2210_01465_amd import api

TOL = 2e-7        # the engine's default stopping tolerance
BINS = 20         # bins of the naive metric's histogram
CURVE = tuple(j / 100 for j in range(16))   # p = 0, 1, ..., 15 %


def _case(name, call, radix, nb="hamming", damping=0.85, sum01=-1, sum23=-1, fail=0.05, sigma=0.2, pairs=3):
    return {"name": name, "call": call, "radix": "x".join(str(r) for r in radix), "nb": nb, "damping": damping,
            "sum01": sum01, "sum23": sum23, "fail": fail, "sigma": sigma, "pairs": pairs}


LARGE = (12, 10, 6, 5, 4, 4, 3, 3, 3, 3)
MID = (9, 8, 6, 5, 4, 4, 3, 2)


def listed():
    return [
        # a first look at a handful of parameters: 160 configurations, all latency
        _case("tiny", "analyze", (5, 4, 4, 2), sum01=6),
        # point-in-polygon kernel: the paper's smallest full space, few failures
        _case("pnpoly", "analyze", (31, 11, 4, 2, 3), fail=0.04),
        # 2-D convolution kernel under the adjacent-value neighbourhood, two thirds failed
        _case("convolution_adjacent", "analyze", (12, 6, 8, 8, 2, 2), nb="adjacent", fail=0.34),
        # matrix-product kernel, 78 % failed, from a serving loop that may not allocate
        _case("gemm_noalloc", "noalloc", (4, 4, 3, 3, 3, 3, 4, 4, 2, 2), fail=0.78),
        # a medium space, one-shot (1.2e5 valid configurations)
        _case("mid", "analyze", MID, sum01=10, sum23=6),
        # the benchmark's space: 1.5 M valid configurations, 23 M edges, rugged
        _case("large", "analyze", LARGE, sum01=10, sum23=5, fail=0.10, sigma=0.5, pairs=5),
        # the same space under the adjacent-value neighbourhood
        _case("large_adjacent", "analyze", LARGE, nb="adjacent", sum01=10, sum23=5, fail=0.10, sigma=0.5, pairs=5),
        # random-descent probabilities (exact sweeps, damping 1) on a plan that is kept
        _case("large_exact", "exact", LARGE, damping=1.0, sum01=10, sum23=5, fail=0.10, sigma=0.5, pairs=5),
        # the fitness flow graph itself, for a program that runs its own graph analysis
        _case("large_graph", "graph", LARGE, sum01=10, sum23=5, fail=0.10, sigma=0.5, pairs=5),
        # long value lists: more candidate neighbours than a node record holds
        _case("long_lists", "analyze", (64, 56, 40, 3), sum01=90, fail=0.10),
        # a study of many kernels on several devices: 26 shapes, 3 devices each, in one call
        {"name": "study78", "call": "batch", "shapes": 26, "devices": 3, "shape_seed": 4, "smallest": 500,
         "largest": 200_000, "nb": "hamming", "damping": 0.85},
        # the paper's figures from ranks at hand: C_p for 16 proportions and the naive metric
        _case("large_figures", "figures", LARGE, sum01=10, sum23=5, fail=0.10, sigma=0.5, pairs=5),
    ]


def draw(rng):
    """A case of the listed ranges that costs no more than the largest listed ones."""
    limit = {c["call"]: work(c)["flops"] for c in listed() if c["name"] in ("large", "study78")}
    while True:
        c = _draw(rng)
        if work(c)["flops"] <= limit.get(c["call"], limit["analyze"]):
            return c


def _draw(rng):
    kind = rng.choice(("analyze", "analyze", "analyze", "execute", "noalloc", "exact", "graph", "figures", "lists",
                       "batch"))
    nb = rng.choice(("hamming", "hamming", "adjacent"))
    if kind == "batch":
        return {"call": "batch", "shapes": rng.randint(3, 20), "devices": rng.randint(1, 3),
                "shape_seed": rng.randrange(1 << 30), "smallest": 200, "largest": rng.randint(5_000, 150_000),
                "nb": nb, "damping": rng.choice((0.8, 0.85, 0.9))}
    if kind == "lists":
        radix = (rng.randint(50, 72), rng.randint(30, 64), rng.randint(20, 44), rng.randint(1, 4))
        c = _case("", "analyze", radix, nb, rng.choice((0.8, 0.85)), fail=round(rng.uniform(0.02, 0.5), 3))
    else:
        top = 250_000 if kind == "noalloc" else 4_000_000
        radix = _radices(rng, math.exp(rng.uniform(math.log(120), math.log(top))))
        small = math.prod(radix) < 500_000
        d = 1.0 if kind == "exact" and rng.random() < 0.5 else rng.choice((0.8, 0.85, 0.9, 0.95) if small else (0.8, 0.85))
        reach = radix[0] + radix[1] - 2
        c = _case("", kind, radix, nb, d, sum01=rng.choice((-1, reach - rng.randint(1, max(1, reach // 2)))),
                  fail=round(rng.uniform(0.01, 0.7), 3), sigma=rng.choice((0.2, 0.5)), pairs=rng.randint(1, 5))
    del c["name"]
    return c


def _radices(rng, target):
    """Between 3 and 10 value lists of 2 to 12 values, product near target, long lists first as often as not."""
    while True:
        radix = [rng.randint(2, 12) for _ in range(rng.randint(3, 10))]
        if target / 1.4 <= math.prod(radix) <= 1.4 * target:
            return tuple(sorted(radix, reverse=True)) if rng.random() < 0.5 else tuple(radix)


def _spaces(case):
    """The spaces of a case, each a dict of plain values as _case() gives."""
    if case["call"] != "batch":
        return [case]
    rng = random.Random(case["shape_seed"])
    # the four kernel spaces of the paper (radices, failed share), then random shapes
    shapes = [((12, 6, 8, 8, 2, 2), 0.69), ((8, 6, 3, 3, 2), 0.52), ((4, 4, 3, 3, 3, 3, 4, 4, 2, 2), 0.78),
              ((31, 11, 4, 2, 3), 0.04)]
    while len(shapes) < case["shapes"]:
        target = math.exp(rng.uniform(math.log(case["smallest"]), math.log(case["largest"])))
        raw = target * rng.uniform(1.2, 3.0)
        radix = _radices(rng, raw)
        shapes.append((radix, round(max(0.02, 1.0 - target / math.prod(radix)), 3)))
    return [_case("", "analyze", radix, case["nb"], case["damping"], fail=min(fail, 0.9))
            for radix, fail in shapes[:case["shapes"]] for _ in range(case["devices"])]


def _radix(space):
    return tuple(int(r) for r in space["radix"].split("x"))


def _excluded(space):
    """Configurations a constraint excludes (+inf) or whose run failed (NaN),
    as two masks: the kernel's own, so the same for every landscape of it."""
    radix = _radix(space)
    n = len(radix)
    index = [torch.arange(r, device="cuda").view([-1 if j == k else 1 for j in range(n)]) for k, r in enumerate(radix)]
    kept = torch.ones(radix, dtype=torch.bool, device="cuda")
    for (a, b), limit in (((0, 1), space["sum01"]), ((2, 3), space["sum23"])):
        if limit >= 0:
            kept &= index[a] + index[b] <= limit
    kept = kept.reshape(-1)
    ids = torch.nonzero(kept).flatten()
    g = torch.Generator(device="cuda").manual_seed(n * 100_003 + ids.numel())
    count = min(round(space["fail"] * ids.numel()), ids.numel() - 1)
    failed = torch.zeros_like(kept)
    failed[ids[torch.randperm(ids.numel(), generator=g, device="cuda")[:count]]] = True
    return ~kept, failed


def _fitness(space, seed):
    """float32[prod(radix)] on the GPU in raw order, from the seed alone."""
    radix = _radix(space)
    n = len(radix)
    g = torch.Generator(device="cuda").manual_seed(int(seed))

    def normal(*shape):
        return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float64)
    logf = 0.05 * normal(*radix)
    for k, r in enumerate(radix):
        logf += 0.3 * normal(r).view([-1 if j == k else 1 for j in range(n)])
    pick = random.Random(n * 1009 + radix[0])
    every = [(a, b) for a in range(n) for b in range(a + 1, n)]
    for a, b in pick.sample(every, min(space["pairs"], len(every))):
        logf += space["sigma"] * normal(radix[a], radix[b]).view([radix[j] if j in (a, b) else 1 for j in range(n)])
    # a runtime is the mean of several runs: no two are equal (the least
    # increase of the ordered values' bits that makes them distinct)
    bits, order = logf.exp().float().reshape(-1).view(torch.int32).sort()
    rank = torch.arange(bits.numel(), dtype=torch.int32, device="cuda")
    bits = torch.cummax(bits - rank, 0).values + rank
    f = torch.empty_like(bits).scatter_(0, order, bits).view(torch.float32)
    excluded, failed = _excluded(space)
    return f.masked_fill_(excluded, math.inf).masked_fill_(failed, math.nan)


def _seeds(seed, count):
    return [int(seed) * 1000 + j for j in range(count)]


def prepare(case, seed):
    spaces = _spaces(case)
    fits = [_fitness(s, q) for s, q in zip(spaces, _seeds(seed, len(spaces)))]
    ctx = api.Context(0)
    state = {"case": case, "ctx": ctx, "radix": [_radix(s) for s in spaces], "fit": fits}
    call = case["call"]
    raw = fits[0].numel()
    if call in ("analyze", "noalloc"):
        # output buffers, as large as the space
        state["out"] = (torch.zeros(raw, dtype=torch.float64, device="cuda"),
                        torch.zeros(raw, dtype=torch.int32, device="cuda"),
                        torch.zeros(raw, dtype=torch.int32, device="cuda"))
    if call in ("execute", "exact", "figures"):
        plan = state["plan"] = api.plan_create(ctx, state["radix"][0], fits[0], case["nb"])
        state["minima"] = torch.zeros(plan.n_valid, dtype=torch.int32, device="cuda")
    if call == "figures":
        state["ranks"] = api.execute(plan, case["damping"])[0]
        state["ratio"] = torch.zeros(plan.n_valid, dtype=torch.float64, device="cuda")
    if call == "batch":
        nodes = [int(torch.isfinite(f).sum()) for f in fits]
        state["first"] = [sum(nodes[:j]) for j in range(len(nodes))]
        state["flags"] = torch.zeros(sum(nodes), dtype=torch.int32, device="cuda")
    return state


def run(state):
    case, ctx = state["case"], state["ctx"]
    call, nb, d = case["call"], case["nb"], case["damping"]
    radix, fit = state["radix"][0], state["fit"][0]
    if call in ("analyze", "noalloc"):
        r = api.analyze(radix, fit, nb, d, ctx=ctx, no_alloc=call == "noalloc", out=state["out"])
        return r.pagerank, state["out"][1], r.valid_raw, r.score   # the minima lead their buffer
    if call in ("execute", "exact"):
        ranks, _, info = api.execute(state["plan"], d, minima=state["minima"], exact=call == "exact")
        return ranks, state["minima"], info["score"]
    if call == "graph":
        plan = api.plan_create(ctx, radix, fit, nb)
        graph = api.plan_export(plan)
        plan.close()
        return graph
    if call == "figures":
        curve = api.score_curve(state["plan"], state["ranks"], CURVE)
        ratio, counts = api.naive_metric(state["plan"], BINS)
        state["ratio"][:ratio.numel()] = ratio
        return torch.tensor(curve, dtype=torch.float64), state["ratio"], torch.tensor(counts)
    results = api.analyze_batch(state["radix"], state["fit"], nb, d, ctx=ctx)
    # the study's ranks in one vector, a flag for every node that is a minimum, the scores
    minima = torch.cat(torch._foreach_add([r.minima for r in results], state["first"]))
    return (torch.cat([r.pagerank for r in results]), state["flags"].index_fill_(0, minima.long(), 1),
            torch.tensor([r.score for r in results], dtype=torch.float64))


def _valid(space):
    """Expected share of valid configurations."""
    radix = _radix(space)
    share = 1.0 - space["fail"]
    for (a, b), limit in (((0, 1), space["sum01"]), ((2, 3), space["sum23"])):
        if limit >= 0:
            kept = sum(1 for i in range(radix[a]) for j in range(radix[b]) if i + j <= limit)
            share *= kept / (radix[a] * radix[b])
    return share


def work(case):
    """Bytes: every input read once, every output written once.  Flops: one
    addition per edge and iteration, with the expected number of edges (half
    the pairs of valid neighbours) and the iterations after which damping has
    shrunk a change by the tolerance's square root (the rate seen on such
    landscapes)."""
    total_bytes = total_flops = 0
    for s in _spaces(case):
        radix = _radix(s)
        raw = math.prod(radix)
        n = raw * _valid(s)
        pairs = sum(r - 1 if s["nb"] == "hamming" else 2.0 * (r - 1) / r for r in radix)
        edges = 0.5 * n * pairs * _valid(s)
        d = min(s["damping"], 0.95)
        sweeps = 0.5 * math.log(TOL) / math.log(d)
        call = case["call"]
        if call == "graph":      # fitness in; node map, out-degrees, row starts and sources out
            total_bytes += 4 * raw + 12 * n + 4 * edges
            total_flops += 2 * edges
        elif call == "figures":  # about one node in fifty is a minimum: its id, fitness, rank; ratio out
            total_bytes += 24 * n / 50
            total_flops += len(CURVE) * n / 50
        elif call in ("execute", "exact"):   # the plan's edges in, ranks out
            total_bytes += 4 * edges + 16 * n
            total_flops += 2 * edges * sweeps
        else:                    # fitness in; ranks and node map out
            total_bytes += 4 * raw + 12 * n
            total_flops += 2 * edges * (1 + sweeps)
    return {"bytes": int(total_bytes), "flops": int(total_flops)}


def _graph(radix, fit, nb):
    """Node count, edge sources and targets (node ids), fitness of the nodes."""
    ok = torch.isfinite(fit)
    nodes = int(ok.sum())
    ids = (torch.cumsum(ok, 0) - 1).view(radix)
    f = torch.where(ok, fit, math.nan).view(radix)
    src, dst = [], []
    for k, r in enumerate(radix):
        for step in range(1, 2 if nb == "adjacent" else r):
            if step >= r:
                break
            fa, fb = f.narrow(k, 0, r - step), f.narrow(k, step, r - step)
            ia, ib = ids.narrow(k, 0, r - step), ids.narrow(k, step, r - step)
            for worse, a, b in ((fa > fb, ia, ib), (fb > fa, ib, ia)):
                src.append(a[worse])
                dst.append(b[worse])
    return nodes, torch.cat(src) if src else ids.new_empty(0), torch.cat(dst) if dst else ids.new_empty(0), fit[ok]


def _stationary(radix, fit, nb, d):
    """Ranks, sinks and node fitness: r = u / sum(u) with u = 1 + d P u, by
    sweeps until nothing changes (the graph has no cycle)."""
    nodes, src, dst, f = _graph(radix, fit, nb)
    deg = torch.bincount(src, minlength=nodes)
    weight = torch.where(deg > 0, d / deg.clamp(min=1).double(), 0.0)
    u = torch.ones(nodes, dtype=torch.float64, device=fit.device)
    for _ in range(nodes + 2):
        v = torch.ones_like(u).index_add_(0, dst, (weight * u)[src])
        change = float((v - u).abs().max())
        u = v
        if change <= 1e-13 * float(u.max()):
            break
    return u / u.sum(), torch.nonzero(deg == 0).flatten(), f


def _near(ranks, sinks, f, p):
    r, fs = ranks[sinks], f[sinks].double()
    best = float(f.min())
    return float(r[fs <= (1.0 + p) * best].sum() / r.sum())


def exact(case, seed):
    if case["call"] == "graph":
        return None   # whole numbers only
    spaces = _spaces(case)
    every, scores = [], []
    for s, q in zip(spaces, _seeds(seed, len(spaces))):
        ranks, sinks, f = _stationary(_radix(s), _fitness(s, q), s["nb"], s["damping"])
        if case["call"] == "figures":
            curve = torch.tensor([_near(ranks, sinks, f, p) for p in CURVE], dtype=torch.float64)
            ratio = torch.zeros_like(ranks)
            ratio[:sinks.numel()] = f.min().double() / f[sinks].double()
            return curve, ratio, None
        every.append(ranks)
        scores.append(_near(ranks, sinks, f, 0.05))
    if case["call"] == "batch":
        return torch.cat(every), None, torch.tensor(scores, dtype=torch.float64)
    if case["call"] in ("execute", "exact"):
        return every[0], None, scores[0]
    return every[0], None, None, scores[0]
