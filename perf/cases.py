"""The calls whose speed matters, one dict of plain values each.

A case is one pass through a public entry point of the package, the way a
scheduler service calls it: the problem handle and the workspace are kept, the
call itself runs with host synchronisation and all.  Workflows have the shapes
and ranges of the synthetic workloads (4-tool diamonds to 32-tool DAGs;
chains, fan-outs, layered and mixed DAGs; latencies, transfers, load-ins and
footprints of the paper's Table 1).  A case fixes the workflow (`dag`); the
seed re-measures it: every latency is scaled by 0.8 to 1.2, as the runtime
monitor's running averages do between rounds.

Makespans and mapping indices are whole numbers and have to be equal.
"""
import math
import random

import numpy as np

import paper_2607_22242_amd as S

CONTENTION_Q16 = [65536, 88474, 117965, 157286]  # 1.00, 1.35, 1.80, 2.40
NEVER = (1 << 62) - 1
INFEASIBLE = (1 << 63) - 1
EXACT_MAPPINGS = 600_000  # mappings that the plain evaluation below scores in some seconds


def listed():
    return [
        # One round of a 4-tool scenario with three modes and a VRAM budget (81
        # mappings): the size the paper's experiments search between two steps
        # of a workflow, where the call's own latency is all there is.
        _case("diamond4", call="search", shape="diamond", n=4, tight=True, dag=1),
        # A mid-sized workflow, three layers of four tools: 3^12 mappings, about
        # one wave of work for the card.
        _case("layered12", call="search", shape="layered", n=12, dag=12),
        # A memory-constrained workflow where queueing and offloading dominate:
        # 3^16 mappings, many of them running out of memory early.
        _case("memlayered16", call="search", shape="layered", n=16, tight=True, dag=16),
        # The largest three-mode search in ordinary use, 3^19 mappings of a DAG
        # over all the tools of Table 1.
        _case("mixed19", call="search", shape="mixed", n=19, dag=3),
        # The same kind of search under the other contention reading (GPU tools
        # share the card's rate): 3^18 mappings.
        _case("sharing18", call="search", shape="mixed", n=18, sharing=True, dag=18),
        # The GPU/CPU space of a wide workflow without a queue: 2^30 mappings
        # (two of the 32 tools are CPU-only), 64-bit indices.
        _case("binary32", call="search", shape="mixed", n=32, binary=True, dag=5),
        # One of eight shards of a 3^19 search, as it is split by index range.
        _case("shard19", call="range", shape="mixed", n=19, dag=3, lo=0.25, hi=0.375),
        # Re-scoring of 13 scenarios x 64 perturbed profiles, 14 tools each.
        _case("batch13x64", call="batch", n=14, scenarios=13, replicas=64, ragged=False, dag=400),
        # The same call as a monitor makes it every round: small scenarios of
        # different sizes (4 to 9 tools), a few profiles each.
        _case("rounds13x8", call="batch", n=9, scenarios=13, replicas=8, ragged=True, dag=420),
        # What-if probes around the current mapping with re-measured latencies:
        # the bounded exploration of every monitoring round.
        _case("reprobes19", call="reprobes", shape="mixed", n=19, dag=3),
        # The exact answer where the space is too large to enumerate: 3^24.
        _case("pruned24", call="pruned", shape="mixed", n=24, tight=True, dag=24),
        # Explicit mappings proposed by another scheduler, scored in one call
        # from host arrays (a ragged number, 64-bit indices).
        _case("score20", call="score", shape="mixed", n=20, tight=True, dag=20, count=200_003),
    ]


def draw(rng):
    """Another case of the same ranges."""
    call = rng.choice(["search"] * 5 + ["range", "batch", "batch", "reprobes", "pruned", "score"])
    c = {"shape": rng.choice(["diamond", "chain", "fanout", "layered", "mixed", "mixed"]),
         "tight": rng.random() < 0.5, "dag": rng.randrange(1000, 1 << 30)}
    if call == "search":
        kind = rng.choice(["three", "three", "sharing", "binary"])
        c.update(n=rng.randint(4, {"three": 18, "sharing": 17, "binary": 28}[kind]),
                 sharing=kind == "sharing", binary=kind == "binary")
    elif call == "range":
        lo = rng.uniform(0.0, 0.9)
        c.update(n=rng.randint(10, 19), lo=lo, hi=lo + math.exp(rng.uniform(math.log(0.001), math.log(0.1))))
    elif call == "batch":
        c.update(n=rng.randint(5, 13), scenarios=rng.randint(1, 13), replicas=rng.randint(1, 64),
                 ragged=rng.random() < 0.5)
    elif call == "reprobes":
        c.update(n=rng.randint(4, 36), sharing=rng.random() < 0.25)
    elif call == "pruned":
        c.update(n=rng.randint(14, 18))
    else:
        c.update(n=rng.randint(4, 36), sharing=rng.random() < 0.25,
                 count=int(math.exp(rng.uniform(math.log(100), math.log(500_000)))))
    return _case(None, call=call, **c)


def prepare(case, seed):
    """Handles, workspace and host inputs of one call."""
    st = {"case": case}
    if case["call"] == "batch":
        base = [_instance(case, s) for s in range(case["scenarios"])]
        st["problems"] = [S.Problem.from_instance(i) for i in base]
        st["handles"] = [p.handle for p in st["problems"]]
        st["replica_problem"], st["lat"] = _replicas(case, base, seed)
        st["ws"] = S.workspace(st["handles"], len(st["replica_problem"]))
        return st
    inst = _instance(case)
    if case["call"] != "reprobes":  # reprobes keep the profiles and pass the new latencies
        inst["tools"] = _measured(inst["tools"], _rng(seed, 1))
    p = st["problem"] = S.Problem.from_instance(inst, sharing=case["sharing"])
    st["ws"] = S.pruned_workspace(p.handle) if case["call"] == "pruned" else S.workspace([p.handle])
    if case["call"] == "range":
        st["lo"], st["hi"] = _bounds(case, p.n_mappings)
    elif case["call"] == "reprobes":
        st["base"], st["lat"] = _probe_inputs(case, inst, seed)
    elif case["call"] == "score":
        st["idx"] = _indices(case, p.n_mappings, seed)
    return st


def run(st):
    call = st["case"]["call"]
    if call == "search":
        p = st["problem"]
        return S.sched_bruteforce_argmin(p.handle, 0, p.n_mappings, st["ws"])
    if call == "range":  # a shard may hold no feasible mapping: its index is then 2^64 - 1
        return np.array(S.sched_bruteforce_argmin(st["problem"].handle, st["lo"], st["hi"], st["ws"]),
                        dtype=np.uint64)
    if call == "batch":
        return np.array(S.sched_eval_batch(st["handles"], st["replica_problem"], st["lat"], st["ws"]),
                        dtype=np.int64)
    if call == "reprobes":
        p = st["problem"]
        return _columns(S.sched_eval_reprobes(p.handle, st["base"], st["ws"], st["lat"]), p.n)
    if call == "pruned":
        index, makespan, _ = S.sched_pruned_argmin(st["problem"].handle, st["ws"])
        return index, makespan
    return S.sched_eval_mappings(st["problem"].handle, st["idx"], st["ws"])


def work(case):
    """Bytes: the inputs and the answer.  flops: the integer operations of a
    sequential event-driven evaluation of each mapping that the call scores
    (per edge 3, per tool 14 and a heap's 2 log2 N, per mapping 6).  A pruned
    search has to score at least the neighbourhood of its answer."""
    out, ops, tables = 16, 0, 0
    if case["call"] == "batch":
        for s in range(case["scenarios"]):
            inst = _instance(case, s)
            ops += case["replicas"] * _size(inst) * _ops(inst)
            tables += case["replicas"] * 32 * inst["n_tools"]
        out = 16 * case["scenarios"] * case["replicas"]
    else:
        inst = _instance(case)
        total = _size(inst)
        tables = 40 * inst["n_tools"]
        if case["call"] == "range":
            lo, hi = _bounds(case, total)
            scored = hi - lo
        elif case["call"] == "score":
            scored, out = case["count"], 16 * case["count"]
        elif case["call"] == "search":
            scored = total
        else:
            scored = 1 + 2 * inst["n_tools"]
            out = 16 if case["call"] == "pruned" else 16 * scored
        ops = scored * _ops(inst)
    return {"bytes": float(tables + out), "flops": float(ops)}


def tolerance(case):
    return "exact"


def exact(case, seed):
    """The call's answer from a plain 64-bit event simulation, where it takes seconds."""
    if case["call"] == "batch":
        base = [_instance(case, s) for s in range(case["scenarios"])]
        if sum(_size(i) for i in base) * case["replicas"] > EXACT_MAPPINGS:
            return None
        rp, lat = _replicas(case, base, seed)
        out, at = [], 0
        for s in rp:
            inst = dict(base[s])
            n = inst["n_tools"]
            inst["tools"] = [list(map(int, lat[at + v])) + [inst["tools"][v][4]] for v in range(n)]
            at += n
            out.append(_argmin(inst, 0, _size(inst), False))
        return np.array(out, dtype=np.int64)
    inst = _instance(case)
    total = _size(inst)
    if case["call"] == "reprobes":
        base, lat = _probe_inputs(case, inst, seed)
        inst["tools"] = [list(map(int, r)) + [t[4]] for r, t in zip(lat, inst["tools"])]
        return _columns(_probes(inst, base, case["sharing"]), inst["n_tools"])
    inst["tools"] = _measured(inst["tools"], _rng(seed, 1))
    if case["call"] == "score":
        return _makespans(inst, _modes_of(inst, _indices(case, total, seed)), case["sharing"])
    lo, hi = _bounds(case, total) if case["call"] == "range" else (0, total)
    if hi - lo > EXACT_MAPPINGS:
        return None
    best = _argmin(inst, lo, hi, case["sharing"])
    return np.array(best, dtype=np.uint64) if case["call"] == "range" else best


# ---------------------------------------------------------------------------
# Workflows.


def _case(name, **kw):
    c = {"shape": "mixed", "tight": False, "binary": False, "sharing": False}
    c.update(kw)
    if name is not None:
        c["name"] = name
    return c


def _rng(*key):
    return random.Random(":".join(map(str, key)))


def _log_uniform(r, a, b):
    return a * math.exp(r.random() * math.log(b / a))


def _instance(case, scenario=None):
    """The case's workflow, or one of a batch's scenarios: chains, fan-outs
    whose footprints all fit, and layered workflows under a tight budget."""
    n, shape, tight, key = case["n"], case["shape"], case["tight"], (case["dag"],)
    if scenario is not None:
        if case["ragged"]:
            n -= scenario % max(1, min(6, n - 3))
        group = scenario * 13 // case["scenarios"] if case["scenarios"] > 1 else case["dag"] % 13
        shape = "chain" if group < 4 else "fanout" if group < 9 else "layered"
        tight, key = shape == "layered", (case["dag"], scenario)
    r = _rng("workflow", *key)
    tools = []
    for _ in range(n):
        gpu = round(_log_uniform(r, 1e3, 1e6))
        tools.append([gpu, max(1, round(gpu * _log_uniform(r, 0.3, 30.0))),
                      round(_log_uniform(r, 1.83e5, 1.47e7)), round(_log_uniform(r, 1e2, 1e5)),
                      r.randint(4096 if tight else 512, 24576)])
    edges = []
    if shape == "chain":
        edges = [[v, v + 1] for v in range(n - 1)]
    elif shape == "diamond":
        edges = [[0, v] for v in range(1, n - 1)] + [[v, n - 1] for v in range(1, n - 1)]
    elif shape == "layered":
        edges = [[u, v] for u in range(n) for v in range(n)
                 if v // 4 == u // 4 + 1 and r.random() < 0.35]
    elif shape == "mixed":
        order = list(range(n))
        r.shuffle(order)
        pairs = {(order[r.randrange(k)], order[k]) for k in range(1, n) for _ in range(2)
                 if r.random() < 0.4}
        edges = [list(e) for e in sorted(pairs)]
    total = sum(t[4] for t in tools)
    if tight:
        budget = total // 4
    elif shape == "fanout" or case["binary"]:
        budget = total
    else:
        budget = 49152
    inst = {"n_tools": n, "tools": tools, "edges": edges, "contention_q16": CONTENTION_Q16,
            "vram_budget_mib": budget}
    if case["binary"]:  # CPU or GPU at once; one tool in 16 has no GPU implementation
        cpu_only = set(r.sample(range(n), n // 16))
        inst["allowed"] = [1 if v in cpu_only else 3 for v in range(n)]
    return inst


def _measured(tools, r):
    """Every latency re-measured, within a fifth of the profile."""
    return [[max(1, round(x * r.uniform(0.8, 1.2))) for x in t[:4]] + list(t[4:]) for t in tools]


def _replicas(case, base, seed):
    rp, lat = [], []
    for s, inst in enumerate(base):
        for k in range(case["replicas"]):
            rp.append(s)
            lat += [t[:4] for t in _measured(inst["tools"], _rng(seed, s, k))]
    return rp, np.array(lat, dtype=np.int64)


def _bounds(case, total):
    lo = int(total * case["lo"])
    return lo, max(lo + 1, min(total, int(total * case["hi"])))


def _indices(case, total, seed):
    r = np.random.RandomState(seed % (1 << 31))
    return (r.random_sample(case["count"]) * total).astype(np.uint64)


def _probe_inputs(case, inst, seed):
    r = _rng(seed, 2)
    return r.randrange(_size(inst)), [t[:4] for t in _measured(inst["tools"], _rng(seed, 1))]


def _columns(probes, n):
    """The probes as columns of the most there can be (rows of -2 below them):
    how many swaps there are depends on the measured latencies."""
    out = {}
    for k in ("index", "makespan_us", "kind", "tool", "mode", "swap_tool"):
        out[k] = np.full(1 + 2 * n + n * (n - 1), -2, dtype=np.int64)
        out[k][:len(probes)] = [p[k] for p in probes]
    return out


def _options(inst):
    allowed = inst.get("allowed") or [7] * inst["n_tools"]
    return [[m for m in range(3) if (a >> m) & 1] for a in allowed]


def _size(inst):
    return math.prod(len(o) for o in _options(inst))


def _ops(inst):
    n = inst["n_tools"]
    return 3.0 * len(inst["edges"]) + n * (14.0 + 2.0 * math.log2(n)) + 6.0


# ---------------------------------------------------------------------------
# The schedule model in plain 64-bit arithmetic, over many mappings at once.


def _modes_of(inst, idx):
    """Modes (mappings x tools) of mapping indices: mixed radix, tool 0 lowest."""
    idx = np.asarray(idx, dtype=np.int64)
    modes = np.empty((len(idx), inst["n_tools"]), dtype=np.int8)
    for v, o in enumerate(_options(inst)):
        modes[:, v] = np.array(o, dtype=np.int8)[idx % len(o)]
        idx = idx // len(o)
    return modes


def _makespans(inst, modes, sharing):
    out = np.full(len(modes), INFEASIBLE, dtype=np.int64)
    for at in range(0, len(modes), 65536):
        _simulate(inst, modes[at:at + 65536], sharing, out[at:at + 65536])
    return out


def _simulate(inst, modes, sharing, out):
    """Event by event: release, immediate starts with the VRAM check, one
    queue admission in (ready time, tool) order, durations, next event."""
    n, budget = inst["n_tools"], inst["vram_budget_mib"]
    gpu_us, cpu_us, load, xfer, mem = np.array(inst["tools"], dtype=np.int64).T
    factor = np.array(inst["contention_q16"], dtype=np.int64)
    rate = ((1 << 33) + factor) // (2 * factor)
    preds = [sorted({u for u, v in inst["edges"] if v == w}) for w in range(n)]
    rows = np.arange(len(modes))
    queue, on_gpu = modes == 2, modes > 0
    base = np.where(queue, gpu_us + load, np.where(on_gpu, gpu_us, cpu_us))
    end = np.full(modes.shape, NEVER, dtype=np.int64)  # finish, once known
    left = np.zeros(modes.shape, dtype=np.int64)       # sharing: work still to do
    started = np.zeros(modes.shape, dtype=bool)
    t = np.zeros(len(modes), dtype=np.int64)
    while len(rows):
        now = t[:, None]
        running = started & (end > now)
        ready = np.zeros(modes.shape, dtype=np.int64)
        for v in range(n):
            for u in preds[v]:
                arrive = end[:, u] + np.where(on_gpu[:, u] != on_gpu[:, v], xfer[v], 0)
                arrive = np.where(end[:, u] <= t, arrive, NEVER)
                ready[:, v] = np.maximum(ready[:, v], arrive)
        due = ~started & (ready <= now)
        starts = due & ~queue
        used = ((running | starts) & on_gpu) @ mem
        dead = ((starts & on_gpu).any(1)) & (used > budget)
        wait = np.where(due & queue, ready, NEVER)
        head = wait.argmin(1)  # earliest ready time, lowest tool number among equals
        each = np.arange(len(rows))
        admit = (wait[each, head] < NEVER) & ~(running & queue).any(1) & (used + mem[head] <= budget)
        starts[each[admit], head[admit]] = True
        k = ((running | starts) & on_gpu).sum(1)
        level = np.clip(k, 1, len(factor)) - 1
        started |= starts
        if sharing:
            end = np.where(starts & ~on_gpu, now + base, end)
            left = np.where(starts & on_gpu, base << 16, left)
            active = (running | starts) & on_gpu
            least = np.where(active, left, NEVER).min(1)
            w = rate[level]
            after = np.where(active.any(1), t - (-least // w), NEVER)
            cpu_end = np.where(started & ~on_gpu & (end > now), end, NEVER).min(1)
            after = np.minimum(after, cpu_end)
        else:
            scaled = (base * factor[level][:, None] + 32768) >> 16
            end = np.where(starts, now + np.where(on_gpu, scaled, base), end)
            after = np.where(started & (end > now), end, NEVER).min(1)
        later = np.where(~started & (ready > now), ready, NEVER).min(1)
        after = np.minimum(after, later)
        dead |= after == NEVER
        if sharing:  # the GPU tools advance to the next event; those out of work end there
            step = np.where(dead, 0, after - t)
            left = np.where(active, left - (step * w)[:, None], left)
            end = np.where(active & (left <= 0) & ~dead[:, None], after[:, None], end)
        done = ~dead & (end < NEVER).all(1)
        out[rows[done]] = end[done].max(1)
        keep = ~(dead | done)
        rows, modes, queue, on_gpu, base, end, left, started, t = (
            x[keep] for x in (rows, modes, queue, on_gpu, base, end, left, started, after))


def _argmin(inst, lo, hi, sharing):
    best = (-1, INFEASIBLE)
    for at in range(lo, hi, 1 << 18):
        ms = _makespans(inst, _modes_of(inst, np.arange(at, min(hi, at + (1 << 18)))), sharing)
        k = int(ms.argmin())
        if ms[k] < best[1]:
            best = (at + k, int(ms[k]))
    return best if best[1] != INFEASIBLE else (S.NO_INDEX, INFEASIBLE)


def _probes(inst, base, sharing):
    """The base mapping, every single-tool move in mode order, and after a
    move to gpu_now that does not fit one swap per tool on gpu_now that may
    queue."""
    options = _options(inst)
    weight = [math.prod(len(o) for o in options[:v]) for v in range(len(options))]
    at = [int(m) for m in _modes_of(inst, [base])[0]]

    def with_mode(x, v, m):
        return x + (options[v].index(m) - options[v].index(at[v])) * weight[v]

    cands = [(base, 0, -1, -1, -1)]
    for i, o in enumerate(options):
        for m in o:
            if m == at[i]:
                continue
            x = with_mode(base, i, m)
            cands.append((x, 1, i, m, -1))
            if m == 1:
                cands += [(with_mode(x, j, 2), 2, i, 1, j) for j in range(len(options))
                          if j != i and at[j] == 1 and 2 in options[j]]
    ms = _makespans(inst, _modes_of(inst, [c[0] for c in cands]), sharing)
    out, move = [], 0
    for (x, kind, tool, mode, swap), t in zip(cands, ms):
        if kind == 1:
            move = t
        if kind != 2 or move == INFEASIBLE:
            out.append({"index": x, "makespan_us": t, "kind": kind, "tool": tool, "mode": mode,
                        "swap_tool": swap})
    return out
