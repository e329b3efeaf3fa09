"""What the framework is asked to do, as cases that can be timed and compared.

A pass is what a program does with the simulator: replay every simulation of
one batch and read the results back.  A batch is a set of programs (operator
traces or operator logs), each at several memory budgets under several
heuristics.  Most programs keep a ``Simulator`` (inputs validated, derived and
uploaded once) and run it; ``run`` of a kept handle is then ``sim.run()`` and
``sim.results()``.  The one-shot cases call ``dtr.run`` / ``dtr.run_log``,
which also validate, derive and upload.

A case is a dict:
  kind     the family of programs (see ``_programs``)
  n        its size parameter: chain length, blocks, layers, trees, forward
           operators, or operators/instructions of a random program
  count    how many programs of that size (each from its own seed)
  budgets  budgets per program, spaced evenly over ``lo``..100 percent of the
           program's peak memory without eviction
  heur     heuristics, separated by commas (or "family": all 16 h'(s, m, c))
  policy   deallocation policies, separated by commas
  search   search approximations, added up (1: ignore small, 2: sample)
  mode     "kept" (a handle, its own workspace), "static" (a handle run with
           the library's static working memory) or "oneshot"

Results are whole numbers and compared exactly.
"""
import math

import numpy as np

from paper_2006_09616_amd import dtr
from paper_2006_09616_amd import workloads as W

HEUR = {name: k for k, name in enumerate(W.HEURISTIC_NAMES)}
POLICY = {"eager": W.POLICY_EAGER, "ignore": W.POLICY_IGNORE, "banish": W.POLICY_BANISH}
SIX = "dtr,eq,local,lru,size,rand"
LOG_KINDS = ("resnetlog", "randomlog")


def _case(name, kind, n, budgets, lo, heur, count=1, policy="eager", search=0, mode="kept"):
    c = dict(kind=kind, n=n, count=count, budgets=budgets, lo=lo, heur=heur, policy=policy, search=search, mode=mode)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest batch a user runs: a 32-layer chain at five budgets; launches and latency are all of it
        _case("chain32", "chain", 32, 5, 19, "dtr"),
        # deep rematerialization (stacks of hundreds of operators) from a serving loop that may not allocate
        _case("chain600 static", "chain", 600, 16, 8, "dtr,eq,lru", mode="static"),
        # a new set of small programs each time: validated, derived, uploaded, run and read in one call
        _case("programs oneshot", "program", 60, 3, 33, SIX + ",estar,msps", count=48, mode="oneshot"),
        # the budget sweep of a residual network's training step under every heuristic of the paper's main figure
        _case("resnet50 sweep", "resnet", 50, 256, 10, SIX),
        # the budget sweep of a transformer encoder
        _case("transformer12 sweep", "transformer", 12, 512, 15, "dtr,eq,lru"),
        # many programs of different lengths, as dynamic models give them: trees, 8 budgets each, h_DTR^eq
        _case("treelstm", "treelstm", 400, 8, 20, "eq", count=192),
        # a long irregular program under the exact e* neighbourhood
        _case("randdag3000", "randdag", 3000, 48, 20, "dtr"),
        # the deallocation study: the same sweep without eager eviction
        _case("resnet50 policies", "resnet", 50, 64, 15, "dtr,local,lru,msps", policy="ignore,banish"),
        # the ablation study: all members of h'(s, m, c)
        _case("resnet50 family", "resnet", 50, 32, 12, "family"),
        # the prototype's search approximations
        _case("treelstm search", "treelstm", 300, 6, 30, "eq,dtr,lru", count=24, search=3),
        # operator logs with views, in-place and multi-output calls: a training step's log under six heuristics
        _case("resnet50 log", "resnetlog", 50, 128, 10, SIX),
        # many short logs, every kind of instruction in them
        _case("random logs", "randomlog", 150, 3, 40, "dtr,eq,lru,msps", count=48),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["chain", "program", "resnet", "transformer", "treelstm", "randdag", "resnetlog", "randomlog"])
    count, policy, search, mode = 1, "eager", 0, "kept"
    heur = rng.choice(["dtr", "eq", "lru", "dtr,eq", "dtr,eq,lru", SIX, "eq,local,size,rand", "msps,estar,local"])
    if kind == "chain":
        n, budgets, lo = _log_uniform(rng, 8, 800), _log_uniform(rng, 1, 40), rng.randint(8, 40)
        mode = rng.choice(["kept", "static"])
        lo = max(lo, -(-400 // n))                       # at least four tensors
    elif kind == "program":
        n, count, budgets, lo = _log_uniform(rng, 10, 400), _log_uniform(rng, 1, 64), rng.randint(1, 5), rng.randint(30, 60)
        mode = rng.choice(["kept", "oneshot"])
    elif kind == "resnet":
        n, budgets, lo = _log_uniform(rng, 4, 60), _log_uniform(rng, 4, 256), rng.randint(10, 40)
        if rng.random() < 0.3:
            heur, policy = "dtr,lru,size", rng.choice(["banish", "eager,banish", "ignore"])
            budgets = min(budgets, 64)
        elif rng.random() < 0.3:
            search = rng.randint(1, 3)
        mode = rng.choice(["kept", "kept", "static"])
    elif kind == "transformer":
        n, budgets, lo = _log_uniform(rng, 1, 14), _log_uniform(rng, 4, 512), rng.randint(15, 40)
    elif kind == "treelstm":
        n, count, budgets, lo = _log_uniform(rng, 16, 320), _log_uniform(rng, 1, 96), rng.randint(1, 8), rng.randint(25, 60)
        heur = rng.choice(["eq", "eq", "eq,lru"])
        search = rng.choice([0, 0, 1])
    elif kind == "randdag":
        n, budgets, lo = _log_uniform(rng, 100, 2500), _log_uniform(rng, 2, 48), rng.randint(25, 60)
        heur = rng.choice(["dtr", "dtr,eq", "msps"])
    elif kind == "resnetlog":
        n, budgets, lo = _log_uniform(rng, 3, 50), _log_uniform(rng, 2, 128), rng.randint(12, 50)
    else:
        n, count, budgets, lo = _log_uniform(rng, 10, 400), _log_uniform(rng, 1, 64), rng.randint(1, 4), rng.randint(30, 60)
        mode = rng.choice(["kept", "oneshot"])
        if rng.random() < 0.4:
            heur, policy = "dtr,lru,local", rng.choice(["banish", "ignore", "eager,banish"])
    return _case(None, kind, n, budgets, lo, heur, count, policy, search, mode)


def _programs(case, seed):
    """The programs and their peaks.  The model-like ones follow the recipes
    of ``workloads``; where a recipe has no random draw, the seed sets a free
    size of it (sequence length, unit cost)."""
    n, kind = case["n"], case["kind"]
    progs, peaks = [], []
    for i in range(case["count"]):
        k = W.splitmix64((seed << 16) + i) & 0x7FFFFFFF
        if kind == "chain":
            p = W.chain_trace(n, size=1, cost=1 + k % 97)
        elif kind == "program":
            p = W.random_program(k, n_ops=max(4, n - k % (n // 2)), n_const=k % 4, backward=k % 2 == 0)
        elif kind == "resnet":
            p = W.resnet_trace(seed=k, blocks=n)
        elif kind == "transformer":
            p = W.transformer_trace(layers=n, seq=448 + k % 129)
        elif kind == "treelstm":
            p = W.treelstm_trace(k, min_leaves=max(2, n // 8), max_leaves=n)
        elif kind == "randdag":
            p = W.random_dag_trace(seed=k, n_forward=n)
        elif kind == "resnetlog":
            p = W.resnet_log(seed=k, blocks=n)
        else:
            p = W.random_log(k, n_steps=max(8, n - k % (n // 2)), n_const=k % 4)
        progs.append(p)
        peaks.append(W.log_peak(p) if kind in LOG_KINDS else W.natural_peak(p))
    return progs, peaks


def _batch(case, seed):
    progs, peaks = _programs(case, seed)
    heurs = list(W.ALL_FAMILY) if case["heur"] == "family" else [HEUR[h] for h in case["heur"].split(",")]
    rows = []
    for pol in case["policy"].split(","):
        for i, peak in enumerate(peaks):
            for h in heurs:
                lo, nb = case["lo"], case["budgets"]
                budgets = W.linear_budgets(peak, lo, 100, nb) if nb > 1 else [peak * lo // 100]
                for b in budgets:
                    rows.append((i, h, max(1, int(b)), (seed << 32) + len(rows), POLICY[pol], case["search"]))
    return progs, W.make_specs(rows)


def prepare(case, seed):
    progs, specs = _batch(case, seed)
    st = dict(case=case, progs=progs, specs=specs, sim=None)
    logs = case["kind"] in LOG_KINDS
    if case["mode"] != "oneshot":
        flags = dtr.OPT_STATIC_SCRATCH if case["mode"] == "static" else 0
        st["sim"] = (dtr.Simulator(None, specs, logs=progs, flags=flags) if logs
                     else dtr.Simulator(progs, specs, flags=flags))
    return st


def run(state):
    sim = state["sim"]
    if sim is None:
        call = dtr.run_log if state["case"]["kind"] in LOG_KINDS else dtr.run
        res = call(state["progs"], state["specs"])
    else:
        if state["case"]["mode"] == "static":
            sim.run_static()
        else:
            sim.run()
        res = sim.results()
    return {f: res[f] for f in res.dtype.names}


def _sizes(case):
    """Operators and operator inputs of the case's programs (of the recipes; a
    random program's or tree's expected ones), and its simulations."""
    n, c = case["n"], case["count"]
    ops = {"chain": 2 * n + 2, "program": 1.1 * n, "resnet": 12 * n + 4, "transformer": 92 * n + 4,
           "treelstm": 20 * 0.56 * n, "randdag": 2 * n, "resnetlog": 18 * n + 9, "randomlog": 0.5 * n}[case["kind"]]
    heurs = 16 if case["heur"] == "family" else len(case["heur"].split(","))
    sims = c * case["budgets"] * heurs * len(case["policy"].split(","))
    return ops * c, 2.0 * ops * c, sims, ops


def work(case):
    """Each program and spec read once, each result written once.  The
    arithmetic no replay can do without: every operator is executed once per
    simulation (clock, memory, locks and release of about two inputs: some 20
    integer operations); how often it is executed again and how many
    candidates are scored depends on the inputs and is left out."""
    ops, edges, sims, per = _sizes(case)
    return {"bytes": ops * (8 + 1 + 4 + 8 + 8) + 4 * edges + sims * (32 + 104), "flops": 20.0 * sims * per}


def tolerance(case):
    return "exact"


# ---- the chain cases in plain Python ---------------------------------------

def _plain(tr, budget, h):
    """One replay of a trace under h_DTR, h_DTR^eq or h_LRU with eager
    eviction, step by step (Section 2, Appendix C), with exact fractions
    compared by cross-multiplication."""
    n, F = tr.n_tensors, tr.n_ops
    ins = [[int(u) for u in tr.op_inputs[tr.op_input_offsets[o]:tr.op_input_offsets[o + 1]]] for o in range(F)]
    out = [int(t) for t in tr.op_output]
    size = [int(v) for v in tr.tensor_size]
    const = [bool(f & W.FLAG_CONSTANT) for f in tr.tensor_flags]
    req = [t for t in range(n) if tr.tensor_flags[t] & W.FLAG_REQUIRED]
    parents, kids, cost, last = [[] for _ in range(n)], [[] for _ in range(n)], [0] * n, {}
    for o in range(F):
        parents[out[o]], cost[out[o]] = ins[o], int(tr.op_cost[o])
        last[out[o]] = max(last.get(out[o], -1), o)
        for u in ins[o]:
            kids[u].append(out[o])
            last[u] = o
    rel = [[] for _ in range(F)]
    for t in range(n):
        if t in last and t not in req:
            rel[last[t]].append(t)
    state = ["const" if const[t] else "new" for t in range(n)]
    locks, stamp, node = [0] * n, [0] * n, [-1] * n
    link, total = [], []                      # union-find: parent link, running cost
    r = dict.fromkeys(dtr.RESULT_FIELDS, 0)
    mem = peak = sum(size[t] for t in range(n) if const[t])
    clock = 0

    class Oom(Exception):
        pass

    def find(x):
        while link[x] != x:
            x = link[x]
        return x

    def reach(t, nbs):
        seen, todo = set(), [t]
        while todo:
            for v in nbs[todo.pop()]:
                if state[v] == "evicted" and v not in seen:
                    seen.add(v)
                    todo.append(v)
        return seen

    def neighbourhood(t):
        if h == W.H_LRU:
            return 0
        r["n_adj_visits"] += len(parents[t]) + len(kids[t])
        if h == W.H_DTR:
            near = reach(t, parents) | reach(t, kids)
            r["n_nbr_visits"] += len(near)
            return sum(cost[v] for v in near)
        near = [v for v in parents[t] + kids[t] if state[v] == "evicted"]
        r["n_nbr_visits"] += len(near)
        return sum(total[k] for k in {find(node[v]) for v in near})

    def evict(t, eager):
        nonlocal mem
        state[t] = "evicted"
        mem -= size[t]
        r["n_eager_evictions" if eager else "n_evictions"] += 1
        node[t] = len(link)
        link.append(len(link))
        total.append(cost[t])
        for v in parents[t] + kids[t]:
            if v != t and state[v] == "evicted":
                a, b = find(node[t]), find(node[v])
                if a != b:
                    link[b] = a
                    total[a] += total[b]

    def call(t, remat):
        nonlocal mem, peak, clock
        for u in parents[t]:
            locks[u] += 1
        for u in parents[t]:
            if state[u] == "evicted":
                call(u, True)
        while mem + size[t] > budget:
            best = None
            for x in range(n):
                if state[x] != "resident" or locks[x]:
                    continue
                r["n_scores"] += 1
                num = 1 if h == W.H_LRU else cost[x] + neighbourhood(x)
                den = (1 if h == W.H_LRU else size[x]) * (clock - stamp[x])
                if best is None or num * best[1] < best[0] * den:
                    best = (num, den, x)
            if best is None:
                raise Oom
            evict(best[2], False)
        for u in parents[t] + [t]:
            stamp[u] = clock
        clock += cost[t]
        r["n_executed_ops"] += 1
        r["n_remats"] += remat
        r["remat_cost" if remat else "base_cost"] += cost[t]
        mem += size[t]
        peak = max(peak, mem)
        if remat:
            total[find(node[t])] -= cost[t]
        state[t] = "resident"
        for u in parents[t]:
            locks[u] -= 1

    at, status = 0, 0
    try:
        if mem > budget:
            raise Oom
        for at in range(F):
            call(out[at], 0)
            for t in sorted(rel[at]):
                if state[t] == "resident" and not locks[t]:
                    evict(t, True)
        at = F
        for t in req:
            locks[t] += 1
            if state[t] == "evicted":
                call(t, 1)
    except Oom:
        status = 1
    r.update(total_cost=r["base_cost"] + r["remat_cost"], peak_memory=peak, final_memory=mem, status=status,
             failed_op=at if status else -1)
    return r


def exact(case, seed):
    """Chains up to a few dozen layers in plain Python; the others take a
    plain replay minutes to hours."""
    if case["kind"] != "chain" or case["n"] * case["budgets"] * len(case["heur"].split(",")) > 2000:
        return None
    if not set(case["heur"].split(",")) <= {"dtr", "eq", "lru"}:
        return None
    progs, specs = _batch(case, seed)
    rows = [_plain(progs[s["trace"]], int(s["budget"]), int(s["heuristic"])) for s in specs]
    kinds = {f: dtr.RESULT_DTYPE[f] for f in dtr.RESULT_DTYPE.names}
    return {f: np.array([r[f] for r in rows], dtype=kinds[f]) for f in kinds}
