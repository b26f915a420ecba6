"""Timed cases of the library: what a program that uses it has it do.

A case names the call it makes ("call"), the formulas it makes it on
("formula" and its sizes) and the options it is made with.  Formulas come from
workloads/ and a seed: random systems of clauses, the theories of the paper's
examples with a few random facts added (clauses of three literals, as a user
adds an assumption to a theory), and random DAGs.

Calls:
  count      fbg.count                 the number of models
  dnf        fbg.eval_dnf              the DNF vector
  models     fbg.enumerate_models      the models, ascending, and their number
  read       fbg.enumerate_dnf         the models read off a stored DNF vector
  step       Batch.eval_dnf + Batch.enumerate  vectors, counts and models of a batch
  counts     Batch.count               the counts of a batch
  slice      Server.launch             one slice of the serving loop
"""

import math
import re

import numpy as np
import torch

import workloads
from paper_1310_6978_amd import fbg
from workloads.formulas import cnf_clause_count


def listed():
    return [
        # the smallest calls a program makes of the library: a theory over 15
        # letters (equivalence relations on 6 elements), counted and listed;
        # latency and launches
        {"name": "count_theory_n15", "call": "count", "formula": "equivalence", "size": 6, "facts": 3},
        {"name": "models_theory_n21", "call": "models", "formula": "equivalence", "size": 7, "facts": 3},
        # an ordinary system of equations: its vector (2 MiB), its count
        {"name": "dnf_cnf_n24", "call": "dnf", "formula": "cnf", "size": 24, "clauses": 88},
        {"name": "count_cnf_n27", "call": "count", "formula": "cnf", "size": 27, "clauses": 100},
        # a large one, 2^35 valuations
        {"name": "count_cnf_n35", "call": "count", "formula": "cnf", "size": 35, "clauses": 136},
        # a formula that is more than clauses: the paper's script (posets with
        # a special element) on 6 elements, 30 letters
        {"name": "count_script_n30", "call": "count", "formula": "special_posets", "size": 6, "facts": 3},
        # many models (millions): triangle-free graphs on 8 vertices
        {"name": "models_dense_n28", "call": "models", "formula": "triangle_free", "size": 8, "facts": 2},
        # few models in a large space, with the uniform cofactor:
        # equivalence relations on 9 elements
        {"name": "models_cofactor_n36", "call": "models", "formula": "equivalence", "size": 9, "facts": 3,
         "cofactor": True, "words_per_lane": 32},
        # the models of a vector that is already there (128 MiB), a system
        # with few enough equations to have many solutions
        {"name": "read_cnf_n30", "call": "read", "formula": "cnf", "size": 30, "clauses": 60},
        # the batched step: vectors, counts and models of 16 systems of 2^32
        # valuations
        {"name": "step_cnf_16xn32", "call": "step", "formula": "cnf", "size": 32, "count": 16},
        # counts of many small general formulas in one call
        {"name": "counts_dag_256", "call": "counts", "formula": "dag", "count": 256, "size_lo": 10, "size": 30,
         "nodes": 2000},
        # a slice of the serving loop: a share of each of 48 requests
        {"name": "slice_48_requests", "call": "slice", "formula": "requests", "count": 48, "size_lo": 12, "size": 36,
         "slice_words": 2.5e11},
    ]


def draw(rng):
    """One more case of the ranges the listed ones stand for (a size is the
    logarithm of the work)."""
    call = rng.choice(["count", "count", "dnf", "models", "models", "read", "step", "counts", "slice"])
    if call in ("count", "models"):
        formula = rng.choice(["cnf", "cnf", "equivalence", "triangle_free", "special_posets", "permutations"])
        case = {"call": call, "formula": formula, "seeded": rng.randrange(1 << 20)}
        if formula == "cnf":
            case["size"] = rng.randint(12, 34 if call == "count" else 31)
            case["clauses"] = int(case["size"] * rng.uniform(2.5, 4.0))
        else:
            lo, hi = {"equivalence": (6, 8), "triangle_free": (6, 8), "special_posets": (5, 6),
                      "permutations": (5, 5)}[formula]
            case["size"] = rng.randint(lo, hi)
            case["facts"] = rng.randint(1, 6)
            if formula != "special_posets" and rng.random() < 0.3:
                case["cofactor"] = True
                case["words_per_lane"] = rng.choice([8, 16, 32])
        return case
    if call in ("dnf", "read"):
        n = rng.randint(12, 31)
        return {"call": call, "formula": "cnf", "size": n, "clauses": int(n * rng.uniform(2.0, 4.0))}
    if call == "step":
        n = rng.randint(14, 31)
        return {"call": call, "formula": "cnf", "size": n, "count": rng.randint(2, 16),
                "clauses": int(n * rng.uniform(3.5, 4.25))}
    if call == "counts":
        return {"call": call, "formula": "dag", "count": rng.randint(24, 200), "size_lo": rng.randint(8, 14),
                "size": rng.randint(20, 30), "nodes": rng.randint(200, 2000)}
    return {"call": call, "formula": "requests", "count": rng.randint(8, 48), "size_lo": 12,
            "size": rng.randint(22, 36), "slice_words": 10.0 ** rng.uniform(10, 11.39)}


# ------------------------------------------------------------------ formulas

def _facts(n, count, rng):
    """`count` random clauses of three literals over n letters."""
    out = []
    for _ in range(count):
        vs = rng.choice(n, size=3, replace=False)
        out.append(" | ".join(("~x%d" if rng.integers(2) else "x%d") % v for v in vs))
    return "".join(c + "\n" for c in out)


def _texts(case, seed):
    """The formulas of a case: [(text, n)]."""
    rng = np.random.default_rng([int(seed), int(case.get("seeded", 0))])
    new = lambda: int(rng.integers(1 << 62))  # noqa: E731
    f, size = case["formula"], case["size"]
    if f == "cnf":
        m = case.get("clauses") or cnf_clause_count(size)
        return [workloads.random_3cnf(size, m, new()) for _ in range(case.get("count", 1))]
    if f == "dag":
        # the letters run through the whole range, the nodes are spread over
        # their logarithm
        lo = case["size_lo"]
        out = []
        for i in range(case["count"]):
            nodes = int(50 * math.exp(rng.random() * math.log(case["nodes"] / 50)))
            out.append(workloads.random_dag(lo + i % (size - lo + 1), nodes, new()))
        return out
    if f == "requests":
        # every tenth a theory, the others systems of clauses
        lo = case["size_lo"]
        out = []
        for i in range(case["count"]):
            if i % 10 == 9:
                t, n = [workloads.permutation_matrices(5), workloads.triangle_free(8),
                        workloads.equivalence_relations(9)][(i // 10) % 3]
                if n <= size:
                    out.append((t, n))
                    continue
            n = lo + int(rng.integers(size - lo + 1))
            out.append(workloads.random_3cnf(n, cnf_clause_count(n), new()))
        return out
    t, n = {"equivalence": workloads.equivalence_relations, "triangle_free": workloads.triangle_free,
            "special_posets": workloads.special_element_posets,
            "permutations": workloads.permutation_matrices}[f](size)
    return [(t + _facts(n, case["facts"], rng), n)]


def _capacity(case):
    """Entries of a list of models: what the theory has without the facts, or
    four times what a random system has on average (the list then ends there
    if there are more)."""
    if case["formula"] == "cnf":
        n = case["size"]
        return 4096 + int(4 * 2.0 ** n * 0.875 ** (case.get("clauses") or cnf_clause_count(n)))
    t, n = _texts(dict(case, facts=0), 0)[0]
    return int(fbg.count(fbg.Program(t, n)).item())


# ----------------------------------------------------------------- the calls

def prepare(case, seed):
    texts = _texts(case, seed)
    call = case["call"]
    flags = fbg.compile_wpl(16) if call == "slice" else 0   # as the serving loop compiles
    progs = [fbg.Program(t, n, flags) for t, n in texts]
    s = {"call": call, "progs": progs}
    p, n = progs[0], texts[0][1]
    if case.get("cofactor"):
        p.set_tuning(case["words_per_lane"], cofactor=True)
    buf = lambda k: torch.full((max(int(k), 1),), -1, dtype=torch.int64, device="cuda")  # noqa: E731
    if call == "dnf":
        s["dnf"] = buf(fbg.dnf_words(n))
    elif call in ("models", "read"):
        cap = _capacity(case)
        s.update(n=n, capacity=cap, models=buf(cap), total=buf(1))
        if call == "read":
            s["dnf"] = fbg.eval_dnf(p)
    elif call == "step":
        b = fbg.Batch(progs)
        s.update(batch=b, dnf=[buf(fbg.dnf_words(k)) for _, k in texts])
        b.set_dnf_outputs(s["dnf"])
        s["models"] = [buf(_capacity(case)) for _ in progs]
        b.set_enum_outputs(s["models"])
        s["counts"] = buf(len(progs))
    elif call == "counts":
        s.update(batch=fbg.Batch(progs), counts=buf(len(progs)))
    elif call == "slice":
        s["server"] = fbg.Server(max_programs=256, max_items=16384, words_per_lane=16, nbuf=6, cofactor=True)
        share = case["slice_words"] / len(progs)
        s["items"] = []
        for i, q in enumerate(progs):
            chunk = max(1, int(share // (max(1, q.info["n_instr"]) * 64 * 16)))
            s["items"].append((i, i, 0, min(chunk, fbg.program_tiles(q, 16))))
    torch.cuda.synchronize()
    return s


def run(s):
    call = s["call"]
    if call == "count":
        return {"count": fbg.count(s["progs"][0])}
    if call == "dnf":
        return {"dnf": fbg.eval_dnf(s["progs"][0], out=s["dnf"])}
    if call == "models":
        m, t = fbg.enumerate_models(s["progs"][0], s["capacity"], out=s["models"], total=s["total"])
        return {"models": m, "total": t}
    if call == "read":
        m, t = fbg.enumerate_dnf(s["dnf"], s["n"], s["capacity"], out=s["models"], total=s["total"])
        return {"models": m, "total": t}
    if call == "step":
        s["batch"].eval_dnf(counts=s["counts"])
        s["batch"].enumerate()
        return {"dnf": s["dnf"], "counts": s["counts"], "models": s["models"]}
    if call == "counts":
        return {"counts": s["batch"].count(out=s["counts"])}
    counts = torch.zeros(len(s["progs"]), dtype=torch.int64, device="cuda")
    s["server"].launch(s["progs"], s["items"], counts)
    return {"counts": counts}


def work(case):
    """Bytes: the results (and a vector that is read).  "flops": two-input
    operations of the formulas on 32-bit words, the time model of the method
    (one per operation of the term and 32 valuations)."""
    texts = _texts(case, 0)
    infos = [fbg.Program(t, n, fbg.compile_wpl(16)).info for t, n in texts]
    ops = [max(1, i["l2in"]) * 2.0 ** max(0, n - 5) for i, (_, n) in zip(infos, texts)]
    if case["call"] == "slice":
        share = case["slice_words"] / len(texts)
        ops = [min(o, share * i["l2in"] / max(1, i["n_instr"])) for o, i in zip(ops, infos)]
    nbytes = 8 * len(texts)
    if case["call"] in ("dnf", "read", "step"):
        nbytes += sum(8 * fbg.dnf_words(n) for _, n in texts)
    if case["call"] in ("models", "read", "step"):
        for t, n in texts:
            nbytes += 8 * min(_capacity(case), int(fbg.count(fbg.Program(t, n)).item()))
    return {"bytes": nbytes, "flops": sum(ops)}


# --------------------------------------------------------------------- exact

_EXACT_VARS = 22


def _vector(text, n):
    """The DNF vector by its definition, as uint64 words (6 <= n): every
    statement evaluated on whole generator rows."""
    w = np.arange(1 << (n - 6), dtype=np.uint64)
    ones = np.full(w.shape, ~np.uint64(0))
    env = {"ONE": ones, "ZERO": np.zeros_like(ones)}
    bit = np.arange(64, dtype=np.uint64)
    for k in range(n):
        if k < 6:
            mask = np.bitwise_or.reduce(((bit >> np.uint64(k)) & np.uint64(1)) << bit)
            env["x%d" % k] = np.full(w.shape, mask)
        else:
            env["x%d" % k] = np.uint64(0) - ((w >> np.uint64(k - 6)) & np.uint64(1))
    acc = ones.copy()
    for line in text.splitlines():
        line = re.sub(r"\b1\b", "ONE", re.sub(r"\b0\b", "ZERO", line.strip()))
        name, eq, expr = line.partition("=")
        if eq:
            env[name.strip()] = eval(expr, {"__builtins__": {}}, env)
        elif line:
            acc &= eval(line, {"__builtins__": {}}, env)
    return acc


def exact(case, seed):
    if case["size"] > _EXACT_VARS or case["call"] == "slice":
        return None
    texts = _texts(case, seed)
    if max(n for _, n in texts) > _EXACT_VARS:
        return None
    vec = [_vector(t, n) for t, n in texts]
    models = [np.flatnonzero(np.unpackbits(v.view(np.uint8), bitorder="little")) for v in vec]
    as_i64 = lambda a: torch.from_numpy(np.ascontiguousarray(a).view(np.int64))  # noqa: E731
    counts = torch.tensor([len(m) for m in models])
    call = case["call"]
    padded = []
    if call in ("models", "read", "step"):
        cap = _capacity(case)
        for m in models:
            padded.append(torch.full((cap,), -1, dtype=torch.int64))
            padded[-1][:min(cap, len(m))] = torch.from_numpy(m[:cap].astype(np.int64))
    if call == "count":
        return {"count": counts}
    if call == "dnf":
        return {"dnf": as_i64(vec[0])}
    if call in ("models", "read"):
        return {"models": padded[0], "total": counts}
    if call == "step":
        return {"dnf": [as_i64(v) for v in vec], "counts": counts, "models": padded}
    return {"counts": counts}
