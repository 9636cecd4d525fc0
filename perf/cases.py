"""Performance cases of the plan evaluator: the calls a plan search makes, through the binding.

Each case is one pass over plans that are already in device memory: iteration times and the best plan
(`kind` "sweep", "small" or "chunks"), the per-stage quantities of a shortlist ("stages") or the
per-device memory of one ("memory").  `workload` names one of the package's five seeded workloads;
`schedule`, `layout`, `mem` and `net` are the options a plan or a cluster may have.  All results are
whole numbers (picoseconds, bytes, indices) fixed by integer rules, so they compare exactly.
"""
import numpy as np
import torch

from paper_2508_05370_amd import binding as B
from paper_2508_05370_amd import workloads as W

GPT2, LLAMA7B, LLAMA70B, MIXTRAL, GPT3 = 1, 2, 3, 4, 5
EXHAUSTIVE_PLANS = 29470

OVERLAP_BIT, ZERO_BUBBLE_BIT = 1 << 13, 1 << 16


def _case(kind, workload, plans, schedule="1f1b", layout="shared", mem=False, net="ring"):
    return dict(kind=kind, workload=workload, plans=plans, schedule=schedule, layout=layout, mem=mem, net=net)


def listed():
    def named(name, c):
        return dict(c, name=name)
    return [
        # one step of a local search: a plan's neighbours, in a serving loop that allocates nothing
        named("search_step_96", _case("small", LLAMA7B, 96)),
        # every plan of a small cluster, enumerated exhaustively
        named("exhaustive_gpt2_29470", _case("sweep", GPT2, EXHAUSTIVE_PLANS)),
        # the stage-by-stage breakdown of a shortlist
        named("stages_llama70b_20011", _case("stages", LLAMA70B, 20011)),
        # peak memory of every device of a shortlist
        named("memory_llama70b_250000", _case("memory", LLAMA70B, 250000)),
        # an ordinary random search on a mid-sized cluster
        named("sweep_llama7b_1M", _case("sweep", LLAMA7B, 1 << 20)),
        # the benchmark's sweep: a large model on a jittered 512-device cluster
        named("sweep_llama70b_16M", _case("sweep", LLAMA70B, 1 << 24)),
        # mixture of experts: EP degrees and skewed expert loads
        named("sweep_mixtral_4M", _case("sweep", MIXTRAL, 1 << 22)),
        # the largest cluster, in chunks on two streams with one reduction
        named("chunks_gpt3_8M", _case("chunks", GPT3, 1 << 23)),
        # replica classes of different TP degree, depth and layer split
        named("per_class_llama70b_3000001", _case("sweep", LLAMA70B, 3000001, layout="per_class")),
        # a search over schedules: plain 1F1B, overlapped gradient sync and the zero-bubble order mixed
        named("schedules_llama70b_2500003", _case("sweep", LLAMA70B, 2500003, schedule="mix")),
        # interleaved 1F1B, two to four model chunks per device
        named("interleaved_llama70b_2M", _case("sweep", LLAMA70B, 1 << 21, schedule="interleaved")),
        # device capacities given: plans that do not fit are dropped
        named("fits_memory_llama70b_4M", _case("sweep", LLAMA70B, 1 << 22, mem=True)),
    ]


def _log_size(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random())) | (1 if rng.random() < 0.5 else 0)


def draw(rng):
    kind = rng.choice(["small", "sweep", "sweep", "sweep", "sweep", "sweep", "chunks", "stages", "memory"])
    workload = rng.choice([LLAMA7B, LLAMA70B, LLAMA70B, MIXTRAL, GPT3])
    layout = rng.choice(["shared", "shared", "shared", "per_class"])
    schedule = "1f1b" if layout == "per_class" else rng.choice(["1f1b", "1f1b", "1f1b", "overlap", "zero_bubble",
                                                                "mix", "interleaved"])
    net = rng.choice(["ring", "ring", "ring", "ring", "tree", "rail", "hier" if layout == "shared" else "contention"])
    mem = kind not in ("memory", "stages") and rng.random() < 0.15
    plans = {"small": (16, 60000), "sweep": (200, 1 << 22), "chunks": (1 << 20, 1 << 22), "stages": (100, 60000),
             "memory": (1000, 400000)}[kind]
    return _case(kind, workload, _log_size(rng, *plans), schedule, layout, mem, net)


def _plans(w, case, seed):
    """Host plans of the case: a range of the workload's seeded generator that the seed chooses (the
    exhaustive workload: its plans in an order that the seed chooses)."""
    n = case["plans"]
    if case["workload"] == GPT2:
        p = W.plans(w)
        order = np.random.default_rng(seed).permutation(EXHAUSTIVE_PLANS)[:n]
        return {k: np.ascontiguousarray(v[..., order]) for k, v in p.items()}
    first = (seed % (1 << 20)) << 26
    if case["layout"] == "per_class":
        return W.het_plans(w, first, n)
    if case["schedule"] == "interleaved":
        return W.interleaved_plans(w, first, n)
    p = W.plans(w, first, n)
    if case["schedule"] == "overlap":
        p["hdr"] |= np.uint32(OVERLAP_BIT)
    elif case["schedule"] == "zero_bubble":
        p["hdr"] |= np.uint32(ZERO_BUBBLE_BIT)
    elif case["schedule"] == "mix":
        bits = np.array([0, OVERLAP_BIT, ZERO_BUBBLE_BIT], dtype=np.uint32)
        p["hdr"] |= bits[np.random.default_rng(seed).integers(0, 3, n)]
    return p


def prepare(case, seed):
    w = W.workload(case["workload"])
    if case["mem"]:
        w = W.with_memory(w)
    flag = {"tree": "ccl_tree", "rail": "rail_only", "hier": "ccl_hier", "contention": "contention"}.get(case["net"])
    cluster = dict(w["cluster"], **{flag: 1}) if flag else w["cluster"]
    n = case["plans"]
    s = dict(case=case, sim=B.Sim(w["model"], cluster), plans=B.device_plans(_plans(w, case, seed)),
             out=torch.empty(n, dtype=torch.int64, device="cuda"),
             best=torch.empty(2, dtype=torch.int64, device="cuda"))
    if case["kind"] == "chunks":
        size = 1 << 22 if n > 1 << 22 else -(-n // 4)
        s["chunks"] = [(o, min(size, n - o)) for o in range(0, n, size)]
        s["slots"] = torch.empty((len(s["chunks"]), 2), dtype=torch.int64, device="cuda")
        s["streams"] = [torch.cuda.Stream() for _ in range(2)]
    return s


def run(s):
    case, sim, dp, out, best = s["case"], s["sim"], s["plans"], s["out"], s["best"]
    kind = case["kind"]
    if kind == "stages":
        return sim.eval_stages(dp)
    if kind == "memory":
        return sim.eval_memory(dp)
    if kind == "small":
        limit = B.SIM_NOALLOC_MAX_PLANS_PER_CLASS if case["layout"] == "per_class" else B.SIM_NOALLOC_MAX_PLANS
        assert case["plans"] <= limit
        sim.eval_plans_noalloc(dp, out=out)
        sim.argmin(out, out=best)
    elif kind == "sweep":
        sim.eval_plans(dp, out=out)
        sim.argmin(out, out=best)
    else:
        main = torch.cuda.current_stream()
        ready = main.record_event()
        for j, (o, m) in enumerate(s["chunks"]):
            st = s["streams"][j % 2]
            st.wait_event(ready)
            sim.eval_plans(dp, n=m, offset=o, out=out[o:o + m], stream=st)
            sim.argmin(out[o:o + m], index_base=o, out=s["slots"][j], stream=st)
        for st in s["streams"]:
            main.wait_stream(st)
        sim.best_reduce(s["slots"], out=best, stream=main)
    return out, best


# Arithmetic a plan cannot do without, in VALU operations: its stages' costs, links and gradient syncs
# (about 1100 on the random workloads), and the schedule's warm-up, two steady iterations and drain
# (about 1200); the memory of its devices takes about 600.
def work(case):
    n = case["plans"]
    plan_in = 120 if case["layout"] == "per_class" else 68
    if case["kind"] == "stages":
        # only the records of stages that exist must be written, but the caller's array is zeroed: all of it
        return dict(bytes=n * (plan_in + 4 * 16 * 4 * 8 + 16), flops=n * 1100)
    if case["kind"] == "memory":
        return dict(bytes=n * (plan_in + 4 * 16 * 8), flops=n * 600)
    return dict(bytes=n * (plan_in + 8 + 8), flops=n * (600 if case["mem"] else 2300))


def tolerance(case):
    return "exact"


def exact(case, seed):
    """None: the outputs are whole numbers defined by integer rules (every division rounds up), compared
    bit for bit; there is no 64-bit approximation to measure an error against."""
    return None
