"""The pipeline recurrence at the edges of its parts, against the CPU oracle, bit for bit.

The recurrence starts from a closed form of the warm-up, runs steady iterations with a shortcut for
periodic schedules, hands schedules that stay aperiodic to the continuation lists, and ends with a drain:
micro-batch counts around each of those lengths for every stage count, every order of passes, lists that
one pass or the other goes on with, and lists that are too small for what they are offered.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

KINDS = {"1f1b": 0, "overlap": 1 << 13, "zero_bubble": 1 << 16}


def _plans(w, stages, n, seed, batch, classes):
    """n plans of every stage count in `stages`: random cuts and types, `classes` replicas of one class each
    (the first with a random share of the micro-batches, at least one each)."""
    rng = np.random.default_rng(seed)
    L, K = w["model"]["L"], len(w["cluster"]["types"])
    tot = n * len(stages)
    p = dict(hdr=np.zeros(tot, np.uint32), cut=np.zeros((16, tot), np.uint8), cls=np.zeros((4, tot), np.uint32),
             types=np.zeros((4, tot), np.uint64))
    i = 0
    for S in stages:
        for _ in range(n):
            p["hdr"][i] = (S - 1) << 4 | (classes - 1) << 8 | int(rng.integers(2)) << 10
            cuts = np.sort(rng.choice(np.arange(1, L), S - 1, replace=False)) if S > 1 else []
            for s, v in enumerate(list(cuts) + [L]):
                p["cut"][s, i] = v
            share = rng.multinomial(batch - classes, np.ones(classes) / classes) + 1
            for c in range(classes):
                p["cls"][c, i] = 1 | int(share[c]) << 16
                p["types"][c, i] = sum(int(rng.integers(K)) << (4 * s) for s in range(S))
            i += 1
    return p


def _check(B, O, model, cluster, p, noalloc=False):
    import torch
    sim = B.Sim(model, cluster)
    dp = B.device_plans(p)
    if noalloc:
        out = torch.empty(len(p["hdr"]), dtype=torch.int64, device="cuda")
        sim.eval_plans_noalloc(dp, out=out)
    else:
        out = sim.eval_plans(dp)
    got = B.times_u64(out)
    want = O.Oracle(model, cluster).eval(p)
    bad = np.nonzero(got != want)[0]
    assert bad.size == 0, "%d of %d plans differ, first %d: gpu %d oracle %d" % (
        bad.size, len(want), bad[0], int(got[bad[0]]), int(want[bad[0]]))
    assert np.count_nonzero(want != np.uint64(2**64 - 1)) > len(want) // 2


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_05370_amd import binding
    return binding


# warm-up only (fewer micro-batches than stages), no or one or two steady iterations, the first pass's
# budget (S + 8) and the first continuation pass's (48) and a few around them, long loops
@pytest.mark.parametrize("batch", [1, 2, 3, 7, 15, 16, 17, 18, 24, 25, 40, 41, 72, 73, 96, 129, 1000])
def test_micro_batch_counts(B, oracle_mod, workloads, batch):
    w = workloads.workload(5)
    model = dict(w["model"], global_batch=batch)
    for kind, bits in KINDS.items():
        for classes in (1, 2, 3, 4):
            if batch < classes:
                continue
            p = _plans(w, range(1, 17), 24, 1000 * batch + classes, batch, classes)
            p["hdr"] |= np.uint32(bits)
            print("case: %s, %d micro-batches, %d classes" % (kind, batch, classes), flush=True)
            _check(B, oracle_mod, model, w["cluster"], p)


# 16-stage plans over slow links through the allocation-free entry point
@pytest.mark.parametrize("kind", list(KINDS))
def test_continuation_lists_no_allocation(B, oracle_mod, workloads, kind):
    w = workloads.workload(2)
    model = dict(w["model"], global_batch=160)
    cluster = dict(w["cluster"], types=[dict(t, nic_MBps=t["nic_MBps"] // 8) for t in w["cluster"]["types"]])
    p = _plans(w, [16], 20000, 7, 160, 2)
    p["hdr"] |= np.uint32(KINDS[kind])
    print("case: %s, %d plans" % (kind, len(p["hdr"])), flush=True)
    _check(B, oracle_mod, model, cluster, p, noalloc=True)


# first lists on either side of the length that the matrix powers take alone, in calls on either side of the one-launch
# limit (2^17 plans); all end within the first continuation pass's budget
@pytest.mark.parametrize("n", [60001, 131072, 131073])
def test_continuation_lists_96(B, oracle_mod, workloads, n):
    w = workloads.workload(2)
    model = dict(w["model"], global_batch=96)
    cluster = dict(w["cluster"], types=[dict(t, nic_MBps=t["nic_MBps"] // 8) for t in w["cluster"]["types"]])
    p = _plans(w, [13], n, 11, 96, 2)
    print("case: %d plans" % n, flush=True)
    _check(B, oracle_mod, model, cluster, p)


def _two_class_plans(w, S, n, seed, batch):
    """n plans of S stages and two classes of one replica each, random cuts, types and shares."""
    rng = np.random.default_rng(seed)
    L, K = w["model"]["L"], len(w["cluster"]["types"])
    p = dict(hdr=np.full(n, (S - 1) << 4 | 1 << 8, np.uint32), cut=np.zeros((16, n), np.uint8),
             cls=np.zeros((4, n), np.uint32), types=np.zeros((4, n), np.uint64))
    p["cut"][:S - 1] = np.sort(np.argsort(rng.random((n, L - 1)), axis=1)[:, :S - 1] + 1, axis=1).T
    p["cut"][S - 1] = L
    share = rng.binomial(batch - 2, 0.5, n).astype(np.uint32) + 1
    for c, m in enumerate((share, np.uint32(batch) - share)):
        p["cls"][c] = 1 | m << 16
        for s in range(S):
            p["types"][c] |= rng.integers(0, K, n).astype(np.uint64) << np.uint64(4 * s)
    return p


# Where plans whose schedules stay aperiodic go, as the host's replay of a sample says before the GPU runs them:
# "power": the first list is short enough for the matrix powers alone;
# "cont":  the first continuation pass runs, and what it leaves fits the second list;
# "full":  both lists are offered more than they hold (links a 32nd as fast).
# In the one-launch kernel (up to 2^17 plans) and the four-launch one, every kind that uses the lists, both layouts
# and both entry points.
@pytest.mark.parametrize("kind,S,slow,batch,n,where", [
    ("1f1b", 13, 8, 600, 20001, "power"),
    ("1f1b", 13, 8, 2400, 60001, "cont"), ("1f1b", 13, 8, 2400, 131072, "cont"), ("1f1b", 13, 8, 2400, 131073, "cont"),
    ("overlap", 13, 8, 2400, 131073, "cont"), ("zero_bubble", 13, 8, 2400, 131073, "cont"),
    ("per_class", 13, 8, 2400, 60001, "cont"),
    ("1f1b", 16, 32, 600, 60001, "full"), ("1f1b", 13, 32, 600, 131073, "full"), ("overlap", 16, 32, 600, 60001, "full"),
    ("zero_bubble", 16, 32, 600, 60001, "full"), ("per_class", 16, 32, 600, 60001, "full"),
    ("noalloc", 16, 16, 600, 60001, "cont"), ("noalloc", 16, 32, 600, 262144, "full")])
def test_continuation_lists(B, oracle_mod, workloads, kind, S, slow, batch, n, where):
    import chain_replay as R
    w = workloads.workload(2)
    model = dict(w["model"], global_batch=batch)
    cluster = dict(w["cluster"], types=[dict(t, nic_MBps=t["nic_MBps"] // slow) for t in w["cluster"]["types"]])
    p = _two_class_plans(w, S, n, 11, batch)
    p["hdr"] |= np.uint32(KINDS.get(kind, 0))
    zb = kind == "zero_bubble"
    ch = R.chains(oracle_mod.Oracle(model, cluster), p, range(400), S, zb)
    left = ch.first_pass(zb)
    offered = left >= R.POWER_MIN
    second = ch.cont_pass(np.where(offered, left, 0)) >= 2 * R.POWER_MIN
    # entries offered to the first list and held there -- four fifths of lists of 224 bytes per plan (of 1300 in
    # the smaller allocation-free call) -- and offered to the second one, a quarter of it
    first = 2 * n * offered.mean()
    held = 0.8 * (1300 if kind == "noalloc" and n < 131072 else 224) * n / (32 * S)
    then = second[offered].mean() * min(first, held)
    print("case: %s, %d plans of %d stages: %.0f then %.0f entries offered, %.0f and %.0f held" % (
        kind, n, S, first, then, held, held / 4), flush=True)
    if where == "power":
        assert 1000 < first < 0.9 * R.CONT_FEW and first < held
    elif where == "cont":
        assert 1.2 * R.CONT_FEW < first < 0.9 * held and 500 < then < 0.9 * held / 4
    else:
        assert first > 1.1 * held > 1.3 * R.CONT_FEW and then > 1.1 * held / 4
    _check(B, oracle_mod, model, cluster, workloads.as_per_class(p) if kind == "per_class" else p,
           noalloc=kind == "noalloc")


# Second lists of more than 32768 entries, which go on lane by lane: all of them (600 micro-batches), and all but the
# few that have thousands of iterations left and keep to the matrix powers (replicas of 5700 short micro-batches among
# replicas of 475)
@pytest.mark.parametrize("kind,far", [("1f1b", False), ("zero_bubble", False), ("per_class", False), ("1f1b", True)])
def test_long_second_list(B, oracle_mod, workloads, kind, far):
    import chain_replay as R
    S, n, batch, slow = 13, 400001, 6000 if far else 600, 32
    w = workloads.workload(2)
    model = dict(w["model"], global_batch=batch)
    cluster = w["cluster"]
    if far:
        model["seq"], cluster = 256, workloads.cluster_random(2, [40, 40, 40])
    cluster = dict(cluster, types=[dict(t, nic_MBps=t["nic_MBps"] // slow) for t in cluster["types"]])
    p = _two_class_plans(w, S, n, 11, batch)
    if far:
        reps = np.where(np.random.default_rng(3).random(n) < 0.06, 1, 12).astype(np.uint32)
        share = np.minimum(p["cls"][0] >> 16, 300).astype(np.uint32)
        p["cls"][0], p["cls"][1] = 1 | share << 16, reps | (np.uint32(batch) - share) << 16
    p["hdr"] |= np.uint32(KINDS.get(kind, 0))
    zb = kind == "zero_bubble"
    ch = R.chains(oracle_mod.Oracle(model, cluster), p, range(400), S, zb)
    left = ch.first_pass(zb)
    offered = left >= R.POWER_MIN
    left = ch.cont_pass(np.where(offered, left, 0))
    second = left >= 2 * R.POWER_MIN
    # (capacities as in test_continuation_lists)
    held = 0.8 * 224 * n / (32 * S)
    then = min(second[offered].mean() * min(2 * n * offered.mean(), held), held / 4)
    print("case: %s, far %d: %.0f entries in the second list, %.2f %% of them far" % (
        kind, far, then, 100 * np.mean(left[second] * S >= 64000)), flush=True)
    assert then > 1.1 * 32768 and np.any(left[second] * S >= 64000) == far
    _check(B, oracle_mod, model, cluster, workloads.as_per_class(p) if kind == "per_class" else p)


# Sweeps over slow links beside the same plans over the workload's own: 3.0 times as long with one matrix power per
# entry of the second list (70000 of them), 2.0 lane by lane
def test_pace_over_slow_links(B, workloads):
    import torch
    w = workloads.workload(2)
    dp = B.device_plans(workloads.plans(w, 0, 1 << 20))
    out = torch.empty(1 << 20, dtype=torch.int64, device="cuda")
    took = []
    for slow in (1, 8):
        print("case: links 1/%d" % slow, flush=True)
        sim = B.Sim(w["model"], dict(w["cluster"], types=[dict(t, nic_MBps=t["nic_MBps"] // slow)
                                                           for t in w["cluster"]["types"]]))
        t = []
        for i in range(14):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            sim.eval_plans(dp, out=out)
            b.record()
            b.synchronize()
            if i >= 3:
                t.append(a.elapsed_time(b))
        took.append(sorted(t)[len(t) // 2])
    print("%.0f us, slow links %.0f" % (took[0] * 1e3, took[1] * 1e3), flush=True)
    assert took[1] < 2.5 * took[0]
