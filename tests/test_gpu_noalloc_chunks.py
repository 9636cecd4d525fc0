"""Calls of the allocation-free entry point near its limits, which it works in chunks: the results of
sim_eval_plans bit for bit around the size where a second chunk begins, also replayed from a HIP graph,
and at its pace.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SHARED_EDGE, PER_CLASS_EDGE = 242282, 60266   # the largest calls of one chunk


@pytest.fixture(scope="module")
def torch():
    import torch as T
    if not T.cuda.is_available():
        pytest.skip("no GPU")
    return T


@pytest.fixture(scope="module")
def B():
    from paper_2508_05370_amd import binding
    return binding


def _plans(workloads, w, layout, n):
    if layout == "per_class":
        return workloads.het_plans(w, 0, n)
    p = workloads.plans(w, 0, n)
    p["hdr"][1::7] |= np.uint32(1 << 13)
    p["hdr"][2::7] |= np.uint32(1 << 16)
    return p


@pytest.mark.parametrize("layout,n,offset", [
    ("shared", SHARED_EDGE, 0), ("shared", SHARED_EDGE + 1, 1), ("shared", 262143, 3),
    ("per_class", PER_CLASS_EDGE, 0), ("per_class", PER_CLASS_EDGE + 1, 1), ("per_class", 65535, 2)])
def test_matches_eval_plans(torch, B, workloads, layout, n, offset):
    w = workloads.workload(3)
    sim = B.Sim(w["model"], w["cluster"])
    dp = B.device_plans(_plans(workloads, w, layout, n + offset))
    print("case: %s, %d plans from %d on" % (layout, n, offset), flush=True)
    want = sim.eval_plans(dp, n=n, offset=offset)
    out = torch.full((n + 1,), -7, dtype=torch.int64, device="cuda")
    sim.eval_plans_noalloc(dp, n=n, offset=offset, out=out)
    assert torch.equal(out[:n], want) and int(out[n]) == -7


@pytest.mark.parametrize("layout,n", [("shared", 262144), ("per_class", 65536)])
def test_replayed_from_a_graph(torch, B, workloads, layout, n):
    w = workloads.workload(3)
    sim = B.Sim(w["model"], w["cluster"])
    dp = B.device_plans(_plans(workloads, w, layout, n))
    out = torch.empty(n, dtype=torch.int64, device="cuda")
    print("case: graph of %d %s plans" % (n, layout), flush=True)
    sim.eval_plans_noalloc(dp, out=out)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        sim.eval_plans_noalloc(dp, out=out)
    for shift in (0, 5, 11):   # other plans in the same buffers between the replays
        for v in dp.values():
            v.copy_(torch.roll(v, shift, -1))
        want = sim.eval_plans(dp)
        out.fill_(-7)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want), shift


# the allocating entry point has continuation lists of 224 bytes per plan; lists that fill up cost a
# factor of three at these sizes, a second chunk's launches half
@pytest.mark.parametrize("layout,n", [("shared", 242000), ("shared", 262144), ("per_class", 30000),
                                      ("per_class", 65536)])
def test_pace(torch, B, workloads, layout, n):
    w = workloads.workload(3)
    sim = B.Sim(w["model"], w["cluster"])
    dp = B.device_plans(_plans(workloads, w, layout, n))
    out = torch.empty(n, dtype=torch.int64, device="cuda")
    print("case: pace of %d %s plans" % (n, layout), flush=True)

    def median(call):
        t = []
        for i in range(14):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            call(dp, out=out)
            b.record()
            b.synchronize()
            if i >= 3:
                t.append(a.elapsed_time(b))
        return sorted(t)[len(t) // 2]
    slow, fast = median(sim.eval_plans_noalloc), median(sim.eval_plans)
    print("allocation-free %.0f us, allocating %.0f" % (slow * 1e3, fast * 1e3), flush=True)
    assert slow < 2.1 * fast
