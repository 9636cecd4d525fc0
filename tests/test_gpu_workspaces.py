"""The workspaces that calls share: one per concurrently used stream, kept between calls and contexts,
given back with the last context, and never shared by calls that may overlap.
"""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


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


def _used(torch):
    torch.cuda.synchronize()
    free, total = torch.cuda.mem_get_info()
    return total - free


def test_kept_and_given_back(torch, B, workloads):
    """Passes over three contexts in turn, each waited for: one workspace (326 bytes per plan), the same
    from pass to pass -- released and taken again, as it was, it now and then cost 10 ms to 2 s -- and gone
    with the contexts."""
    import gc
    gc.collect()   # (contexts of earlier tests)
    w = workloads.workload(3)
    n = 2_000_001
    dp = B.device_plans(workloads.plans(w, 0, n))
    out = torch.empty(n, dtype=torch.int64, device="cuda")
    first = B.Sim(w["model"], w["cluster"])
    first.eval_plans(dp, n=100, out=out)
    first.close()
    start = _used(torch)
    sims = [B.Sim(w["model"], w["cluster"]) for _ in range(3)]
    used = []
    for i in range(60):
        sims[i % 3].eval_plans(dp, out=out)
        used.append(_used(torch) - start)
    print("bytes used: %s" % sorted(set(used)), flush=True)
    assert len(set(used[3:])) == 1 and used[-1] < 1.2 * 326 * n + (64 << 20)
    for s in sims:
        s.close()
    assert _used(torch) - start < 64 << 20


def test_streams_and_sizes(torch, B, workloads):
    """Calls of many sizes on more streams than workspaces are kept for, two contexts and both layouts,
    with nothing waited for between them."""
    w = workloads.workload(3)
    n = 120_000
    sims = [B.Sim(w["model"], w["cluster"]) for _ in range(2)]
    plans = [B.device_plans(workloads.plans(w, 0, n)), B.device_plans(workloads.het_plans(w, 0, n))]
    want = [sims[0].eval_plans(p) for p in plans]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(11)]
    rng = np.random.default_rng(5)
    jobs = []
    for i in range(220):
        m = int(rng.integers(1, n)) if i % 3 else n
        o, kind, st = int(rng.integers(0, n - m + 1)), i % 2, streams[int(rng.integers(11))]
        with torch.cuda.stream(st):
            out = torch.full((m,), -7, dtype=torch.int64, device="cuda")
        sims[(i // 2) % 2].eval_plans(plans[kind], n=m, offset=o, out=out, stream=st)
        jobs.append((kind, o, m, out))
    torch.cuda.synchronize()
    bad = [(k, o, m) for k, o, m, out in jobs if not torch.equal(out, want[k][o:o + m])]
    assert not bad, bad[:5]


def test_threads(torch, B, workloads):
    """Threads with a stream each: times and stage records, one context."""
    w = workloads.workload(2)
    n = 50_000
    sim = B.Sim(w["model"], w["cluster"])
    dp = B.device_plans(workloads.plans(w, 0, n))
    want, (rec, cls) = sim.eval_plans(dp), sim.eval_stages(dp, n=2000)
    torch.cuda.synchronize()
    wrong = []

    def work(i):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            for j in range(20):
                m = n - 1000 * ((i + j) % 5)
                t = sim.eval_plans(dp, n=m, stream=st)
                r, c = sim.eval_stages(dp, n=2000, stream=st)
                st.synchronize()
                if not (torch.equal(t, want[:m]) and torch.equal(r, rec) and torch.equal(c, cls)):
                    wrong.append((i, j))
    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong, wrong[:5]
