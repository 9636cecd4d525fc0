"""Outputs of eval_memory and eval_stages whose kernels share work across lanes: calls that end inside a
wavefront, and plans with few and many stages next to each other, against the CPU oracle, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_05370_amd import binding
    return binding


def _batches(W, w, n):
    yield "shared", W.plans(w, 0, n)
    yield "per class", W.het_plans(w, 0, n)
    yield "interleaved", W.interleaved_plans(w, 0, n)
    p = W.plans(w, 0, n)
    p["cut"][0, ::3] = 0          # every third plan breaks a rule
    yield "invalid", p


@pytest.mark.parametrize("n", [1, 63, 64, 65, 130, 257])
@pytest.mark.parametrize("idx", [3, 4])
def test_memory_and_stage_records(B, oracle_mod, workloads, n, idx):
    w = workloads.workload(idx)
    sim, o = B.Sim(w["model"], w["cluster"]), oracle_mod.Oracle(w["model"], w["cluster"])
    for name, p in _batches(workloads, w, n):
        print("case: %s, %d plans" % (name, n), flush=True)
        dp = B.device_plans(p)
        mem = sim.eval_memory(dp).cpu().numpy().view(np.uint64)
        st, cl = (x.cpu().numpy() for x in sim.eval_stages(dp))
        for i in range(n):
            want = o.stage_mem(p, i)
            assert np.array_equal(mem[i], np.full((4, 16), 2**64 - 1, np.uint64) if want is None else want), (name, i)
            d = o.detail(p, i)
            if d is None:
                assert not cl[i].any() and not st[i].any(), (name, i)
                continue
            for c in range(d["G"]):
                for s, (f, b) in enumerate(zip(d["f"][c], d["b"][c])):
                    assert (int(st[i, c, s, 0]), int(st[i, c, s, 1])) == (f, b), (name, i, c, s)
                if name != "interleaved":
                    S = d["S_class"][c]
                    assert [int(x) for x in st[i, c, :S, 3]] == d["tdp"][c], (name, i, c)
                    assert [int(x) for x in st[i, c, :S - 1, 2]] == d["c"][c][:S - 1], (name, i, c)
                assert not st[i, c, len(d["f"][c]):].any(), (name, i, c)
