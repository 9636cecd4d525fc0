"""Clusters of sixteen device types, the most a plan can name, whose table images are as large as the
evaluation kernels take into LDS, against the CPU oracle bit for bit.

The lanes' counters take 256 bytes per type and wavefront beside the image: at 64 KB of it a block asks for
up to 128 KB (the per-class layout's sync pass) and 116 KB (the kernel of every kind of plan).
"""
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


# nodes per type and devices per node: the whole image in LDS (65024 of at most 65536 bytes), all but the
# device rows (65536), nothing (more than that)
@pytest.mark.parametrize("nodes,dpn", [(10, 8), (88, 4), (90, 4)])
@pytest.mark.parametrize("kind,n", [("plain", 20011), ("plain", 131075), ("overlap", 20011), ("zero_bubble", 20011),
                                    ("interleaved", 20011), ("per_class", 20011)])
def test_sixteen_types(B, oracle_mod, workloads, nodes, dpn, kind, n):
    m = workloads.model("llama-70b")
    c = workloads.cluster_random(9, [nodes] * 16, dpn=dpn, nic_choices=(200, 400), pcie=False, jitter=True)
    gen = {"interleaved": workloads.random_plans_il, "per_class": workloads.random_plans_het}
    p = gen.get(kind, workloads.random_plans)(m, c, 77, 0, n)
    p["hdr"] |= np.uint32({"overlap": 1 << 13, "zero_bubble": 1 << 16}.get(kind, 0))
    print("case: 16 types of %d nodes of %d, %d %s plans" % (nodes, dpn, n, kind), flush=True)
    got = B.times_u64(B.Sim(m, c).eval_plans(B.device_plans(p)))
    want = oracle_mod.Oracle(m, c).eval(p)
    bad = np.nonzero(got != want)[0]
    assert bad.size == 0, "%d of %d plans differ, first %d: gpu %d oracle %d" % (
        bad.size, n, bad[0], int(got[bad[0]]), int(want[bad[0]]))
    used = p["types"][:, want != np.uint64(2**64 - 1)]
    assert used.size > 2 * n and len({int(t >> np.uint64(4 * s)) & 15 for t in used[0, :500] for s in range(4)}) == 16
