"""Code of the library's headers that also compiles for the host, checked there (CPU only): the
continuation pass's jump bound, and the sizes of the workspaces.

The kernels are compiled with -ffinite-math-only, under which an infinity or a NaN is an undefined
value: the arithmetic of the bound must not raise either.
"""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2508_05370_amd", "csrc")

HARNESS = r"""
#include <fenv.h>
#include "device.h"

// the allocation-free workspace: bytes of it, and of a call of n plans its bytes with its continuation lists, and those
// of the lists
extern "C" uint64_t noalloc_bytes() { return hetsim::kNoAllocBytes; }
extern "C" void noalloc_call(int64_t n, int het, uint64_t* r) {
  r[1] = hetsim::noalloc_cont(n, het);
  r[0] = hetsim::work_bytes(n, het, r[1]);
}

// bytes of the workspace a call takes where the largest allocation is `most` (0: none)
extern "C" uint64_t taken(int nbuf, int64_t ch, int het, uint64_t most) {
  size_t got = 0, cont = 0;
  const bool ok = hetsim::alloc_work(
      [&](size_t bytes) {
        got = bytes <= most ? bytes : 0;
        return got ? (void*)&got : nullptr;
      },
      nbuf, ch, het, &cont);
  return ok && got == nbuf * hetsim::work_bytes(ch, het, cont) ? got : 0;
}

// lead_bits over n pairs; returns the floating-point exceptions that an infinity or a NaN raises
extern "C" int lead_bits_all(const double* dx, const double* dr, int64_t n, uint32_t* bits) {
  feclearexcept(FE_ALL_EXCEPT);
  for (int64_t i = 0; i < n; ++i) bits[i] = hetsim::lead_bits(dx[i], dr[i], [](float y) { return 1.0f / y; });
  return fetestexcept(FE_DIVBYZERO | FE_INVALID | FE_OVERFLOW);
}
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    d = tmp_path_factory.mktemp("host_build")
    src, lib = str(d / "harness.hip"), str(d / "harness.so")
    with open(src, "w") as f:
        f.write(HARNESS)
    subprocess.run(["hipcc", "--offload-host-only", "-O0", "-std=c++17", "-fPIC", "-shared", "-I", CSRC, "-I",
                    os.path.join(ROOT, "include"), src, "-o", lib], check=True, stderr=subprocess.PIPE)
    return C.CDLL(lib)


def _lead_bits(host, dx, dr):
    dx, dr = np.ascontiguousarray(dx, np.float64), np.ascontiguousarray(dr, np.float64)
    bits = np.empty(dx.size, np.uint32)
    host.lead_bits_all.argtypes = [C.c_void_p, C.c_void_p, C.c_int64, C.c_void_p]
    return host.lead_bits_all(dx.ctypes.data, dr.ctypes.data, dx.size, bits.ctypes.data), bits


def test_jump_bound_is_finite_and_right(host):
    """An argument of max(x, y) that leads by |dx| and loses |dr| per step leads for |dx| / |dr| steps
    (bits of an fp32 number, shortened by 1e-5 where they are used: rounding dx and dr to fp32, the
    reciprocal and the product lose less than 4 * 2^-24 of it); every other pair gives bits above any
    number's, so that a minimum drops them.  Ties and equal rates, the commonest pairs, included."""
    v = [0, 1, 2, 3, 7, 1000, 2**24 + 1, 2**40, 2**52, 2**53 - 1, 2**62]
    v = np.array([-x for x in v] + v, np.float64)
    dx, dr = (a.ravel() for a in np.meshgrid(v, v))
    rng = np.random.default_rng(1)
    r = rng.integers(-2**53, 2**53, (2, 20000)) >> rng.integers(0, 53, (2, 20000))
    dx, dr = np.concatenate([dx, r[0]]), np.concatenate([dr, r[1]])
    raised, bits = _lead_bits(host, dx, dr)
    assert raised == 0
    meets = (dx != 0) & (dr != 0) & (np.sign(dx) != np.sign(dr))
    assert np.all(bits[~meets] > np.float32(1e9).view(np.uint32))
    want = -dx[meets] / dr[meets]
    assert np.all(np.abs(bits[meets].view(np.float32) - want) <= 4 * 2.0**-24 * want + 1e-30)


@pytest.mark.parametrize("het", [0, 1])
def test_allocation_free_workspace(host, het):
    """Every call of the allocation-free entry point fits its static workspace, at most 82 MiB, with
    continuation lists of at least sim_eval_plans' 224 bytes per plan: random plans leave 28-58 there,
    sweeps over slow links more than 96, and a full list keeps whole wavefronts to the end of their
    longest pipeline."""
    from paper_2508_05370_amd import binding as B
    host.noalloc_bytes.restype = C.c_uint64
    total = host.noalloc_bytes()
    assert total <= 82 << 20
    most = B.SIM_NOALLOC_MAX_PLANS_PER_CLASS if het else B.SIM_NOALLOC_MAX_PLANS
    r = (C.c_uint64 * 2)()
    for n in list(range(1, 300)) + list(range(301, most, 97)) + [most - 1, most]:
        host.noalloc_call(C.c_int64(n), het, r)
        used, lists = r
        assert used <= total and lists >= max(224 * n, 1 << 20), (n, used, lists)


@pytest.mark.parametrize("het,per_plan", [(0, 168), (1, 744)])
def test_workspace_where_memory_is_short(host, het, per_plan):
    """A call goes on with smaller continuation lists where the device has no room for the full ones: it
    then needs at most 2 MiB (counters, and the smallest lists) beside the bytes per plan that it took
    before there were lists."""
    host.taken.restype = C.c_uint64

    def taken(nbuf, n, most):
        return host.taken(nbuf, C.c_int64(n), het, C.c_uint64(most))
    for nbuf, n in [(1, 1), (1, 4096), (1, 100003), (1, 1 << 20), (1, 1 << 22), (2, 1 << 21)]:
        plenty, short = taken(nbuf, n, 1 << 40), nbuf * (per_plan * n + (2 << 20))
        assert 0 < taken(nbuf, n, short) <= short and plenty >= taken(nbuf, n, short)
        assert taken(nbuf, n, plenty) == plenty and taken(nbuf, n, 1 << 10) == 0


@pytest.mark.parametrize("het,other", [(0, 110), (1, 700)])
def test_small_calls_have_longer_lists(host, het, other):
    """Lists of a call, from its workspace without the other buffers (about `other` bytes per plan): 224
    bytes per plan, in calls of up to 300000 plans as much as 64 MiB or 896 bytes per plan, the smaller."""
    host.taken.restype = C.c_uint64
    for n in (1, 1000, 30000, 60000, 120000, 240000, 300000, 1 << 20, 1 << 22):
        lists = host.taken(1, C.c_int64(n), het, C.c_uint64(1 << 40)) - other * n
        want = max(224 * n, min(896 * n, 64 << 20), 1 << 20)
        assert abs(lists - want) < (2 << 20) + want // 16, (n, lists, want)
