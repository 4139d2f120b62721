"""The memory that making the dense matrix of the smallest levels takes: bounded
where a small domain lies in a large lattice, within a server's budget, and not
needed for the V-cycle where it cannot be had."""
import os
import subprocess
import sys
import time

import numpy as np
import pytest

import workloads as W

try:  # import at collection time: the first import on a fresh machine is slow
    import torch  # noqa: F401
except ImportError:  # pragma: no cover
    torch = None

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

def test_large_lattices_are_passed_over():
    """8 columns on the lattices up to level 4 (129^3 nodes) would take 630 MB;
    up to level 3 they take 80 MB."""
    from paper_2508_11608_amd import Problem

    P = Problem(W.Workload("small-ball", 3, 2, 6, centers=((0.02, 0.01, 0.03),), semi=((0.06,) * 3,)))
    try:
        assert P.ndofs(3) < P.ndofs(4) <= 2048
        r = torch.from_numpy(W.random_vector(P.ndofs(), seed=5)).cuda()
        P.timing(["cut_solve"])
        P.vcycle(r)
        launches = [P.timing_read("cut_solve", l)[0] for l in range(6)]
        P.timing([])
        print(f"\n  cut colour steps by level: {launches}", flush=True)
        assert launches[4] > 0 and not any(launches[:4])
    finally:
        P.close()


def test_server_budget_without_room_for_it():
    """A budget of exactly one hierarchy and its columns: the matrix is made
    without scratch, with the same bits."""
    from paper_2508_11608_amd import Server, footprint

    w = W.disc_q2()
    fb, n = footprint(w, fp32=True, multi=True)
    xs = []
    for budget in (fb + 2 * 8 * 8 * n, 8 << 30):
        srv = Server(budget, 1)
        t = srv.submit(w, fourier=W.fourier_modes(2, 77), fp32=True)
        while (got := srv.poll(t, n)) is None:
            time.sleep(0.001)
        srv.close()
        assert got[0]["status"] == 0
        xs.append(got[1])
    assert np.array_equal(xs[0], xs[1])


SHIM = r"""
#include <dlfcn.h>
#include <stddef.h>
static size_t limit = (size_t)-1;
void fail_from(size_t n) { limit = n; }
int hipMalloc(void** p, size_t n) {
  static int (*real)(void**, size_t);
  if (!real) {
    void* h = dlopen("libamdhip64.so.7", RTLD_NOW | RTLD_NOLOAD);
    if (h) *(void**)&real = dlsym(h, "hipMalloc");
  }
  if (!real || n >= limit) return 2;  /* hipErrorOutOfMemory */
  return real(p, n);
}
"""
CHILD = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)  # its hipMalloc comes before the runtime's
shim.fail_from.argtypes = [ctypes.c_size_t]
import torch
import workloads as W
from paper_2508_11608_amd import Problem
NEVER = 2**64 - 1
w = W.ball_q2().with_levels(4)
out = []
for limit in (NEVER, 32 << 20, 16 << 20):  # nothing fails; the scratch does; the matrix (23 MB) does
    shim.fail_from(limit)
    P = Problem(w)
    r = torch.from_numpy(W.random_vector(P.ndofs(), seed=6)).cuda()
    z = P.vcycle(r)
    shim.fail_from(NEVER)
    P.timing(["cut_solve"])
    assert torch.equal(P.vcycle(r), z)
    out.append((z, P.timing_read("cut_solve", 1)[0]))
    P.close()
(z0, n0), (z1, n1), (z2, n2) = out
assert n0 == 0 and n1 == 0 and n2 > 0, (n0, n1, n2)  # steps run on level 1
assert torch.equal(z0, z1)
assert float((z0 - z2).abs().max() / z0.abs().max()) < 1e-11
print("child ok")
"""


def test_short_memory(tmp_path):
    """Device allocations that fail, in a process of its own whose hipMalloc is
    the test's: without scratch the same bits, without the matrix every level is
    run (equal to rounding)."""
    src, lib = tmp_path / "shim.c", tmp_path / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(lib), str(src), "-ldl"], check=True)
    env = dict(os.environ, PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, "-c", CHILD, str(lib)], cwd=ROOT, env=env, capture_output=True, text=True,
                       timeout=100)
    print(r.stdout + r.stderr[-2000:], flush=True)
    assert r.returncode == 0 and "child ok" in r.stdout
