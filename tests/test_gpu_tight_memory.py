"""A solve with a dense nonsymmetric operator on a device that has no room for
several exponentials at a time forms them one after the other, to the same bits.
The device's room is set from the host: a small library that stands before the
HIP runtime in symbol lookup refuses allocations past a limit (in a process of
its own)."""
import os
import subprocess
import sys

import pytest

from tests.gpu_common import announce

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#include <dlfcn.h>
#include <stddef.h>
#include <map>
#include <mutex>
static std::mutex mu;
static std::map<void*, size_t> live;
static size_t now, top, limit;
static void* real(const char* name) {
  static void* lib = dlopen("libamdhip64.so.7", RTLD_LAZY | RTLD_NOLOAD);
  return dlsym(lib, name);
}
extern "C" {
int hipMalloc(void** p, size_t bytes) {
  static auto f = (int (*)(void**, size_t))real("hipMalloc");
  std::lock_guard<std::mutex> g(mu);
  if (limit && now + bytes > limit) return 2;  // hipErrorOutOfMemory
  const int rc = f(p, bytes);
  if (rc == 0) { live[*p] = bytes; now += bytes; top = now > top ? now : top; }
  return rc;
}
int hipFree(void* p) {
  static auto f = (int (*)(void*))real("hipFree");
  std::lock_guard<std::mutex> g(mu);
  auto it = live.find(p);
  if (it != live.end()) { now -= it->second; live.erase(it); }
  return f(p);
}
void room_set(size_t bytes) { limit = bytes; top = now; }
size_t room_top() { return top; }
}
"""

CHILD = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
shim.room_set.argtypes = [ctypes.c_size_t]
shim.room_top.restype = ctypes.c_size_t
import numpy as np
import workloads as wl
from paper_1805_08990_amd import _binding as b

n, h = 700, 0.01
A = wl.random_nonsymmetric(n, seed=3)
A = A - 1.2 * np.linalg.norm(A, 2) * np.eye(n)
C = wl.random_C(1, n, 5)

def solve(split, precision, room):
    c = b.Context(0)
    shim.room_set(room)
    try:
        opts = b.SolveOptions(T=2 * h, h=h, tol=1e-10, split=split, precision=precision, max_rank=32)
        L, D, _ = c.solve("dle", opts, A, C)
        return np.array(L), np.array(D), shim.room_top()
    finally:
        shim.room_set(0)
        c.close()

for precision in ("fp64", "mixed"):
    L, D, most = solve("F12", precision, 0)
    one = solve("F1F2", precision, 0)[2]  # e^{hA^T} alone: no quadrature nodes
    room = one + 3 * 8 * n * n            # and a node, its product, and one to spare
    print(f"[case] tight memory {precision}: {most >> 20} MiB at most, {room >> 20} given", flush=True)
    assert most > room + 4 * 8 * n * n, "the limit would not be felt"
    Lt, Dt, top = solve("F12", precision, room)
    assert top <= room
    assert np.array_equal(L, Lt) and np.array_equal(D, Dt)
"""


def test_exponentials_one_after_the_other(tmp_path):
    announce("tight memory")
    src, lib = tmp_path / "room.cpp", tmp_path / "libroom.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", str(lib), str(src), "-ldl"], check=True, timeout=60)
    child = tmp_path / "child.py"
    child.write_text(CHILD)
    r = subprocess.run([sys.executable, "-u", str(child), str(lib)], cwd=ROOT, timeout=100, capture_output=True,
                       text=True, env={**os.environ, "PYTHONPATH": ROOT})
    print(r.stdout, flush=True)
    assert r.returncode == 0, r.stdout + r.stderr
