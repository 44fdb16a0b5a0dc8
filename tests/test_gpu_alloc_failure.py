"""A workspace that cannot grow: the call reports FMM_ENOMEM (or does without),
and the context is as usable as before it.

Every device allocation that a solve makes to grow the context is made to fail
in turn, alone or together with the one that would restore the former size.  The
solves run in a process of their own, in which hipMalloc passes through a small
library that refuses the calls it is told to."""
import os
import shutil
import subprocess
import sys

import pytest

from conftest import ROOT, gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU"),
              pytest.mark.skipif(shutil.which("gcc") is None, reason="needs gcc")]

SHIM = r"""
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stddef.h>
static int first, count, seen;
void refuse(int k, int n) { first = k; count = n; seen = 0; }
int calls(void) { return seen; }
int hipMalloc(void **p, size_t n) {
  static int (*real)(void **, size_t);
  if (!real) {
    void *h = dlopen("libamdhip64.so.7", RTLD_LAZY | RTLD_NOLOAD);
    real = (int (*)(void **, size_t))dlsym(h ? h : RTLD_NEXT, "hipMalloc");
  }
  const int at = seen++;
  if (at >= first && at < first + count) return real(p, (size_t)1 << 60);  /* out of memory */
  return real(p, n);
}
"""

CHILD = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
shim.refuse(0, 0)
import numpy as np, torch
import paper_1712_10116_amd.fmm as F
from paper_1712_10116_amd import workloads as W
eps, theta, leaf = float(sys.argv[2]), float(sys.argv[3]), int(sys.argv[4])
count, call = int(sys.argv[5]), sys.argv[6]
n = 6000
pos, _, m = W.uniform_sphere(n, seed=34)
dev = [dict(pos=torch.from_numpy(pos[:, k:].copy()).cuda(), mass=torch.from_numpy(m[k:].copy()).cuda())
       for k in [0] + 1500 * [n - 1] + 700 * [n]]
prm = dict(eps=eps, theta=theta, p=4)

def solve(s):
    if call == "grad":
        return s.forces_grad(dev[0]["pos"], dev[0]["mass"], **prm)
    if call == "batch":
        return [x for o in s.forces_batched(dev, **prm)[:100] for x in o]
    return s.forces(dev[0]["pos"], dev[0]["mass"], **prm)

def solver():
    return F.Solver(n + 2000, p_max=4, leaf_size=leaf, kernel=0, precision=0)

s = solver()
ref = [x.clone() for x in solve(s)]
torch.cuda.synchronize()
del s
failed = k = 0
while True:
    s = solver()
    shim.refuse(k, count)
    try:
        out = solve(s)
        torch.cuda.synchronize()
        made = shim.calls()
    except F.FMMError as e:
        assert e.status == F.FMM_ENOMEM, (k, e.status, e)
        made = shim.calls()
        failed += 1
        shim.refuse(0, 0)
        out = solve(s)
        torch.cuda.synchronize()
    shim.refuse(0, 0)
    for again in range(2):
        for a, b in zip(out, ref):
            assert (a - b).abs().max() <= 1e-12 * b.abs().max(), (k, again)
        out = solve(s)
    print("refused", k, "of", made, "failed", failed, flush=True)
    s.close()
    if k >= made:
        break
    k += 1
assert k > 0
print("done", k, failed)
"""


@pytest.mark.parametrize("count", [1, 2])
@pytest.mark.parametrize("call,eps,theta,leaf", [
    ("forces", 1.0, 0.5, 4),    # every pair near: P2P and open lists, items, partial rows
    ("forces", 0.001, 0.25, 8),  # long far lists
    ("grad", 1.0, 0.5, 16),     # and the gradient's staging
    ("batch", 0.01, 0.5, 64),   # the request table, and cells: more systems than them
])
def test_context_survives_failed_growth(tmp_path, call, eps, theta, leaf, count):
    src, so = tmp_path / "shim.c", str(tmp_path / "shim.so")
    src.write_text(SHIM)
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", str(src), "-o", so, "-ldl"], check=True)
    r = subprocess.run([sys.executable, "-u", "-c", CHILD, so, str(eps), str(theta), str(leaf),
                        str(count), call], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-3000:]
    print(r.stdout)
    assert "done" in r.stdout
