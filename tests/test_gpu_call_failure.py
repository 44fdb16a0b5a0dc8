"""A HIP call that fails in the middle of a solve: FMM_EDEVICE, never a result
decided by a header that was not copied, and the next solve as before.

Every event record, event wait and asynchronous copy of a solve is refused in
turn, on each route of a solve, in a process in which these calls pass through a
small library."""
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
static int at = -1, seen;
void refuse(int k) { at = k; seen = 0; }
int calls(void) { return seen; }
static void *real(const char *name) {
  void *h = dlopen("libamdhip64.so.7", RTLD_LAZY | RTLD_NOLOAD);
  return dlsym(h ? h : RTLD_NEXT, name);
}
#define ERROR 1  /* hipErrorInvalidValue */
int hipEventRecord(void *e, void *s) {
  static int (*f)(void *, void *);
  if (!f) f = (int (*)(void *, void *))real("hipEventRecord");
  return seen++ == at ? ERROR : f(e, s);
}
int hipStreamWaitEvent(void *s, void *e, unsigned flags) {
  static int (*f)(void *, void *, unsigned);
  if (!f) f = (int (*)(void *, void *, unsigned))real("hipStreamWaitEvent");
  return seen++ == at ? ERROR : f(s, e, flags);
}
int hipMemcpyAsync(void *d, const void *p, size_t n, int kind, void *s) {
  static int (*f)(void *, const void *, size_t, int, void *);
  if (!f) f = (int (*)(void *, const void *, size_t, int, void *))real("hipMemcpyAsync");
  return seen++ == at ? ERROR : f(d, p, n, kind, s);
}
"""

CHILD = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
shim.refuse(-1)
import torch
import paper_1712_10116_amd.fmm as F
from paper_1712_10116_amd import workloads as W
n, predict = int(sys.argv[2]), sys.argv[3] == "True"
pos, _, m = W.plummer(n, seed=77)
tp, tm = torch.from_numpy(pos).cuda(), torch.from_numpy(m).cuda()
out = [torch.zeros(3, n, dtype=torch.float64, device="cuda"),
       torch.zeros(n, dtype=torch.float64, device="cuda")]
s = F.Solver(n, p_max=4, leaf_size=16, kernel=0, precision=0)
s.set_level_prediction(predict)

def solve():
    s.forces(tp, tm, eps=0.01, theta=0.5, p=4, acc=out[0], pot=out[1])

for _ in range(3):
    solve()
ref = [x.clone() for x in out]
torch.cuda.synchronize()
k = 0
while True:
    shim.refuse(k)
    try:
        solve()
        made, refused = shim.calls(), False
    except F.FMMError as e:
        assert e.status == F.FMM_EDEVICE, (k, e)
        made, refused = shim.calls(), True
    shim.refuse(-1)
    assert refused == (k < made), (k, made)
    for x in out:
        x.zero_()
    solve()
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(out, ref)), k
    if not refused:
        break
    k += 1
print("refused", k, "calls in turn")
assert k >= 6
"""


@pytest.mark.parametrize("n,predict", [(900, False), (5000, False), (30000, False), (30000, True)])
def test_failed_call_is_reported(tmp_path, n, predict):
    src, so = tmp_path / "shim.c", str(tmp_path / "shim.so")
    src.write_text(SHIM)
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", str(src), "-o", so, "-ldl"], check=True)
    r = subprocess.run([sys.executable, "-u", "-c", CHILD, so, str(n), str(predict)], cwd=ROOT,
                       capture_output=True, text=True, timeout=100)
    print(r.stdout)
    assert r.returncode == 0 and "refused" in r.stdout, r.stdout[-2000:] + r.stderr[-3000:]
