"""Host-side sizing rules of the HIP library, compiled for the CPU from its headers.

* rows of the cells' expansions start on 16 bytes at every maximum degree that a
  context accepts;
* a buffer that cannot grow has its former size, or none: never a capacity
  without memory behind it;
* the shares that a leaf's near list is cut into are bounded, and so is the
  memory of their partial sums;
* the walk's form for a tree not yet built follows its size, not the last tree's;
* the merge sort is taken where it measured faster than the radix sort, with
  merges enough for the largest system wherever it starts in a tile;
* grids that grow with the tree stay below 2^32 threads;
* queued kernels heed no overflow bit that a kernel beside them may set."""
import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1712_10116_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

pytestmark = pytest.mark.skipif(shutil.which(HIPCC) is None, reason="needs hipcc")


def _run(tmp_path, body, before=""):
    src = tmp_path / "rules.hip"
    src.write_text('#include "context.h"\n#include <stdio.h>\n%s\nint main() {\n%s\n}\n'
                   % (before, body))
    exe = str(tmp_path / "rules")
    subprocess.run([HIPCC, "-std=c++17", "-O0", "--cuda-host-only", "-Wno-unused-value",
                    "-Wno-unused-result", "-I", CSRC, str(src), "-o", exe], check=True,
                   capture_output=True)
    return subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split()


def test_rows_start_on_16_bytes(tmp_path):
    out = _run(tmp_path, 'for (int p = 1; p <= 8; ++p) printf("%d %d ", coeff_row(p), folded_row(p));')
    for p in range(1, 9):
        coeffs, folded = int(out[2 * p - 2]), int(out[2 * p - 1])
        for row, values in ((coeffs, (p + 1) * (p + 2) * (p + 3) // 6), (folded, (p + 1) ** 2)):
            assert row % 2 == 0 and values <= row <= values + 1


ALLOCATOR = r"""
#include <stdlib.h>
#include <algorithm>
static int refused, cleared;  // calls still to refuse; errors taken from the runtime
extern "C" hipError_t hipMalloc(void **p, size_t n) {
  if (refused > 0) { --refused; return hipErrorOutOfMemory; }
  *p = malloc(n);
  return hipSuccess;
}
extern "C" hipError_t hipFree(void *p) { free(p); return hipSuccess; }
extern "C" hipError_t hipGetLastError(void) { ++cleared; return hipSuccess; }
void fmm_dfree(fmm_ctx *c, void *p) {
  if (!p) return;
  c->allocs.erase(std::find(c->allocs.begin(), c->allocs.end(), p));
  (void)hipFree(p);
}
"""


def test_failed_growth_leaves_no_capacity_without_memory(tmp_path):
    out = _run(tmp_path, """
  fmm_ctx c{};
  int32_t *p = nullptr;
  int64_t cap = 0;
  for (int k = 0; k < 3; ++k) {
    fmm_regrow(&c, &p, &cap, 100);
    refused = k;
    cleared = 0;
    const bool ok = fmm_regrow(&c, &p, &cap, 200);
    refused = 0;
    printf("%d %d %d %d %d ", ok, (int)cap, p != nullptr, (int)c.allocs.size(), cleared);
  }
  printf("%d %d", fmm_regrow(&c, &p, &cap, 50), (int)cap);  // and grows again from nothing
""", ALLOCATOR)
    assert [int(x) for x in out] == [1, 200, 1, 1, 0, 0, 100, 1, 1, 1, 0, 0, 0, 0, 2, 1, 50]


def test_shares_are_bounded(tmp_path):
    ns = [1, 1024, 1025, 32768, 131072, 262144, 262145, 524288, 524289, 1 << 20, (1 << 20) + 1,
          1 << 24, 1 << 30]
    cnts = [0, 1, 64, 65, 256, 257, 8192, 8193, 8449, 32768, 32769, 1 << 20, (1 << 31) - 64]
    out = [int(x) for x in _run(tmp_path, """
  const int ns[] = {%s}, cnts[] = {%s};
  for (int n : ns) {
    const int most = p2p_share_max(n);
    printf("%%d ", most);
    for (int c : cnts) printf("%%d ", p2p_share_chunks(c, most, 4));
  }
""" % (",".join(map(str, ns)), ",".join(map(str, cnts))))]
    for n in ns:
        most, out = out[0], out[1:]
        assert 32 <= most <= 128 and (most == 128 or n * most <= 2 ** 25 or most == 32)
        assert n * most <= max(2 ** 25, 32 * n)
        for c in cnts:
            per, out = out[0], out[1:]
            assert per >= 4 and -(-c // (64 * per)) <= most
            assert per == 4 or -(-c // (64 * (per - 1))) > most  # no longer than need be


def test_kernels_heed_final_overflow_bits(tmp_path):
    src = os.path.join(CSRC, "eval.hip")
    out = _run(tmp_path, """
  printf("%d %d %d %d %d", OVF_BUILD, OVF_WALK, OVF_ANY, OVF_ITEMS,
         OVF_M2L | OVF_P2P | OVF_OPEN | OVF_STACK | OVF_PATH);
""")
    build, walk, every, plan_sets, walk_sets = (int(x) for x in out)
    assert build & (walk_sets | plan_sets) == 0 and walk & plan_sets == 0
    assert build | walk_sets == walk and walk | plan_sets == every
    heeds = {}  # kernel -> mask, from the kernels that look at the bits
    with open(src) as a, open(os.path.join(CSRC, "m2l_staged.h")) as b:
        for part in (a.read() + b.read()).split("__global__")[1:]:
            name = re.search(r"\b(k_\w+)\(", part).group(1)
            for mask in re.findall(r"(?:tree_incomplete|node_count|level_range)<(OVF_\w+)>\(t", part):
                heeds.setdefault(name, set()).add(mask)
    beside_walk = {"k_p2m", "k_m2m", "k_m2m_small"}
    beside_plan = {"k_m2l", "k_m2l_staged", "k_l2l", "k_l2l_small"}
    assert heeds == dict({k: {"OVF_BUILD"} for k in beside_walk},
                         **{k: {"OVF_WALK"} for k in beside_plan},
                         **{k: {"OVF_ANY"} for k in ("k_p2p", "k_l2p")})


def test_walk_form_follows_the_size_of_the_tree_to_come(tmp_path):
    cases = [  # split cells and particles of the last tree, particles of the next
        (0, 0, 1000, 0), (0, 10, 10, 1), (0, 10, 1 << 20, 0), (100, 30000, 30000, 1),
        (100, 30000, 400000, 1), (100, 30000, 1 << 20, 0), (1598, 300007, 300007, 1),
        (1600, 300007, 300007, 0), (2769, 1 << 20, 1 << 20, 0), (2769, 1 << 20, 300000, 1),
        (1 << 27, 1 << 30, 1 << 30, 0), (0, 1, 1 << 30, 0)]
    out = _run(tmp_path, "".join('printf("%%d ", walk_paths_expected(%dll, %dll, %dll));'
                                 % c[:3] for c in cases))
    assert [int(x) for x in out] == [c[3] for c in cases]


def test_near_field_grid_stays_launchable(tmp_path):
    trees = [(1, 0), (1000, 90), (131072, 17408), (131073, 17408), (1 << 24, 4000000),
             (1 << 25, 1 << 25), (1 << 28, (1 << 28) - 1), (100000, (1 << 28) - 1), (100000, 68350),
             (100000, 4096), (100000, 4097), (100000, 32769), (1024, 1), (100000, 22)]
    out = _run(tmp_path, "".join('printf("%%d ", p2p_grid_items(%d, %d));' % t for t in trees)
               + 'printf("%d", GRID_WAVES);')
    for (n, cells), waves in zip(trees, map(int, out)):
        assert 1 <= waves and waves * 64 < 2 ** 32
        most = int(out[-1])
        assert waves == most or waves >= n // 64 + cells  # every 64 sinks of uncut leaves
        assert waves <= max(1, min(most, max((8 if n <= 131072 else 2) * cells, n // 64 + cells)))
        if n <= 131072:  # not many without an item
            assert waves <= max(32768, n // 64 + cells)


def test_sort_rule(tmp_path):
    # (largest system, systems, us of the radix sort, us of the merge sort)
    measured = [
        (32768, 1, 131.9, 57.9), (131072, 1, 139.5, 71.8), (262144, 1, 151.4, 105.6),
        (300007, 1, 152.9, 145.6), (393216, 1, 160.6, 159.6), (430000, 1, 162.2, 185.0),
        (524288, 1, 169.2, 218.8), (1 << 20, 1, 197.8, 373.7), (3000, 43, 162.0, 47.7),
        (131072, 4, 192.8, 143.0), (131072, 8, 223.7, 232.7), (100003, 5, 191.3, 139.8),
        (100003, 10, 223.5, 231.5), (200003, 2, 184.2, 148.8), (200003, 5, 221.6, 283.5),
        (262144, 2, 190.7, 179.3), (16384, 64, 242.8, 186.6), (16384, 1024, 3490.9, 2647.4),
        (262144, 4, 222.5, 300.9),
        (300007, 3, 218.5, 308.7), (65536, 64, 682.6, 853.8), (10007, 1676, 3168.9, 2505.2),
        (3000, 5592, 3199.7, 1821.9), (524288, 32, 2779.9, 5288.3)]
    edges = [(n, n, 1) for n in (1, 1024, 1025, 16384, 16385, 262144, 262145, 393216, 393217)]
    edges += [(917504, 100000, 10), (917505, 100000, 10), (589824, 200000, 3), (589825, 200000, 3),
              (2000, 2, 1000), (1 << 30, 16384, 70000), (1 << 30, 16385, 70000)]
    calls = [(n * k, n, k) for n, k, _, _ in measured] + edges
    out = [int(x) for x in _run(tmp_path, "".join(
        'printf("%%d ", sort_merges(%d, %d, %d));' % c for c in calls))]
    for (n, k, radix, merge), m in zip(measured, out):
        assert (m >= 0) == (merge < radix), (n, k, m)
    for (n, n_max, k), m in zip(calls, out):
        reach = n if k == 1 else n_max + 1023
        assert m < 0 or 1024 * 16 ** m >= reach > (1024 * 16 ** (m - 1) if m else 0)
    assert out[len(measured):] == [0, 0, 1, 1, 2, 2, 3, 3, -1, 2, -1, 2, -1, 1, 2, -1]


def test_small_leaves_share_whole_chunks(tmp_path):
    cases = [(n, w, leaf) for n in (1024, 1025, 32768, 32769, 131073, 524288, 524289)
             for w in (256, 384) for leaf in (1, 2, 4, 8, 16, 32, 64, 128, 4096)]
    out = [int(x) for x in _run(tmp_path, "".join(
        'printf("%%d %%d ", p2p_share_windows(%d), p2p_leaf_chunks(p2p_share_windows(%d), %d, %d));'
        % (n, n, w, leaf) for n, w, leaf in cases))]
    for k, (n, window, leaf) in enumerate(cases):
        g, chunks = out[2 * k], out[2 * k + 1]
        if g == 0:
            assert (n <= 1024 or n > 524288) and chunks == 4
        elif chunks > 1:  # a share holds no more than its windows where leaves are half full
            assert 32 * leaf * chunks <= g * window < 32 * leaf * (chunks + 1)
        else:  # a chunk of half full leaves holds more than half a share
            assert 64 * leaf > g * window
