// Host side of the C ABI declared in include/fmm355.h.
//
// A context owns one device workspace sized from max_n at creation.  Every
// call is queued on the context's stream; a build waits to read the tree's
// header, once where tree, walk and evaluation are queued without its sizes, for
// the tree's and for the lists' sizes otherwise (and again after a buffer that
// turned out too small has been regrown).
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <cmath>
#include <new>
#include <type_traits>
#include <vector>

#include "../../include/fmm355.h"
#include "common.h"
#include "context.h"
#include "hhs_kernels.h"

static PhaseTimer *timer_of(fmm_ctx *c) { return c->timer.on ? &c->timer : nullptr; }

fmm_status fmm_fail(fmm_ctx *c, fmm_status st, const char *fmt, ...) {
  if (c) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(c->err, sizeof(c->err), fmt, ap);
    va_end(ap);
  }
  return st;
}

#define HIPCHK(c, call)                                                                       \
  do {                                                                                        \
    hipError_t e_ = (call);                                                                   \
    if (e_ != hipSuccess)                                                                     \
      return fail((c), FMM_EDEVICE, "%s failed: %s", #call, hipGetErrorString(e_));          \
  } while (0)

#define fail fmm_fail
#define dalloc fmm_dalloc
#define dfree fmm_dfree

void fmm_dfree(fmm_ctx *c, void *p) {
  if (!p) return;
  auto it = std::find(c->allocs.begin(), c->allocs.end(), p);
  if (it != c->allocs.end()) c->allocs.erase(it);
  (void)hipFree(p);
}

// Places several arrays in one device allocation: each costs the driver 5 to 10 us
// whatever its size, and a context has some forty.  place() is called with a
// Placer twice, for the size (a null base) and for the addresses.
struct Placer {
  char *base = nullptr;
  size_t at = 0;
  template <typename T>
  void operator()(T *&p, size_t count, size_t bytes = 0) {  // bytes: of an element, if T is void
    if constexpr (!std::is_void<T>::value) bytes = sizeof(T);
    p = (T *)(base + at);
    at += (count * bytes + 255) & ~(size_t)255;
  }
};

template <typename F>
static bool dalloc_block(fmm_ctx *c, F place) {
  Placer size, block;
  place(size);
  if (!dalloc(c, &block.base, (int64_t)size.at)) return false;
  place(block);
  return true;
}

// node-sized arrays (nbeg first: free_nodes)
static bool alloc_nodes(fmm_ctx *c, int64_t cap) {
  DevTree &t = c->t;
  if (cap >= ((int64_t)1 << 28)) return false;  // node ids carry a 3-bit tag in the walk
  const size_t n = (size_t)cap;
  const size_t real = c->prm.precision == FMM_PREC_MIXED ? sizeof(float) : sizeof(double);
  const bool ok = dalloc_block(c, [&](Placer &at) {
    at(t.nbeg, n), at(t.nend, n), at(t.nlev, n), at(t.nparent, n), at(t.nchild0, n);
    at(t.nnchild, n), at(t.ngeo, n), at(t.bounds, 8 * n), at(t.m2l_off, n), at(t.m2l_cnt, n);
    at(t.p2p_off, n), at(t.p2p_cnt, n), at(t.open_off, n), at(t.open_cnt, n), at(t.nreq, n);
    at(t.ninfo, n), at(t.nshare, n), at(t.part_off, n);
    at(t.M, n * t.kmax, real), at(t.L, n * t.kmax, real), at(t.Mh, n * t.khmax, real);
  });
  t.cap_nodes = ok ? cap : 0;
  return ok;
}

static void free_nodes(fmm_ctx *c) {
  dfree(c, c->t.nbeg);
  c->t.nbeg = nullptr;
  c->t.cap_nodes = 0;
}

// entries of a list buffer, at most: offsets into it are int32
static const int64_t MAX_LIST = INT32_MAX;

// capacities of a context that has grown nothing
static int64_t first_nodes(const fmm_ctx *c) { return 8 * c->max_n / c->prm.leaf_size + 1024; }
static int64_t first_list(int which, int64_t cap_nodes) {
  return std::min<int64_t>((which == OVF_M2L ? 96 : which == OVF_P2P ? 32 : 16) * cap_nodes, MAX_LIST);
}

// Request-sized arrays (regrown when a batch holds more requests).  The
// request table, its particle offsets and its block offsets share one device
// region, mirrored by pinned host staging slots, so a table is sent in one copy.
static size_t req_region_bytes(int cap) {
  return sizeof(DevReq) * (size_t)cap + 2 * sizeof(int32_t) * (size_t)(cap + 1);
}

static bool alloc_reqs(fmm_ctx *c, int cap) {
  DevTree &t = c->t;
  for (int k = 0; k < fmm_ctx::UP_SLOTS; ++k)
    if (c->up_ev_set[k]) (void)hipEventSynchronize(c->up_ev[k]);
  void *ptrs[] = {t.reqs, t.box, t.bbox_part};
  for (void *p : ptrs) dfree(c, p);
  t.reqs = nullptr;
  t.box = nullptr;
  t.bbox_part = nullptr;
  t.cap_req = 0;  // until all of it is there
  const size_t bytes = req_region_bytes(cap);
  char *region = nullptr;
  if (!dalloc(c, &region, (int64_t)bytes)) return false;
  t.reqs = (DevReq *)region;
  if (!dalloc(c, &t.box, cap) ||
      !dalloc(c, &t.bbox_part, (int64_t)cap * FMM_BBOX_BLOCKS * FMM_BBOX_COLS))
    return false;
  t.req_off = (int32_t *)(region + sizeof(DevReq) * (size_t)cap);
  t.blk_off = t.req_off + cap + 1;
  for (int k = 0; k < fmm_ctx::UP_SLOTS; ++k) {
    if (c->up_pin[k]) (void)hipHostFree(c->up_pin[k]);
    c->up_pin[k] = nullptr;
    if (hipHostMalloc((void **)&c->up_pin[k], bytes) != hipSuccess) {
      (void)hipGetLastError();
      return false;
    }
  }
  t.cap_req = cap;
  c->up_bytes = bytes;
  c->up_valid = false;
  return true;
}

extern "C" fmm_status fmm_create(const fmm_params *prm, int64_t max_n, void *stream,
                                 fmm_ctx **out) {
  if (!prm || !out) return FMM_EINVAL;
  *out = nullptr;
  if (max_n < 1 || max_n > (int64_t)1 << 30) return FMM_EINVAL;
  if (prm->p_max < 1 || prm->p_max > 8 || prm->leaf_size < 1 || prm->leaf_size > 4096 ||
      (prm->kernel != FMM_KERNEL_WENDLAND_C2 && prm->kernel != FMM_KERNEL_PLUMMER) ||
      (prm->precision != FMM_PREC_FP64 && prm->precision != FMM_PREC_MIXED))
    return FMM_EINVAL;
  fmm_ctx *c = new (std::nothrow) fmm_ctx();
  if (!c) return FMM_ENOMEM;
  c->prm = *prm;
  c->max_n = max_n;
  c->small_max = SMALL_N;
  c->predict_levels = false;
  c->lvl_hist_n = 0;
  c->stream = (hipStream_t)stream;
  if (hipGetDevice(&c->device) != hipSuccess) {
    delete c;
    return FMM_EDEVICE;
  }
  DevTree &t = c->t;
  memset(&t, 0, sizeof(t));
  bool pins = hipHostMalloc((void **)&c->pin_hdr, sizeof(Header)) == hipSuccess &&
              hipStreamCreateWithFlags(&c->side, hipStreamNonBlocking) == hipSuccess &&
              hipEventCreateWithFlags(&c->fork, hipEventDisableTiming) == hipSuccess &&
              hipEventCreateWithFlags(&c->join, hipEventDisableTiming) == hipSuccess &&
              hipEventCreateWithFlags(&c->hdr_ev, hipEventDisableTiming) == hipSuccess &&
              hipEventCreateWithFlags(&c->up_done, hipEventDisableTiming) == hipSuccess;
  for (int k = 0; pins && k < fmm_ctx::UP_SLOTS; ++k)
    pins = hipEventCreateWithFlags(&c->up_ev[k], hipEventDisableTiming) == hipSuccess;
  if (!pins) {
    fmm_destroy(c);
    return FMM_ENOMEM;
  }
  t.kmax = coeff_row(prm->p_max);
  t.khmax = folded_row(prm->p_max);
  t.cap_n = max_n;
  int64_t n = max_n;
  int64_t cap_nodes = first_nodes(c);
  // radix histograms: one column per tile; also the cells per level and block
  // of the tree build
  const int64_t sort_tiles = (n + SORT_TILE - 1) / SORT_TILE;
  const int64_t sort_hist_n = std::max<int64_t>(256 * sort_tiles, FMM_MAXLEVEL * ((n + 1023) / 1024)) + 256;
  bool ok = dalloc_block(c, [&](Placer &at) {
    at(t.key, n), at(t.key2, n), at(t.slot, n), at(t.slot2, n), at(t.sx, n), at(t.sy, n);
    at(t.sz, n), at(t.sm, n), at(t.sm32, n), at(t.leaf_of, n), at(t.near, 4 * n), at(t.pak, n);
    at(t.scan_part, FMM_SCAN_BLOCKS), at(t.slot_req, n), at(t.sort_hist, sort_hist_n);
    at(t.sort_dtot, 256), at(t.scan_blk, n / 1024 + 64), at(t.hdr, 1);
  }) && alloc_reqs(c, 16) && alloc_nodes(c, cap_nodes);
  if (ok) {
    t.cap_m2l = first_list(OVF_M2L, cap_nodes);
    t.cap_p2p = first_list(OVF_P2P, cap_nodes);
    t.cap_open = first_list(OVF_OPEN, cap_nodes);
    // near-field items and partial rows: small systems are cut fine (up to a
    // share per window), large ones only at long lists.  Uncut, a leaf has an
    // item per 64 particles begun, which always fit.
    t.p2p_src_window = p2p_window_sources(prm->precision == FMM_PREC_MIXED);
    t.cap_items = 2 * cap_nodes + std::max(std::min<int64_t>(8 * n, 65536), n / 64);
    t.cap_part = std::min<int64_t>(4 * n, n / 4 + (4 << 20)) + std::min<int64_t>(16 * n, 65536);
    ok = dalloc(c, &t.items, t.cap_items) && dalloc(c, &t.part, t.cap_part) &&
         dalloc(c, &t.m2l_src, t.cap_m2l) && dalloc(c, &t.p2p_src, t.cap_p2p) &&
         dalloc(c, &t.open_buf0, t.cap_open) && dalloc(c, &t.open_buf1, t.cap_open);
  }
  ok = ok && dalloc(c, &c->inv_part, FMM_INV_BLOCKS * 12);
  if (!ok) {
    fmm_destroy(c);
    return FMM_ENOMEM;
  }
  if (hipMemsetAsync(t.hdr, 0, sizeof(Header), c->stream) != hipSuccess ||
      hipStreamSynchronize(c->stream) != hipSuccess) {
    fmm_destroy(c);
    return FMM_EDEVICE;
  }
  *out = c;
  return FMM_OK;
}

extern "C" fmm_status fmm_destroy(fmm_ctx *c) {
  if (!c) return FMM_EINVAL;
  (void)hipStreamSynchronize(c->stream);
  if (c->timer.ready)
    for (int i = 0; i < PhaseTimer::CAP; ++i) {
      (void)hipEventDestroy(c->timer.a[i]);
      (void)hipEventDestroy(c->timer.b[i]);
    }
  if (c->own_run) hhs_run_destroy(c->own_run);
  for (void *p : c->allocs) (void)hipFree(p);
  for (int k = 0; k < fmm_ctx::UP_SLOTS; ++k) {
    if (c->up_pin[k]) (void)hipHostFree(c->up_pin[k]);
    if (c->up_ev[k]) (void)hipEventDestroy(c->up_ev[k]);
  }
  if (c->pin_hdr) (void)hipHostFree(c->pin_hdr);
  if (c->pin_split) (void)hipHostFree(c->pin_split);
  if (c->side) {
    (void)hipStreamSynchronize(c->side);
    (void)hipStreamDestroy(c->side);
  }
  if (c->fork) (void)hipEventDestroy(c->fork);
  if (c->join) (void)hipEventDestroy(c->join);
  if (c->hdr_ev) (void)hipEventDestroy(c->hdr_ev);
  if (c->up_done) (void)hipEventDestroy(c->up_done);
  delete c;
  return FMM_OK;
}

extern "C" const char *fmm_last_error(const fmm_ctx *c) { return c ? c->err : "null context"; }

extern "C" fmm_status fmm_set_small_path(fmm_ctx *c, int enable) {
  if (!c || enable < 0 || enable > 2) return FMM_EINVAL;
  c->small_max = enable == 0 ? -1 : SMALL_N;
  return FMM_OK;
}

extern "C" fmm_status fmm_set_level_prediction(fmm_ctx *c, int enable) {
  if (!c) return FMM_EINVAL;
  c->predict_levels = enable != 0;
  c->lvl_hist_n = 0;
  return FMM_OK;
}

// split levels of the recent builds (0: none recorded)
static int predicted_levels(const fmm_ctx *c) {
  int m = 0;
  for (int i = 0; i < std::min(c->lvl_hist_n, fmm_ctx::LEVEL_HIST); ++i) m = std::max(m, c->lvl_hist[i]);
  return m;
}

static void record_levels(fmm_ctx *c, int levels) {
  c->lvl_hist[c->lvl_hist_n % fmm_ctx::LEVEL_HIST] = levels;
  c->lvl_hist_n++;
}

static fmm_status check_requests(fmm_ctx *c, int n_req, const fmm_request *reqs, bool eval,
                                 int64_t *n_all) {
  if (!c) return FMM_EINVAL;
  if (n_req < 1 || !reqs) return fail(c, FMM_EINVAL, "need at least one request");
  int64_t n = 0;
  for (int r = 0; r < n_req; ++r) {
    const fmm_request &q = reqs[r];
    if (q.n_active < 0 || q.n_total < 0 || q.n_total > (int64_t)INT32_MAX)
      return fail(c, FMM_EINVAL, "request %d: bad sizes", r);
    if (q.n_active > 0 && !q.active && q.n_total != q.n_active)
      return fail(c, FMM_EINVAL, "request %d: n_total=%lld inconsistent with n_active=%lld", r,
                  (long long)q.n_total, (long long)q.n_active);
    if (q.n_active > 0 && !q.pos) return fail(c, FMM_EINVAL, "request %d: pos is NULL", r);
    if (eval && q.n_active > 0 && q.mass && (!q.acc || !q.pot))
      return fail(c, FMM_EINVAL, "request %d: NULL acc/pot", r);
    n += q.n_active;
  }
  if (n > c->max_n)
    return fail(c, FMM_EINVAL, "%lld active particles exceed max_n=%lld", (long long)n,
                (long long)c->max_n);
  *n_all = n;
  return FMM_OK;
}

// Stage the request table in the next pinned slot and send it in one copy,
// unless it equals the table last sent.  Blocks per request for the box
// reduction: ceil(n / 2048), at least 1 and at most FMM_BBOX_BLOCKS.
static fmm_status upload_requests(fmm_ctx *c, int n_req, const fmm_request *reqs, int *n_blk) {
  DevTree &t = c->t;
  if (n_req > t.cap_req && !alloc_reqs(c, std::max(n_req, 2 * t.cap_req)))
    return fail(c, FMM_ENOMEM, "request table for %d requests", n_req);
  const int k = c->up_next;
  if (c->up_ev_set[k]) HIPCHK(c, hipEventSynchronize(c->up_ev[k]));
  char *stage = c->up_pin[k];
  memset(stage, 0, c->up_bytes);
  DevReq *hr = (DevReq *)stage;
  int32_t *ho = (int32_t *)(stage + sizeof(DevReq) * (size_t)t.cap_req);
  int32_t *hb = ho + t.cap_req + 1;
  int off = 0, blk = 0;
  for (int r = 0; r < n_req; ++r) {
    const fmm_request &q = reqs[r];
    hr[r].pos = q.pos;
    hr[r].active = q.active;
    hr[r].mass = q.mass;
    hr[r].acc = q.acc;
    hr[r].pot = q.pot;
    hr[r].sinks = q.sinks;
    hr[r].n_total = q.n_total;
    hr[r].off = off;
    hr[r].n = (int32_t)q.n_active;
    ho[r] = off;
    hb[r] = blk;
    off += (int)q.n_active;
    blk += (int)std::min<int64_t>(FMM_BBOX_BLOCKS, std::max<int64_t>(1, (q.n_active + 2047) / 2048));
  }
  ho[n_req] = off;
  hb[n_req] = blk;
  t.n_req = n_req;
  if (!(c->up_valid && c->up_last.size() == c->up_bytes &&
        memcmp(c->up_last.data(), stage, c->up_bytes) == 0)) {
    HIPCHK(c, hipMemcpyAsync(t.reqs, stage, c->up_bytes, hipMemcpyHostToDevice, c->stream));
    HIPCHK(c, hipEventRecord(c->up_ev[k], c->stream));
    c->up_ev_set[k] = true;
    c->up_next = (k + 1) % fmm_ctx::UP_SLOTS;
    c->up_last.assign(stage, stage + c->up_bytes);
    c->up_valid = true;
  }
  if (n_blk) *n_blk = blk;
  return FMM_OK;
}

// header readback through pinned memory; waits for the stream
static fmm_status read_header(fmm_ctx *c) {
  HIPCHK(c, hipMemcpyAsync(c->pin_hdr, c->t.hdr, sizeof(Header), hipMemcpyDeviceToHost, c->stream));
  HIPCHK(c, hipStreamSynchronize(c->stream));
  memcpy(&c->hh, c->pin_hdr, sizeof(Header));
  return FMM_OK;
}

// Regrow the list buffer that overflowed.  A walk that overflows stops
// writing, so `need` (the entries it tried to place) can undercount what the
// whole walk needs: the capacity at least doubles each time (from the first
// one if an earlier growth failed and left none).
static fmm_status regrow_lists(fmm_ctx *c, int which, int64_t need) {
  DevTree &t = c->t;
  const int64_t old = which == OVF_M2L ? t.cap_m2l : which == OVF_P2P ? t.cap_p2p : t.cap_open;
  if (need > MAX_LIST || old == MAX_LIST)
    return fail(c, FMM_EOVERFLOW, "interaction lists of more than 2^31 - 1 entries");
  const int64_t cap = std::min(
      MAX_LIST, std::max(need + need / 4 + 1024, old > 0 ? 2 * old : first_list(which, t.cap_nodes)));
  if (which == OVF_M2L) {
    if (!fmm_regrow(c, &t.m2l_src, &t.cap_m2l, cap)) return fail(c, FMM_ENOMEM, "M2L list regrow failed");
  } else if (which == OVF_P2P) {
    if (!fmm_regrow(c, &t.p2p_src, &t.cap_p2p, cap)) return fail(c, FMM_ENOMEM, "P2P list regrow failed");
  } else {
    int64_t cap0 = old, cap1 = old;
    const bool ok = fmm_regrow(c, &t.open_buf0, &cap0, cap) && fmm_regrow(c, &t.open_buf1, &cap1, cap);
    t.cap_open = std::min(cap0, cap1);
    if (!ok) return fail(c, FMM_ENOMEM, "open list regrow failed");
  }
  return FMM_OK;
}

// Regrow the near-field items and partial rows to what a plan counted (every
// workgroup counts its cells, also when they do not fit).  Without the memory
// for them this context cuts no list any more: that takes no rows, and the items
// that it has from the start.  Sums then differ in rounding only.
static fmm_status regrow_items(fmm_ctx *c, int64_t items, int64_t rows) {
  DevTree &t = c->t;
  const bool ok =
      (items <= t.cap_items || fmm_regrow(c, &t.items, &t.cap_items, items + items / 4)) &&
      (rows <= t.cap_part ||
       (rows <= INT32_MAX && fmm_regrow(c, &t.part, &t.cap_part,
                                        std::min<int64_t>(rows + rows / 4, INT32_MAX))));
  if (!ok && t.uncut) return fail(c, FMM_ENOMEM, "P2P item regrow failed");
  if (!ok) t.uncut = 1;
  return FMM_OK;
}

static void set_eval_args(fmm_ctx *c, EvalArgs &e, int64_t n_all, int p, double eps) {
  e.n = (int)n_all;
  e.p = p;
  e.kernel = c->prm.kernel;
  e.mixed = c->prm.precision == FMM_PREC_MIXED;
  e.eps = eps;
  e.tm = timer_of(c);
  e.side = c->side;
  e.fork = c->fork;
  e.join = c->join;
}

static void count_evaluation(fmm_ctx *c, int n_req, const fmm_request *reqs) {
  c->stat_calls++;
  for (int r = 0; r < n_req; ++r)
    if (reqs[r].mass) c->stat_parts += reqs[r].n_active;
}

// Build (and, with p_fused > 0, evaluate at order p_fused): when the
// predicted sequence runs, the evaluation is queued behind the walk before the
// host reads the tree header, with the tree's sizes taken on the device; if
// the header then shows that the prediction fell short or a workspace
// overflowed, the build is redone the classic way and *evaluated stays false
// (the caller evaluates again, overwriting whatever the queued kernels wrote).
static fmm_status build_impl(fmm_ctx *c, int n_req, const fmm_request *reqs, double eps,
                             double theta, int p_fused, bool *evaluated, bool *upward) {
  int64_t n_all = 0;
  fmm_status st = check_requests(c, n_req, reqs, p_fused > 0, &n_all);
  if (st != FMM_OK) return st;
  if (!(theta > 0.0) || !(eps >= 0.0) || !std::isfinite(theta) || !std::isfinite(eps))
    return fail(c, FMM_EINVAL, "need theta > 0 and eps >= 0");
  c->tree_valid = false;
  if (c->t.cap_nodes < 1 && !alloc_nodes(c, first_nodes(c)))  // an earlier growth failed
    return fail(c, FMM_ENOMEM, "no node workspace");
  int n_blk = 0;
  st = upload_requests(c, n_req, reqs, &n_blk);
  if (st != FMM_OK) return st;
  BuildArgs a = {};
  a.n = (int)n_all;
  for (int r = 0; r < n_req; ++r) a.n_max = std::max(a.n_max, (int)reqs[r].n_active);
  a.n_req = n_req;
  a.n_blk = n_blk;
  a.leaf_size = c->prm.leaf_size;
  a.eps = eps;
  a.theta = theta;
  a.tm = timer_of(c);
  auto finish = [&](int depth) {
    c->n_nodes = c->hh.lvl_start[FMM_NLEVELS];
    c->depth = depth;
    c->last = c->hh;
    c->tree_valid = true;
    c->b_reqs.assign(reqs, reqs + n_req);
    c->b_n = n_all;
    c->b_eps = eps;
    c->b_theta = theta;
    c->stat_builds++;
    return FMM_OK;
  };
  auto tree_depth = [&]() {
    int depth = 0;
    for (int l = 0; l < FMM_NLEVELS; ++l)
      if (c->hh.lvl_start[l + 1] > c->hh.lvl_start[l]) depth = l;
    return depth;
  };
  // The walk's path form does not take open lists of more than WALK_OPEN cells
  // (wide softening).  It is tried once a build, and after it failed the next
  // PATH_HOLD builds of systems of that size (within a quarter) or larger walk by
  // levels at once: else a build of such a system is queued, built and walked two
  // or three times over.
  bool paths_ok = c->path_hold <= 0 || a.n_max < c->path_hold_n;
  if (!paths_ok) --c->path_hold;
  auto heed_path = [&]() {
    if (!(c->hh.overflow & OVF_PATH)) return;
    paths_ok = false;
    c->path_hold = PATH_HOLD;
    c->path_hold_n = a.n_max - a.n_max / 4;
  };
  // an error found behind a queued evaluation (whose kernels then do nothing):
  // nothing reads the caller's arrays any more when it is returned
  auto fail_queued = [&](fmm_status e, const char *what) {
    (void)hipStreamSynchronize(c->stream);
    return fail(c, e, "%s", what);
  };
  // 0. small trees: everything is queued without reading a size back (the walk's
  // path form, M2M and L2L in one workgroup, sizes read on the device), with
  // one header readback at the end; anything that needs more room falls
  // through to the general path.  Batches of up to SMALL_N particles are built
  // by one workgroup.  A system has about 2 (uniform) to 5 (concentrated) cells
  // per leaf_size particles; the host's wait for the level sizes cost about
  // 25 us of a 12,526-particle solve.
  const bool direct = build_tree_direct_ok(a.leaf_size);
  const bool one_wg = n_all <= c->small_max;  // any leaf size: up to it, nothing is split
  if (one_wg || (direct && paths_ok && c->small_max >= 0 &&
                 n_all <= SMALL_TREE_LEAVES * (int64_t)a.leaf_size)) {
    if (one_wg) {
      HIPCHK(c, launch_build_small(c->t, a, c->stream));
    } else {
      HIPCHK(c, launch_sort(c->t, a, c->stream));
      HIPCHK(c, launch_build_tree_direct(c->t, a, FMM_MAXLEVEL, c->stream));
    }
    // no system is split: as many cells as systems.  A solve of 28 particles: 77 us
    // with the size read back, 102 queued as a tree of unknown size, 74 so
    const bool roots_only = a.n_max <= a.leaf_size;
    const int cells = (int)std::min<int64_t>(
        c->t.cap_nodes, roots_only ? n_req : 5 * (n_all / a.leaf_size) + 64);
    const bool fuse = p_fused > 0 && n_all > 0;
    EvalArgs e = {};
    if (fuse) {
      set_eval_args(c, e, n_all, p_fused, eps);
      e.dev = true;
      if (roots_only) {  // no M2M or L2L, and a walk too short for P2M to run beside
        e.n_nodes = n_req;
        e.exact = true;
      } else {
        e.n_nodes = cells;
        e.small_tree = true;
        HIPCHK(c, hipEventRecord(c->fork, c->stream));
        HIPCHK(c, hipStreamWaitEvent(c->side, c->fork, 0));
        HIPCHK(c, launch_upward(c->t, e, c->side));
        HIPCHK(c, hipEventRecord(c->up_done, c->side));
      }
    }
    // (with its own launch for the cursors a walk lets the upward pass start first:
    // 1,000 particles 126.7 -> 124.2 us)
    HIPCHK(c, launch_traverse_paths(c->t, a, cells, roots_only, c->stream));
    if (fuse) {
      e.upward_done = !roots_only;
      e.up_done = c->up_done;
      e.plan = &a;
      e.pin_hdr = c->pin_hdr;
      e.hdr_ev = c->hdr_ev;
      HIPCHK(c, launch_evaluate(c->t, e, c->stream));
      HIPCHK(c, hipEventSynchronize(c->hdr_ev));
      memcpy(&c->hh, c->pin_hdr, sizeof(Header));
    } else {
      HIPCHK(c, launch_p2p_plan(c->t, a, c->stream));
      st = read_header(c);
      if (st != FMM_OK) return st;
    }
    if (c->hh.nonfinite) return fail_queued(FMM_ENONFINITE, "non-finite input position");
    if (c->hh.overflow & OVF_STACK) return fail_queued(FMM_EOVERFLOW, "walk descent stack overflow");
    if (!(c->hh.overflow & OVF_ANY)) {
      // a tree of one workgroup says nothing about the depth of larger ones
      if (!one_wg) record_levels(c, std::min(FMM_MAXLEVEL, c->hh.max_prefix + 1));
      st = finish(tree_depth());
      if (st == FMM_OK && fuse) {
        count_evaluation(c, n_req, reqs);
        *evaluated = true;
      }
      return st;
    }
    heed_path();
  }
  // 1a. split levels predicted from recent builds: tree and walk queued behind
  // the sort, one readback.  The tree equals the one built below whenever the
  // prediction covers the split depth (levels past it split nothing); if it
  // does not, or a workspace overflowed, the classic sequence runs.
  const int pred = c->predict_levels ? predicted_levels(c) : 0;
  if (pred > 0) {
    int32_t prev[FMM_NLEVELS + 2];  // level starts of the last tree: grid estimates
    memcpy(prev, c->last.lvl_start, sizeof(prev));
    const int prev_nodes = c->n_nodes;
    // the evaluation's grids come from the last tree: only for a batch of
    // the same systems within a quarter of its size
    const bool fuse = p_fused > 0 && n_all > 0 && n_req == (int)c->b_reqs.size() &&
                      4 * n_all >= 3 * c->b_n && 4 * n_all <= 5 * c->b_n;
    HIPCHK(c, launch_sort(c->t, a, c->stream));
    if (build_tree_direct_ok(a.leaf_size))
      HIPCHK(c, launch_build_tree_direct(c->t, a, pred, c->stream));
    else
      HIPCHK(c, launch_build_tree(c->t, a, pred, c->stream));
    if (fuse) {  // mass gather, P2M and M2M on the second stream, beside the walk
      EvalArgs u = {};
      set_eval_args(c, u, n_all, p_fused, eps);
      u.n_nodes = std::max(prev_nodes, 1);
      u.lvl_start_host = prev;
      u.depth = pred;
      u.dev = true;
      HIPCHK(c, hipEventRecord(c->fork, c->stream));
      HIPCHK(c, hipStreamWaitEvent(c->side, c->fork, 0));
      HIPCHK(c, launch_upward(c->t, u, c->side));
      HIPCHK(c, hipEventRecord(c->up_done, c->side));
    }
    if (paths_ok && walk_paths_expected(prev_nodes - c->last.n_leaves, c->b_n, n_all)) {
      const int64_t cells = prev_nodes * n_all / c->b_n;
      HIPCHK(c, launch_traverse_paths(c->t, a, (int)std::min(c->t.cap_nodes, cells + cells / 4 + 64),
                                      false, c->stream));
    } else {
      HIPCHK(c, launch_traverse_dev(c->t, a, pred, c->stream));
    }
    if (!fuse) {
      HIPCHK(c, launch_p2p_plan(c->t, a, c->stream));
      HIPCHK(c, hipMemcpyAsync(c->pin_hdr, c->t.hdr, sizeof(Header), hipMemcpyDeviceToHost,
                               c->stream));
      HIPCHK(c, hipEventRecord(c->hdr_ev, c->stream));
    } else {
      EvalArgs e = {};
      set_eval_args(c, e, n_all, p_fused, eps);
      e.plan = &a;
      e.pin_hdr = c->pin_hdr;
      e.hdr_ev = c->hdr_ev;
      e.n_nodes = std::max(prev_nodes, 1);
      e.lvl_start_host = prev;
      e.depth = pred;
      e.dev = true;
      e.upward_done = true;
      e.up_done = c->up_done;
      HIPCHK(c, launch_evaluate(c->t, e, c->stream));
    }
    HIPCHK(c, hipEventSynchronize(c->hdr_ev));
    memcpy(&c->hh, c->pin_hdr, sizeof(Header));
    if (c->hh.nonfinite) return fail_queued(FMM_ENONFINITE, "non-finite input position");
    const int need = std::min(FMM_MAXLEVEL, c->hh.max_prefix + 1);
    if (need <= pred && !(c->hh.overflow & OVF_ANY)) {
      record_levels(c, need);
      st = finish(tree_depth());
      if (st == FMM_OK && fuse) {
        count_evaluation(c, n_req, reqs);
        *evaluated = true;
      }
      return st;
    }
    heed_path();
  }
  // 1. tree; one readback of the level sizes (exact launches for the walk).
  // With the direct build the split depth need not be read first.
  int max_level = 0;
  for (int attempt = 0;; ++attempt) {
    if (attempt == 4) return fail(c, FMM_EOVERFLOW, "node workspace still too small");
    HIPCHK(c, launch_sort(c->t, a, c->stream));
    if (direct) HIPCHK(c, launch_build_tree_direct(c->t, a, FMM_MAXLEVEL, c->stream));
    st = read_header(c);
    if (st != FMM_OK) return st;
    if (c->hh.nonfinite) return fail(c, FMM_ENONFINITE, "non-finite input position");
    // no cell below level split_depth + 1 holds more than leaf_size particles
    max_level = std::min(FMM_MAXLEVEL, c->hh.max_prefix + 1);
    if (!direct && !(c->hh.overflow & OVF_NODES)) {
      HIPCHK(c, launch_build_tree(c->t, a, max_level, c->stream));
      st = read_header(c);
      if (st != FMM_OK) return st;
    }
    if (!(c->hh.overflow & OVF_NODES)) break;
    int64_t need = std::max<int64_t>(std::max<int64_t>((int64_t)c->hh.lvl_start[FMM_NLEVELS],
                                                       n_req),
                                     2 * c->t.cap_nodes);
    const int64_t old = c->t.cap_nodes;
    free_nodes(c);
    if (!alloc_nodes(c, need + need / 4)) {
      (void)alloc_nodes(c, old);  // as it was, for later builds
      return fail(c, FMM_ENOMEM, "node workspace regrow to %lld failed", (long long)need);
    }
  }
  const int depth = tree_depth();
  int32_t lvl[FMM_NLEVELS + 2];
  memcpy(lvl, c->hh.lvl_start, sizeof(lvl));
  a.lvl_host = lvl;
  a.depth = depth;
  // with the masses known (fmm_forces), the mass gather, P2M and M2M need only
  // the tree: they run on the second stream beside the walk, which leaves
  // most of the chip idle
  bool up = false;
  if (p_fused > 0 && n_all > 0) {
    EvalArgs u = {};
    set_eval_args(c, u, n_all, p_fused, eps);
    u.n_nodes = lvl[FMM_NLEVELS];
    u.lvl_start_host = lvl;
    u.depth = depth;
    HIPCHK(c, hipEventRecord(c->fork, c->stream));
    HIPCHK(c, hipStreamWaitEvent(c->side, c->fork, 0));
    HIPCHK(c, launch_upward(c->t, u, c->side));
    HIPCHK(c, hipEventRecord(c->up_done, c->side));
    up = true;
  }
  // 2. symmetric walk; regrow a list buffer that turned out too small.  With
  // the masses known the evaluation is queued behind the first walk before the
  // header is read (no host round trip between them): its kernels take the
  // node count and level bounds from the header and do nothing if a list
  // buffer overflowed; then the lists are regrown, the walk is redone and
  // *evaluated stays false (the caller evaluates again).
  const bool few_groups = lvl[FMM_NLEVELS] - c->hh.n_leaves <= WALK_PATH_GROUPS;
  for (int attempt = 0; attempt < 10; ++attempt) {
    if (paths_ok && few_groups)
      HIPCHK(c, launch_traverse_paths(c->t, a, lvl[FMM_NLEVELS], false, c->stream));
    else
      HIPCHK(c, launch_traverse(c->t, a, c->stream));
    bool queued = false;
    if (up && evaluated && attempt == 0) {
      // the header copy goes behind the walk and the near-field plan, on the
      // side stream; the host waits for the copy only
      EvalArgs e = {};
      set_eval_args(c, e, n_all, p_fused, eps);
      e.plan = &a;
      e.pin_hdr = c->pin_hdr;
      e.hdr_ev = c->hdr_ev;
      e.n_nodes = lvl[FMM_NLEVELS];
      e.lvl_start_host = lvl;
      e.depth = depth;
      e.dev = true;
      e.exact = true;
      e.upward_done = true;
      e.up_done = c->up_done;
      HIPCHK(c, launch_evaluate(c->t, e, c->stream));
      queued = true;
      HIPCHK(c, hipEventSynchronize(c->hdr_ev));
      memcpy(&c->hh, c->pin_hdr, sizeof(Header));
    } else {
      HIPCHK(c, launch_p2p_plan(c->t, a, c->stream));
      st = read_header(c);
      if (st != FMM_OK) return st;
    }
    const Header &h = c->hh;
    if (h.overflow & OVF_STACK) return fail(c, FMM_EOVERFLOW, "walk descent stack overflow");
    if (h.overflow & (OVF_M2L | OVF_P2P | OVF_OPEN | OVF_ITEMS | OVF_PATH)) {
      heed_path();
      if (h.overflow & OVF_M2L) {
        st = regrow_lists(c, OVF_M2L, (int64_t)h.m2l_cursor);
        if (st != FMM_OK) return st;
      }
      if (h.overflow & OVF_P2P) {
        st = regrow_lists(c, OVF_P2P, (int64_t)h.p2p_cursor);
        if (st != FMM_OK) return st;
      }
      if (h.overflow & OVF_OPEN) {
        unsigned long long mx = 0;
        for (int l = 0; l < FMM_NLEVELS; ++l) mx = std::max(mx, h.open_cursor[l]);
        st = regrow_lists(c, OVF_OPEN, (int64_t)mx);
        if (st != FMM_OK) return st;
      }
      if (h.overflow & OVF_ITEMS) {
        st = regrow_items(c, h.item_cursor, (int64_t)h.part_cursor);
        if (st != FMM_OK) return st;
      }
      continue;
    }
    record_levels(c, max_level);
    st = finish(depth);
    if (st == FMM_OK && upward) *upward = up;
    if (st == FMM_OK && queued) {
      count_evaluation(c, n_req, reqs);
      *evaluated = true;
    }
    return st;
  }
  return fail(c, FMM_EOVERFLOW, "list workspace still too small after regrowth");
}

extern "C" fmm_status fmm_build_batched(fmm_ctx *c, int n_req, const fmm_request *reqs,
                                        double eps, double theta) {
  return build_impl(c, n_req, reqs, eps, theta, 0, nullptr, nullptr);
}

static fmm_status evaluate_impl(fmm_ctx *c, int n_req, const fmm_request *reqs, int p,
                                bool upward_done);

// A runtime call that failed may have left one stream's work without the other's
// to wait for: neither runs on into the next build.
static fmm_status settled(fmm_ctx *c, fmm_status st) {
  if (c && st == FMM_EDEVICE) {
    (void)hipStreamSynchronize(c->side);
    (void)hipStreamSynchronize(c->stream);
    (void)hipGetLastError();
  }
  return st;
}

extern "C" fmm_status fmm_evaluate_batched(fmm_ctx *c, int n_req, const fmm_request *reqs, int p) {
  return settled(c, evaluate_impl(c, n_req, reqs, p, false));
}

// upward_done: the build of these requests already queued the mass gather,
// P2M and M2M (build_impl with p_fused = p)
static fmm_status evaluate_impl(fmm_ctx *c, int n_req, const fmm_request *reqs, int p,
                                bool upward_done) {
  int64_t n_all = 0;
  fmm_status st = check_requests(c, n_req, reqs, true, &n_all);
  if (st != FMM_OK) return st;
  bool same = c->tree_valid && n_req == (int)c->b_reqs.size();
  for (int r = 0; same && r < n_req; ++r) {
    const fmm_request &a = reqs[r], &b = c->b_reqs[r];
    same = a.pos == b.pos && a.active == b.active && a.n_active == b.n_active &&
           a.n_total == b.n_total;
  }
  if (!same) return fail(c, FMM_ESTALE, "no tree built for these particles");
  if (p < 1 || p > c->prm.p_max || !eval_order_supported(p))
    return fail(c, FMM_EINVAL, "order p=%d unsupported (1..%d)", p, std::min(c->prm.p_max, 6));
  st = upload_requests(c, n_req, reqs, nullptr);
  if (st != FMM_OK) return st;
  EvalArgs e = {};
  set_eval_args(c, e, n_all, p, c->b_eps);
  e.n_nodes = c->n_nodes;
  e.lvl_start_host = c->hh.lvl_start;
  e.depth = c->depth;
  e.upward_done = upward_done;
  e.up_done = c->up_done;
  HIPCHK(c, launch_evaluate(c->t, e, c->stream));
  count_evaluation(c, n_req, reqs);
  return FMM_OK;
}

extern "C" fmm_status fmm_forces_batched(fmm_ctx *c, int n_req, const fmm_request *reqs,
                                         double eps, double theta, int p) {
  if (c && (p < 1 || p > c->prm.p_max || !eval_order_supported(p)))
    return fail(c, FMM_EINVAL, "order p=%d unsupported", p);
  bool evaluated = false, upward = false;
  fmm_status st = build_impl(c, n_req, reqs, eps, theta, p, &evaluated, &upward);
  if (st != FMM_OK || evaluated) return settled(c, st);
  return settled(c, evaluate_impl(c, n_req, reqs, p, upward));
}

static fmm_request one_request(const double *pos, const double *mass, int64_t n_total,
                               const int32_t *active, int64_t n_active, double *acc, double *pot) {
  fmm_request q = {};
  q.pos = pos;
  q.n_total = n_total;
  q.active = active;
  q.n_active = n_active;
  q.mass = mass;
  q.acc = acc;
  q.pot = pot;
  return q;
}

extern "C" fmm_status fmm_build(fmm_ctx *c, const double *pos, int64_t n_total,
                                const int32_t *active, int64_t n_active, double eps,
                                double theta) {
  fmm_request q = one_request(pos, nullptr, n_total, active, n_active, nullptr, nullptr);
  return fmm_build_batched(c, 1, &q, eps, theta);
}

extern "C" fmm_status fmm_evaluate(fmm_ctx *c, const double *pos, const double *mass,
                                   int64_t n_total, const int32_t *active, int64_t n_active, int p,
                                   double *acc, double *pot) {
  fmm_request q = one_request(pos, mass, n_total, active, n_active, acc, pot);
  return fmm_evaluate_batched(c, 1, &q, p);
}

extern "C" fmm_status fmm_forces(fmm_ctx *c, const double *pos, const double *mass,
                                 int64_t n_total, const int32_t *active, int64_t n_active,
                                 double eps, double theta, int p, double *acc, double *pot) {
  fmm_request q = one_request(pos, mass, n_total, active, n_active, acc, pot);
  return fmm_forces_batched(c, 1, &q, eps, theta, p);
}

extern "C" fmm_status fmm_forces_grad(fmm_ctx *c, const double *pos, const double *mass,
                                      int64_t n_total, const int32_t *active, int64_t n_active,
                                      double eps, double theta, int p, double *acc, double *pot,
                                      double *grad) {
  if (!c) return FMM_EINVAL;
  if (n_active > 0 && !grad) return fail(c, FMM_EINVAL, "grad is NULL");
  if (!c->gstage && !dalloc(c, &c->gstage, 6 * c->max_n))
    return fail(c, FMM_ENOMEM, "force-gradient staging");
  fmm_status st = fmm_forces(c, pos, mass, n_total, active, n_active, eps, theta, p, acc, pot);
  if (st != FMM_OK || n_active == 0) return st;
  const int64_t rows = (int64_t)c->hh.part_cursor;
  if (6 * rows > c->gpart_len && !fmm_regrow(c, &c->gpart, &c->gpart_len, 6 * (rows + rows / 4))) {
    c->t.uncut = 1;  // as in regrow_items
    st = fmm_forces(c, pos, mass, n_total, active, n_active, eps, theta, p, acc, pot);
    if (st != FMM_OK) return st;
  }
  HIPCHK(c, launch_force_gradient(c->t, c->n_nodes, (int)n_active, p, c->prm.kernel,
                                  c->prm.precision == FMM_PREC_MIXED, eps, c->gstage, c->gpart,
                                  grad, c->stream));
  return FMM_OK;
}

extern "C" fmm_status fmm_evaluate_dipole(fmm_ctx *c, const double *pos, const double *mass,
                                          int64_t n_total, const int32_t *active,
                                          int64_t n_active, int p, const double *vec, double *u,
                                          double *phi) {
  if (!c) return FMM_EINVAL;
  if (n_active > 0 && (!vec || !u || !phi || !mass))
    return fail(c, FMM_EINVAL, "NULL mass, vec, u or phi");
  if (c->tree_valid && c->b_reqs.size() != 1)
    return fail(c, FMM_EINVAL, "the vector-source pass needs a single-system tree");
  fmm_request q = one_request(pos, mass, n_total, active, n_active, u, phi);
  int64_t n_all = 0;
  fmm_status st = check_requests(c, 1, &q, true, &n_all);
  if (st != FMM_OK) return st;
  const fmm_request &b = c->b_reqs.empty() ? q : c->b_reqs[0];
  if (!c->tree_valid || b.pos != pos || b.active != active || b.n_active != n_active ||
      b.n_total != n_total)
    return fail(c, FMM_ESTALE, "no tree built for these particles");
  if (p < 1 || p > c->prm.p_max || !eval_order_supported(p))
    return fail(c, FMM_EINVAL, "order p=%d unsupported (1..%d)", p, std::min(c->prm.p_max, 6));
  if (n_active == 0) return FMM_OK;
  if (!c->dvec && !dalloc(c, &c->dvec, 3 * c->max_n))
    return fail(c, FMM_ENOMEM, "vector-source scratch");
  st = upload_requests(c, 1, &q, nullptr);
  if (st != FMM_OK) return st;
  EvalArgs e = {};
  set_eval_args(c, e, n_all, p, c->b_eps);
  e.n_nodes = c->n_nodes;
  e.lvl_start_host = c->hh.lvl_start;
  e.depth = c->depth;
  HIPCHK(c, launch_dipole(c->t, e, vec, c->dvec, c->stream));
  return FMM_OK;
}

extern "C" fmm_status fmm_tree_info(fmm_ctx *c, int64_t info[9]) {
  if (!c || !info) return FMM_EINVAL;
  if (!c->tree_valid) return fail(c, FMM_ESTALE, "no tree");
  const Header &h = c->hh;
  int64_t leaves = h.n_leaves;
  info[0] = c->b_n;  // active particles over all requests
  info[1] = c->n_nodes;
  info[2] = (int64_t)(h.m2l_cursor / 2);
  info[3] = ((int64_t)h.p2p_cursor - leaves) / 2 + leaves;
  info[4] = c->depth;
  info[5] = leaves;
  info[6] = (int64_t)h.m2l_cursor;
  info[7] = (int64_t)h.p2p_cursor;
  info[8] = (int64_t)h.p2p_pairs;
  return FMM_OK;
}

template <typename T>
static hipError_t d2h(std::vector<T> &v, const T *d, int64_t n, hipStream_t s) {
  v.resize((size_t)std::max<int64_t>(n, 0));
  if (n <= 0) return hipSuccess;
  return hipMemcpyAsync(v.data(), d, sizeof(T) * n, hipMemcpyDeviceToHost, s);
}

extern "C" fmm_status fmm_export_tree(fmm_ctx *c, int64_t *perm, int32_t *level, uint64_t *prefix,
                                      int64_t *begin, int64_t *end, int32_t *is_leaf,
                                      double *centre, double *half, int64_t *m2l_pairs,
                                      int64_t *p2p_pairs, double *box) {
  if (!c) return FMM_EINVAL;
  if (!c->tree_valid) return fail(c, FMM_ESTALE, "no tree");
  if (c->b_reqs.size() != 1) return fail(c, FMM_EINVAL, "export needs a single-request tree");
  const int64_t n = c->b_n, nn = c->n_nodes;
  const DevTree &t = c->t;
  std::vector<int32_t> nbeg, nend, nlev, nnch, slot, moff, mcnt, msrc, poff, pcnt, psrc;
  std::vector<uint64_t> key;
  std::vector<double4> geo;
  Box hb;
  hipStream_t s = c->stream;
  // single request: slot == active slot
  HIPCHK(c, d2h(nbeg, t.nbeg, nn, s));
  HIPCHK(c, d2h(nend, t.nend, nn, s));
  HIPCHK(c, d2h(nlev, t.nlev, nn, s));
  HIPCHK(c, d2h(nnch, t.nnchild, nn, s));
  HIPCHK(c, d2h(geo, t.ngeo, nn, s));
  HIPCHK(c, d2h(slot, t.slot, n, s));
  HIPCHK(c, d2h(key, t.key, n, s));
  HIPCHK(c, d2h(moff, t.m2l_off, nn, s));
  HIPCHK(c, d2h(mcnt, t.m2l_cnt, nn, s));
  HIPCHK(c, d2h(poff, t.p2p_off, nn, s));
  HIPCHK(c, d2h(pcnt, t.p2p_cnt, nn, s));
  HIPCHK(c, d2h(msrc, t.m2l_src, (int64_t)c->hh.m2l_cursor, s));
  HIPCHK(c, d2h(psrc, t.p2p_src, (int64_t)c->hh.p2p_cursor, s));
  HIPCHK(c, hipMemcpyAsync(&hb, t.box, sizeof(Box), hipMemcpyDeviceToHost, s));
  HIPCHK(c, hipStreamSynchronize(s));
  if (n == 0) {  // the root of an empty system: no walk wrote its lists, no key its prefix
    mcnt.assign(nn, 0);
    pcnt.assign(nn, 1);  // itself, as fmm_tree_info counts
    poff.assign(nn, 0);
    psrc.assign(1, 0);
    key.assign(1, 0);
  }
  // canonical pre-order id: nodes sorted by (begin, level)
  std::vector<int64_t> order(nn), canon(nn);
  for (int64_t i = 0; i < nn; ++i) order[i] = i;
  std::sort(order.begin(), order.end(), [&](int64_t a, int64_t b) {
    if (nbeg[a] != nbeg[b]) return nbeg[a] < nbeg[b];
    return nlev[a] < nlev[b];
  });
  for (int64_t r = 0; r < nn; ++r) canon[order[r]] = r;
  if (perm)
    for (int64_t i = 0; i < n; ++i) perm[i] = slot[i];
  for (int64_t r = 0; r < nn; ++r) {
    int64_t i = order[r];
    if (level) level[r] = nlev[i];
    if (prefix) prefix[r] = key[nbeg[i]] >> (3 * (FMM_MAXLEVEL - nlev[i]));
    if (begin) begin[r] = nbeg[i];
    if (end) end[r] = nend[i];
    if (is_leaf) is_leaf[r] = nnch[i] == 0;
    if (centre) {
      centre[3 * r] = geo[i].x;
      centre[3 * r + 1] = geo[i].y;
      centre[3 * r + 2] = geo[i].z;
    }
    if (half) half[r] = geo[i].w;
  }
  auto pairs = [&](const std::vector<int32_t> &off, const std::vector<int32_t> &cnt,
                   const std::vector<int32_t> &src, int64_t *out) {
    std::vector<std::pair<int64_t, int64_t>> v;
    for (int64_t a = 0; a < nn; ++a)
      for (int q = 0; q < cnt[a]; ++q) {
        int64_t b = src[off[a] + q];
        int64_t ca = canon[a], cb = canon[b];
        if (ca <= cb) v.emplace_back(ca, cb);
      }
    std::sort(v.begin(), v.end());
    for (size_t k = 0; k < v.size(); ++k) {
      out[2 * k] = v[k].first;
      out[2 * k + 1] = v[k].second;
    }
  };
  if (m2l_pairs) pairs(moff, mcnt, msrc, m2l_pairs);
  if (p2p_pairs) pairs(poff, pcnt, psrc, p2p_pairs);
  if (box) {
    box[0] = hb.o[0];
    box[1] = hb.o[1];
    box[2] = hb.o[2];
    box[3] = hb.L;
    box[4] = hb.s;
  }
  return FMM_OK;
}

extern "C" fmm_status fmm_invariants(fmm_ctx *c, const double *pos, const double *vel,
                                     const double *mass, const double *acc, const double *pot,
                                     int64_t n, double out[12]) {
  if (!c || !out || n < 0) return FMM_EINVAL;
  const int nblk = FMM_INV_BLOCKS;
  launch_invariants(pos, vel, mass, acc, pot, n, c->inv_part, nblk, c->stream);
  std::vector<double> part(nblk * 12);
  HIPCHK(c, hipMemcpyAsync(part.data(), c->inv_part, sizeof(double) * nblk * 12,
                           hipMemcpyDeviceToHost, c->stream));
  HIPCHK(c, hipStreamSynchronize(c->stream));
  for (int k = 0; k < 12; ++k) {
    double s = 0.0;
    for (int b = 0; b < nblk; ++b) s += part[b * 12 + k];
    out[k] = s;
  }
  return FMM_OK;
}

extern "C" fmm_status fmm_profile_enable(fmm_ctx *c, int enable) {
  if (!c) return FMM_EINVAL;
  PhaseTimer &tm = c->timer;
  if (enable && !tm.ready) {
    for (int i = 0; i < PhaseTimer::CAP; ++i) {
      HIPCHK(c, hipEventCreate(&tm.a[i]));
      HIPCHK(c, hipEventCreate(&tm.b[i]));
    }
    tm.ready = true;
  }
  if (tm.on) tm.flush();
  tm.on = enable != 0;
  tm.mask = enable == 2 ? (1u << PH_M2L | 1u << PH_P2P) : ~0u;
  tm.n = 0;
  for (int k = 0; k < PH_N; ++k) {
    tm.ms[k] = 0.0;
    tm.cnt[k] = 0;
  }
  return FMM_OK;
}

extern "C" fmm_status fmm_profile_read(fmm_ctx *c, double ms[7], int64_t calls[7]) {
  if (!c || !ms || !calls) return FMM_EINVAL;
  c->timer.flush();
  for (int k = 0; k < PH_N; ++k) {
    ms[k] = c->timer.ms[k];
    calls[k] = c->timer.cnt[k];
  }
  return FMM_OK;
}
