// Morton-ordered oct-tree build on gfx950.
//
// Steps (all device-side; the host only queues launches):
//   1. root box: per-axis min/max of the active positions; centre
//      c = (lo+hi)/2, side L = max extent (1 if zero), origin o = c - L/2,
//      scale s = 2^21/L;
//   2. 63-bit Morton keys from q_d = clamp(floor((x_d - o_d) s), 0, 2^21-1),
//      x bits at 3b+2, y at 3b+1, z at 3b;
//   3. stable sort of (key, active slot): tiles sorted in LDS and merged by
//      rank, or for large systems and batches (sort_merges) an LSD radix
//      sort, 8 passes of 8 bits, ranks inside a wavefront from 8 ballots per 64
//      keys;
//   4. top-down split (the paper's recursive build, Sec. 2.3, done level by
//      level): a cell of level l < 21 holding more than leaf_size particles
//      gets one child per non-empty octant of its key range; children of a
//      level are emitted in Morton order after a count / scan / emit sweep;
//   5. geometric centre z = o + (i + 1/2) L 2^-l and half side h = L 2^-(l+1)
//      of every cell; cell-local FP32 offsets of every particle.
// All decisions are the same IEEE double expressions as in the definition
// above, built with -ffp-contract=off, so keys, octant membership and centres
// are reproducible bit for bit.
#include <algorithm>

#include "common.h"
#include "hhs_kernels.h"

#define SORT_WAVES 16                          // wavefronts per radix tile
#define SORT_ITEMS (SORT_TILE / (SORT_WAVES * 64))
#define SORT_THREADS (SORT_WAVES * 64)
#define BBOX_COLS FMM_BBOX_COLS

// ---------------------------------------------------------------------------
// request of every slot (binary search in the request offsets)
// ---------------------------------------------------------------------------

// request of every active slot, for the request passes of the radix sort
__global__ __launch_bounds__(FMM_BLOCK) void k_slot_req(DevTree t, int n) {
  int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s < n) t.slot_req[s] = upper_index(t.req_off, t.n_req, s);
}

// ---------------------------------------------------------------------------
// root box of every request
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(FMM_BLOCK) void k_bbox_partial(DevTree t) {
  const int r = upper_index(t.blk_off, t.n_req, blockIdx.x);
  const DevReq q = t.reqs[r];
  const int lb = blockIdx.x - t.blk_off[r], nbr = t.blk_off[r + 1] - t.blk_off[r];
  double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  int bad = 0;
  for (int i = lb * blockDim.x + threadIdx.x; i < q.n; i += nbr * blockDim.x) {
    int64_t g = q.active ? q.active[i] : i;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      double x = q.pos[d * q.n_total + g];
      bad |= !isfinite(x);
      lo[d] = fmin(lo[d], x);
      hi[d] = fmax(hi[d], x);
    }
  }
  __shared__ double red[6][FMM_BLOCK];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    red[d][threadIdx.x] = lo[d];
    red[3 + d][threadIdx.x] = hi[d];
  }
  bad = __syncthreads_or(bad);
  for (int o = FMM_BLOCK / 2; o > 0; o >>= 1) {
    if (threadIdx.x < o) {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        red[d][threadIdx.x] = fmin(red[d][threadIdx.x], red[d][threadIdx.x + o]);
        red[3 + d][threadIdx.x] = fmax(red[3 + d][threadIdx.x], red[3 + d][threadIdx.x + o]);
      }
    }
    __syncthreads();
  }
  if (threadIdx.x < 7)
    t.bbox_part[blockIdx.x * BBOX_COLS + threadIdx.x] =
        threadIdx.x < 6 ? red[threadIdx.x][0] : (bad ? 1.0 : 0.0);
}

// c = (lo+hi)/2, L = max extent (1 if 0), o = c - L/2, s = 2^21/L
__device__ __forceinline__ void finish_box(Box &bx, double lo[3], double hi[3], bool empty) {
  if (empty)
    for (int d = 0; d < 3; ++d) lo[d] = hi[d] = 0.0;
  double c[3], L = 0.0;
  for (int d = 0; d < 3; ++d) {
    c[d] = 0.5 * (lo[d] + hi[d]);
    double e = hi[d] - lo[d];
    if (e > L) L = e;
  }
  if (L == 0.0) L = 1.0;
  for (int d = 0; d < 3; ++d) {
    bx.o[d] = c[d] - 0.5 * L;
    bx.lo[d] = lo[d];
    bx.hi[d] = hi[d];
  }
  bx.L = L;
  bx.s = 2097152.0 / L;
}

// ---------------------------------------------------------------------------
// Morton keys
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t spread3(uint64_t x) {
  x &= 0x1fffffull;
  x = (x | x << 32) & 0x1f00000000ffffull;
  x = (x | x << 16) & 0x1f0000ff0000ffull;
  x = (x | x << 8) & 0x100f00f00f00f00full;
  x = (x | x << 4) & 0x10c30c30c30c30c3ull;
  x = (x | x << 2) & 0x1249249249249249ull;
  return x;
}

__device__ __forceinline__ uint32_t compact3(uint64_t x) {
  x &= 0x1249249249249249ull;
  x = (x ^ (x >> 2)) & 0x10c30c30c30c30c3ull;
  x = (x ^ (x >> 4)) & 0x100f00f00f00f00full;
  x = (x ^ (x >> 8)) & 0x1f0000ff0000ffull;
  x = (x ^ (x >> 16)) & 0x1f00000000ffffull;
  x = (x ^ (x >> 32)) & 0x1fffffull;
  return (uint32_t)x;
}

__device__ __forceinline__ uint64_t quantise(double x, double o, double s) {
  double q = floor((x - o) * s);
  const double qmax = 2097151.0;
  if (!(q >= 0.0)) q = 0.0;
  if (q > qmax) q = qmax;
  return (uint64_t)q;
}

// key and packed position of active slot s, of request r
__device__ __forceinline__ uint64_t make_key(const DevTree &t, int s, int r, double4 &pos) {
  const DevReq q = t.reqs[r];
  const int i = s - q.off;
  int64_t g = q.active ? q.active[i] : i;
  const Box &bx = t.box[r];
  const double x = q.pos[g], y = q.pos[q.n_total + g], z = q.pos[2 * q.n_total + g];
  uint64_t qx = quantise(x, bx.o[0], bx.s);
  uint64_t qy = quantise(y, bx.o[1], bx.s);
  uint64_t qz = quantise(z, bx.o[2], bx.s);
  pos = make_double4(x, y, z, 0.0);
  t.pak[s] = pos;
  return (spread3(qx) << 2) | (spread3(qy) << 1) | spread3(qz);
}

// keys and slots into key2 / slot2 when the sort that follows makes an odd
// number of passes (so that its result lands in key / slot)
__global__ __launch_bounds__(FMM_BLOCK) void k_keys(DevTree t, int n, int odd) {
  int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n) return;
  const int r = t.n_req > 1 ? t.slot_req[s] : 0;
  double4 pos;
  (odd ? t.key2 : t.key)[s] = make_key(t, s, r, pos);
  (odd ? t.slot2 : t.slot)[s] = s;
}

// ---------------------------------------------------------------------------
// stable LSD radix sort, 8-bit digits
// ---------------------------------------------------------------------------
// digit of element i: bits [shift, shift+8) of its key (by_req = 0) or of the
// request of its slot (by_req = 1; these passes come last, so the final order
// is by (request, key, slot))
__device__ __forceinline__ uint32_t sort_digit(const uint64_t *key, const int32_t *slot,
                                               const int32_t *slot_req, int i, int shift,
                                               int by_req) {
  return by_req ? ((uint32_t)slot_req[slot[i]] >> shift) & 255u
                : (uint32_t)(key[i] >> shift) & 255u;
}

__global__ __launch_bounds__(SORT_THREADS) void k_sort_hist(const uint64_t *__restrict__ key,
                                                            const int32_t *__restrict__ slot,
                                                            const int32_t *__restrict__ slot_req,
                                                            int n, int shift, int by_req,
                                                            uint32_t *__restrict__ hist, int nblk) {
  __shared__ uint32_t h[256];
  if (threadIdx.x < 256) h[threadIdx.x] = 0;
  __syncthreads();
  const int base = blockIdx.x * SORT_TILE;
#pragma unroll
  for (int it = 0; it < SORT_ITEMS; ++it) {
    const int i = base + it * SORT_THREADS + threadIdx.x;
    if (i < n) atomicAdd(&h[sort_digit(key, slot, slot_req, i, shift, by_req)], 1u);
  }
  __syncthreads();
  if (threadIdx.x < 256) hist[threadIdx.x * nblk + blockIdx.x] = h[threadIdx.x];
}

// Per-digit exclusive scan over the blocks: hist[d][0..nblk) in place, digit
// total to dtot[d].  One workgroup per digit, coalesced tiles of 256.
__global__ __launch_bounds__(FMM_BLOCK) void k_sort_digit_scan(uint32_t *hist, int nblk,
                                                               uint32_t *dtot) {
  __shared__ uint32_t v[FMM_BLOCK];
  uint32_t *h = hist + (size_t)blockIdx.x * nblk;
  uint32_t run = 0;
  for (int base = 0; base < nblk; base += FMM_BLOCK) {
    int i = base + threadIdx.x;
    uint32_t x = i < nblk ? h[i] : 0u;
    v[threadIdx.x] = x;
    __syncthreads();
    for (int off = 1; off < FMM_BLOCK; off <<= 1) {
      uint32_t y = threadIdx.x >= off ? v[threadIdx.x - off] : 0u;
      __syncthreads();
      v[threadIdx.x] += y;
      __syncthreads();
    }
    if (i < nblk) h[i] = run + v[threadIdx.x] - x;
    run += v[FMM_BLOCK - 1];
    __syncthreads();
  }
  if (threadIdx.x == 0) dtot[blockIdx.x] = run;
}

// Exclusive scan of one value per thread over threads 0..255 of a block
// (the others pass 0 and get 0); every thread of the block must call it.
__device__ __forceinline__ uint32_t scan256(uint32_t v, uint32_t *wsum) {
  const int w = threadIdx.x >> 6;
  uint32_t ex = 0;
  if (threadIdx.x < 256) {
    int tot;
    ex = (uint32_t)wave_excl_scan_int((int)v, &tot);
    if ((threadIdx.x & 63) == 0) wsum[w] = (uint32_t)tot;
  }
  __syncthreads();
  if (threadIdx.x < 256)
    for (int ww = 0; ww < w; ++ww) ex += wsum[ww];
  __syncthreads();
  return ex;
}

// One radix pass over a tile of SORT_TILE keys: every key's rank among the
// tile's keys of its digit (8 ballots per 64 keys, waves in index order, so
// the pass is stable), the tile reordered by digit in LDS, then written out
// in tile order so that consecutive threads store consecutive addresses of a
// digit's run.
// hist holds each digit's exclusive prefix over the tiles and dtot the digit
// totals.
__global__ __launch_bounds__(SORT_THREADS) void k_sort_scatter(
    const uint64_t *__restrict__ kin, const int32_t *__restrict__ sin, uint64_t *__restrict__ kout,
    int32_t *__restrict__ sout, const int32_t *__restrict__ slot_req, int n, int shift, int by_req,
    const uint32_t *__restrict__ hist, int nblk, const uint32_t *__restrict__ dtot) {
  // keys | slots | digits of the reordered tile; the per-wave digit counters
  // of the ranking step live in the front of the same space before that
  __shared__ __align__(16) unsigned char smem[SORT_TILE * 13];
  __shared__ uint32_t lstart[256], gbase[256], wsum[SORT_WAVES];
  uint64_t *skey = (uint64_t *)smem;
  int32_t *sslot = (int32_t *)(smem + 8 * SORT_TILE);
  uint8_t *sdig = smem + 12 * SORT_TILE;
  uint32_t(*cnt)[256] = (uint32_t(*)[256])smem;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  for (int d = tid; d < SORT_WAVES * 256; d += SORT_THREADS) (&cnt[0][0])[d] = 0;
  // global start of each digit: exclusive scan of the digit totals, plus the
  // counts of the earlier tiles
  uint32_t dtotal = 0, tprefix = 0;
  if (tid < 256) {
    dtotal = dtot[tid];
    tprefix = hist[tid * nblk + blockIdx.x];
  }
  const uint32_t dbase = scan256(dtotal, wsum);
  const int tile = blockIdx.x * SORT_TILE;
  const int base = tile + w * 64 * SORT_ITEMS;
  uint64_t k[SORT_ITEMS];
  int32_t sv[SORT_ITEMS];
  uint32_t dg[SORT_ITEMS], rank[SORT_ITEMS];
  const unsigned long long below = lanes_below_mask();
#pragma unroll
  for (int it = 0; it < SORT_ITEMS; ++it) {
    const int i = base + it * 64 + lane;
    const bool valid = i < n;
    k[it] = valid ? kin[i] : 0;
    sv[it] = valid ? sin[i] : 0;
  }
#pragma unroll
  for (int it = 0; it < SORT_ITEMS; ++it) {
    const int i = base + it * 64 + lane;
    const bool valid = i < n;
    const uint32_t d = by_req ? (valid ? ((uint32_t)slot_req[sv[it]] >> shift) & 255u : 0u)
                              : (uint32_t)(k[it] >> shift) & 255u;
    dg[it] = d;
    unsigned long long m = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const unsigned long long bal = __ballot((d >> b) & 1u);
      m &= ((d >> b) & 1u) ? bal : ~bal;
    }
    const uint32_t prior = cnt[w][d];
    rank[it] = prior + (uint32_t)__popcll(m & below);
    __builtin_amdgcn_wave_barrier();
    if (valid && (m & below) == 0) cnt[w][d] = prior + (uint32_t)__popcll(m);
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  // per digit: offsets of the waves inside the tile (in place), tile count
  uint32_t tcount = 0;
  if (tid < 256) {
#pragma unroll
    for (int ww = 0; ww < SORT_WAVES; ++ww) {
      const uint32_t c = cnt[ww][tid];
      cnt[ww][tid] = tcount;
      tcount += c;
    }
  }
  const uint32_t ls = scan256(tcount, wsum);
  if (tid < 256) {
    lstart[tid] = ls;
    gbase[tid] = dbase + tprefix - ls;
  }
  __syncthreads();
  int lpos[SORT_ITEMS];
#pragma unroll
  for (int it = 0; it < SORT_ITEMS; ++it) lpos[it] = (int)(lstart[dg[it]] + cnt[w][dg[it]] + rank[it]);
  __syncthreads();  // the counters are overwritten below
#pragma unroll
  for (int it = 0; it < SORT_ITEMS; ++it) {
    if (base + it * 64 + lane < n) {
      skey[lpos[it]] = k[it];
      sslot[lpos[it]] = sv[it];
      sdig[lpos[it]] = (uint8_t)dg[it];
    }
  }
  __syncthreads();
  const int tn = min(SORT_TILE, n - tile);
#pragma unroll
  for (int it = 0; it < SORT_ITEMS; ++it) {
    const int j = it * SORT_THREADS + tid;
    if (j < tn) {
      const uint32_t dst = gbase[sdig[j]] + (uint32_t)j;
      kout[dst] = skey[j];
      sout[dst] = sslot[j];
    }
  }
}

// ---------------------------------------------------------------------------
// Merge sort, where sort_merges finds it the faster: tiles of 1024 slots sorted
// in LDS (the kernel that makes the keys), then 16 runs at a time merged by rank.  An element's place in the
// merged run is its place in its own run plus, for each other run, the number
// of keys before it there, a binary search; the searches of 8 runs go on side
// by side, so a merge costs some 20 dependent reads whatever its size.  The 8
// radix passes cost 9 us each in launches and latency below 65,536 particles,
// and 17 with their histogram and digit-scan launches above.  Sorts, in all:
// 12,526 particles 34 us (radix 73 + 6 in 10 launches), 100,003 53 (140
// in 25), 300,007 128 (149); at 2^20 the searches read more than the passes
// (radix 171 us).
//
// Several systems: their slots are contiguous, and so are their sorted
// positions, in every run: position q belongs to the same system before and
// after, and an element is ranked among its own system's part of a run only.
// A system's runs are counted from the tile its first slot is in.  Equal keys
// keep slot order: runs before its own count keys up to and including an
// element's, runs after it keys below.
// ---------------------------------------------------------------------------
// Sorted LDS runs of RUN elements merged four at a time: the element at
// position p of kin (its system's slots lie in [s0, s1) of the tile) moves to
// its place in kout.
template <int RUN>
__device__ __forceinline__ void lds_merge4(const uint64_t *kin, const uint16_t *iin, uint64_t *kout,
                                           uint16_t *iout, int p, bool valid, int s0, int s1) {
  if (!valid) return;
  const uint64_t k = kin[p];
  const int g0 = p & ~(4 * RUN - 1), m = (p / RUN) & 3;
  int at = max(s0, g0) + p - max(s0, g0 + m * RUN);
  int lo[3], hi[3];
#pragma unroll
  for (int u = 0; u < 3; ++u) {
    const int j = u + (u >= m ? 1 : 0);
    lo[u] = max(s0, g0 + j * RUN);
    hi[u] = max(lo[u], min(s1, g0 + j * RUN + RUN));
    at -= lo[u];
  }
  // RUN + 1 possible places: this many halvings always end the search
#pragma unroll
  for (int st = RUN; st > 0; st >>= 1)
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      const int mid = (lo[u] + hi[u]) >> 1;
      const uint64_t x = kin[min(mid, MSORT_TILE - 1)];
      const bool right = lo[u] < hi[u] && (x < k || (u < m && x == k));
      const bool left = lo[u] < hi[u] && !right;
      lo[u] = right ? mid + 1 : lo[u];
      hi[u] = left ? mid : hi[u];
    }
#pragma unroll
  for (int u = 0; u < 3; ++u) at += lo[u];
  kout[at] = k;
  iout[at] = iin[p];
}

struct TileLds {
  uint64_t ka[MSORT_TILE], kb[MSORT_TILE];
  uint16_t ia[MSORT_TILE], ib[MSORT_TILE];
  double x[MSORT_TILE], y[MSORT_TILE], z[MSORT_TILE];
};

// Keys of the slots of one tile, sorted to kout / sout; last: also the sorted
// positions.  A workgroup of MSORT_TILE threads.
__device__ __forceinline__ void sort_tile(const DevTree &t, int n, int tile, uint64_t *kout,
                                          int32_t *sout, bool last, TileLds &L) {
  const int p = threadIdx.x, q = tile * MSORT_TILE + p;
  const bool valid = q < n;
  int s0 = 0, s1 = 0;  // the system's slots, within the tile
  uint64_t key = 0;
  if (valid) {
    const int r = t.n_req > 1 ? upper_index(t.req_off, t.n_req, q) : 0;
    s0 = max(t.req_off[r] - tile * MSORT_TILE, 0);
    s1 = min(t.req_off[r + 1] - tile * MSORT_TILE, MSORT_TILE);
    double4 pos;
    key = make_key(t, q, r, pos);
    L.x[p] = pos.x;
    L.y[p] = pos.y;
    L.z[p] = pos.z;
  }
  L.ka[p] = key;
  __builtin_amdgcn_wave_barrier();
  // runs of 64: rank by counting
  const int w0 = p & ~63;
  {
    const int a = max(s0, w0), b = min(s1, w0 + 64);
    int at = a;
#pragma unroll 16
    for (int j = 0; j < 64; ++j) {
      const uint64_t x = L.ka[w0 + j];
      at += (w0 + j >= a && w0 + j < b && (x < key || (x == key && w0 + j < p))) ? 1 : 0;
    }
    if (valid) {
      L.kb[at] = key;
      L.ib[at] = (uint16_t)p;
    }
  }
  __syncthreads();
  lds_merge4<64>(L.kb, L.ib, L.ka, L.ia, p, valid, s0, s1);
  __syncthreads();
  lds_merge4<256>(L.ka, L.ia, L.kb, L.ib, p, valid, s0, s1);
  __syncthreads();
  if (valid) {
    const int i = L.ib[p];
    kout[q] = L.kb[p];
    sout[q] = tile * MSORT_TILE + i;
    if (last) {
      t.sx[q] = L.x[i];
      t.sy[q] = L.y[i];
      t.sz[q] = L.z[i];
    }
  }
}

__global__ __launch_bounds__(MSORT_TILE) void k_sort_tiles(DevTree t, int n, uint64_t *kout,
                                                           int32_t *sout, bool last) {
  __shared__ TileLds lds;
  sort_tile(t, n, blockIdx.x, kout, sout, last, lds);
}

// Runs of R sorted elements (of every system, from the tile its first slot is
// in) merged MSORT_FAN at a time; last: also the sorted positions.
__global__ __launch_bounds__(FMM_BLOCK) void k_sort_merge(DevTree t, int n, int R,
                                                          const uint64_t *__restrict__ kin,
                                                          const int32_t *__restrict__ sin,
                                                          uint64_t *__restrict__ kout,
                                                          int32_t *__restrict__ sout, bool last) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= n) return;
  const int r = t.n_req > 1 ? upper_index(t.req_off, t.n_req, q) : 0;
  const int off0 = t.req_off[r], off1 = t.req_off[r + 1];
  const uint64_t k = kin[q];
  const int slot = sin[q];
  double4 pos;
  if (last) pos = t.pak[slot];
  const int o = off0 & ~(MSORT_TILE - 1);
  const int run = (q - o) / R, m = run & (MSORT_FAN - 1);
  const int64_t g0 = o + (int64_t)(run - m) * R;  // first slot of the runs merged here
  unsigned at = (unsigned)max((int64_t)off0, g0) + q -
                (unsigned)max((int64_t)off0, g0 + (int64_t)m * R);
  for (int h = 0; h < MSORT_FAN; h += 8) {
    if (h > 0 && g0 + (int64_t)h * R >= off1) break;
    int lo[8], hi[8], len = 0;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int64_t a = g0 + (int64_t)(h + u) * R;
      lo[u] = (int)min((int64_t)off1, max((int64_t)off0, a));
      hi[u] = h + u == m ? lo[u] : (int)max((int64_t)lo[u], min((int64_t)off1, a + R));
      at -= (unsigned)lo[u];
      len = max(len, hi[u] - lo[u]);
    }
    for (; len > 0; len >>= 1) {  // len + 1 places: bit length of len halvings
      uint64_t x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = kin[min((lo[u] + hi[u]) >> 1, n - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int mid = (lo[u] + hi[u]) >> 1;
        const bool right = x[u] < k || (h + u < m && x[u] == k);
        if (lo[u] < hi[u]) {
          lo[u] = right ? mid + 1 : lo[u];
          hi[u] = right ? hi[u] : mid;
        }
      }
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) at += (unsigned)lo[u];
  }
  kout[at] = k;
  sout[at] = slot;
  if (last) {
    t.sx[at] = pos.x;
    t.sy[at] = pos.y;
    t.sz[at] = pos.z;
  }
}

// Deepest level at which a cell holds more than leaf_size particles: a cell
// holds more than leaf_size particles exactly when some sorted key and the key
// leaf_size positions later (same request) share its prefix.  Cells below that
// level are leaves, so the split stops there.
__global__ __launch_bounds__(FMM_BLOCK) void k_split_depth(DevTree t, int n, int stride) {
  int best = 0;
  const uint64_t *key = t.key;
  Header *hdr = t.hdr;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i + stride < n;
       i += gridDim.x * blockDim.x) {
    if (t.n_req > 1) {  // sorted positions are grouped by request, in request order
      const int r = upper_index(t.req_off, t.n_req, i);
      if (i + stride >= t.req_off[r + 1]) continue;
    }
    uint64_t x = key[i] ^ key[i + stride];
    int digits = x == 0 ? FMM_MAXLEVEL : (__clzll(x) - 1) / 3;
    best = max(best, digits);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) best = max(best, __shfl_xor(best, off, 64));
  __shared__ int wbest[FMM_BLOCK / 64];
  if ((threadIdx.x & 63) == 0) wbest[threadIdx.x >> 6] = best;
  __syncthreads();
  if (threadIdx.x == 0) {  // one atomic per block
    for (int w = 1; w < FMM_BLOCK / 64; ++w) best = max(best, wbest[w]);
    if (best > 0) atomicMax(&hdr->max_prefix, best);
  }
}

// ---------------------------------------------------------------------------
// sorted particle data
// ---------------------------------------------------------------------------
// The key pass left each active slot's position in one 32-byte record, so
// the random read of the gather touches one memory sector per particle
// instead of one in each of the three coordinate arrays.
__device__ __forceinline__ void gather_at(const DevTree &t, int j) {
  const double4 r = t.pak[t.slot[j]];
  t.sx[j] = r.x;
  t.sy[j] = r.y;
  t.sz[j] = r.z;
}

__global__ __launch_bounds__(FMM_BLOCK) void k_gather_sorted(DevTree t, int n) {
  int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j < n) gather_at(t, j);
}

// ---------------------------------------------------------------------------
// level-by-level split
// ---------------------------------------------------------------------------
__device__ __forceinline__ double4 cell_geometry(const Box &b, uint64_t prefix, int lev) {
  uint32_t ix = compact3(prefix >> 2), iy = compact3(prefix >> 1), iz = compact3(prefix);
  double w = ldexp(b.L, -lev);
  double4 g;
  g.x = b.o[0] + ((double)ix + 0.5) * w;
  g.y = b.o[1] + ((double)iy + 0.5) * w;
  g.z = b.o[2] + ((double)iz + 0.5) * w;
  g.w = ldexp(b.L, -(lev + 1));
  return g;
}

// header of a new tree (one thread) and the root of request r, covering its
// sorted range [off, off + n)
__device__ __forceinline__ void header_init(const DevTree &t, bool nonfinite) {
  Header *h = t.hdr;
  const int R = t.n_req;
  h->lvl_start[0] = 0;
  for (int l = 1; l < FMM_NLEVELS + 2; ++l) h->lvl_start[l] = R;
  h->overflow = (R > t.cap_nodes ? OVF_NODES : 0) | (nonfinite ? OVF_INPUT : 0);
  h->nonfinite = nonfinite ? 1 : 0;
  h->max_prefix = 0;
  h->n_leaves = 0;
  // as k_reset_lists, but for the open lists: a first walk by paths needs no launch for it
  h->m2l_cursor = 0;
  h->p2p_cursor = 0;
  h->p2p_pairs = 0;
  h->item_cursor = 0;
  h->part_cursor = 0;
}

__device__ __forceinline__ void root_init(const DevTree &t, int r, int leaf_size) {
  if (r >= t.cap_nodes) return;
  t.nbeg[r] = t.req_off[r];
  t.nend[r] = t.req_off[r + 1];
  t.nlev[r] = 0;
  t.nparent[r] = -1;
  t.nchild0[r] = -1;
  t.nnchild[r] = 0;
  t.nreq[r] = r;
  t.ngeo[r] = cell_geometry(t.box[r], 0ull, 0);
  if (t.req_off[r + 1] - t.req_off[r] <= leaf_size) atomicAdd((int *)&t.hdr->n_leaves, 1);
}

// Box of request r from its blocks' partial boxes, by one wavefront; returns
// whether a position was not finite.
__device__ __forceinline__ bool box_of_request(const DevTree &t, int r) {
  const int lane = threadIdx.x & 63;
  const int b0 = t.blk_off[r], b1 = t.blk_off[r + 1];
  double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  bool bad = false;
  for (int b = b0 + lane; b < b1; b += 64) {
    const double *part = t.bbox_part + (int64_t)b * BBOX_COLS;
    for (int d = 0; d < 3; ++d) {
      lo[d] = fmin(lo[d], part[d]);
      hi[d] = fmax(hi[d], part[3 + d]);
    }
    bad |= part[6] != 0.0;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1)
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      lo[d] = fmin(lo[d], __shfl_xor(lo[d], off, 64));
      hi[d] = fmax(hi[d], __shfl_xor(hi[d], off, 64));
    }
  if (lane == 0) finish_box(t.box[r], lo, hi, t.reqs[r].n == 0);
  return __ballot(bad) != 0ull;
}

// Boxes, header and roots of a batch of few requests, by one workgroup (a
// wavefront per request); batches of more take k_header_init and k_boxes.
#define INIT_WAVES 16
__global__ __launch_bounds__(INIT_WAVES * 64) void k_init(DevTree t, int leaf_size) {
  bool bad = false;
  for (int r = threadIdx.x >> 6; r < t.n_req; r += INIT_WAVES) bad |= box_of_request(t, r);
  const int any = __syncthreads_or(bad);
  if (threadIdx.x == 0) header_init(t, any != 0);
  __syncthreads();
  for (int r = threadIdx.x; r < t.n_req; r += INIT_WAVES * 64) root_init(t, r, leaf_size);
}

__global__ void k_header_init(DevTree t) { header_init(t, false); }

__global__ __launch_bounds__(FMM_BLOCK) void k_boxes(DevTree t, int leaf_size) {
  const int r = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  if (r >= t.n_req) return;
  const bool bad = box_of_request(t, r);
  if ((threadIdx.x & 63) == 0) {
    if (bad) {
      atomicOr(&t.hdr->nonfinite, 1);
      atomicOr(&t.hdr->overflow, OVF_INPUT);
    }
    root_init(t, r, leaf_size);
  }
}

__device__ __forceinline__ int lower_bound_digit(const uint64_t *__restrict__ key, int b, int e,
                                                 int shift, uint32_t oct) {
  while (b < e) {
    int mid = (b + e) >> 1;
    if (((uint32_t)(key[mid] >> shift) & 7u) < oct)
      b = mid + 1;
    else
      e = mid;
  }
  return b;
}

__device__ __forceinline__ void level_chunk(const Header *h, int l, int &s, int &e) {
  int ls = h->lvl_start[l], le = h->lvl_start[l + 1];
  int cnt = le - ls;
  int per = (cnt + gridDim.x - 1) / gridDim.x;
  s = ls + blockIdx.x * per;
  e = min(le, s + per);
}

// children of node i of level l: octant boundaries of its key range into
// bounds[i][0..8), the number of non-empty octants into nnchild[i]
__device__ __forceinline__ int count_node(const DevTree &t, int i, int l, int leaf_size) {
  const int shift = 3 * (FMM_MAXLEVEL - (l + 1));
  int b = t.nbeg[i], en = t.nend[i];
  int nc = 0;
  if (en - b > leaf_size && l < FMM_MAXLEVEL) {
    int bd[9];
    bd[0] = b;
    bd[8] = en;
    for (uint32_t o = 1; o < 8; ++o) bd[o] = lower_bound_digit(t.key, bd[o - 1], en, shift, o);
    for (int o = 0; o < 8; ++o) {
      t.bounds[(int64_t)i * 8 + o] = bd[o];
      nc += bd[o + 1] > bd[o];
    }
  }
  t.nnchild[i] = nc;
  return nc;
}

// emit the nc children of node i (level l) at ids first, first+1, ...;
// returns how many of them are leaves
__device__ __forceinline__ int emit_node(const DevTree &t, int i, int l, int nc, int first,
                                         int leaf_size) {
  if (nc == 0) {
    t.nchild0[i] = -1;
    return 0;
  }
  int leaves = 0;
  t.nchild0[i] = first;
  const int rq = t.nreq[i];
  const Box box = t.box[rq];
  int c = first;
  for (int o = 0; o < 8; ++o) {
    int b = t.bounds[(int64_t)i * 8 + o];
    int en = o < 7 ? t.bounds[(int64_t)i * 8 + o + 1] : t.nend[i];
    if (en > b) {
      if (c < t.cap_nodes) {
        t.nbeg[c] = b;
        t.nend[c] = en;
        t.nlev[c] = l + 1;
        t.nparent[c] = i;
        t.nchild0[c] = -1;
        t.nnchild[c] = 0;
        t.nreq[c] = rq;
        uint64_t prefix = t.key[b] >> (3 * (FMM_MAXLEVEL - (l + 1)));
        t.ngeo[c] = cell_geometry(box, prefix, l + 1);
      }
      leaves += (en - b <= leaf_size || l + 1 == FMM_MAXLEVEL);
      ++c;
    }
  }
  return leaves;
}

// count_node with its searches spread over an aligned group of 8 lanes: lane
// o finds the first particle of octant >= o in the whole key range of the
// cell (its keys are sorted by octant, so this is the bound the sequential
// search finds), and the group counts the non-empty octants.  Same bounds
// and count as count_node.
__device__ __forceinline__ int count_node8(const DevTree &t, int i, int l, int leaf_size, int o) {
  const int shift = 3 * (FMM_MAXLEVEL - (l + 1));
  const int b = t.nbeg[i], en = t.nend[i];
  int nc = 0;
  if (en - b > leaf_size && l < FMM_MAXLEVEL) {
    const int bd = o == 0 ? b : lower_bound_digit(t.key, b, en, shift, (uint32_t)o);
    t.bounds[(int64_t)i * 8 + o] = bd;
    const int nx = __shfl_down(bd, 1, 8);  // lane o + 1's bound (o = 7: its own)
    const bool nonempty = o < 7 ? nx > bd : en > bd;
    const unsigned long long m = __ballot(nonempty);
    nc = __popcll((m >> (__lane_id() & 56)) & 0xFFull);
  }
  if (o == 0) t.nnchild[i] = nc;
  return nc;
}

__global__ __launch_bounds__(FMM_BLOCK) void k_tree_count(DevTree t, int l, int leaf_size) {
  int s, e;
  level_chunk(t.hdr, l, s, e);
  const int o = threadIdx.x & 7;
  int sum = 0;
  for (int i = s + (threadIdx.x >> 3); i < e && i < t.cap_nodes; i += blockDim.x >> 3) {
    const int nc = count_node8(t, i, l, leaf_size, o);
    if (o == 0) sum += nc;
  }
  __shared__ int red[FMM_BLOCK];
  red[threadIdx.x] = sum;
  __syncthreads();
  for (int o = FMM_BLOCK / 2; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) t.scan_part[blockIdx.x] = red[0];
}


// Sum of v over a block of FMM_BLOCK threads (all of them call it).
__device__ __forceinline__ int block_sum(int v, int *part) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
  __syncthreads();
  int tot = 0;
#pragma unroll
  for (int w = 0; w < FMM_BLOCK / 64; ++w) tot += part[w];
  __syncthreads();
  return tot;
}

// Children of the splitting cells of level l; a child is a leaf when it holds
// at most leaf_size particles or sits at the deepest level, and leaves are
// counted here.  Each block first takes its offset among the children of the level (the
// child counts of the earlier blocks, from k_tree_count) and the level's
// total; block 0 records where the next level ends.
__global__ __launch_bounds__(FMM_BLOCK) void k_tree_emit(DevTree t, int l, int leaf_size) {
  static_assert(FMM_SCAN_BLOCKS == FMM_BLOCK, "one block count per thread");
  int s, e;
  level_chunk(t.hdr, l, s, e);
  __shared__ int sc[FMM_BLOCK];
  __shared__ int part[FMM_BLOCK / 64];
  const int cnt = t.scan_part[threadIdx.x];
  const int before = block_sum((int)threadIdx.x < (int)blockIdx.x ? cnt : 0, part);
  const int level_total = block_sum(cnt, part);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    Header *h = t.hdr;
    const int next = h->lvl_start[l + 1] + level_total;
    for (int k = l + 2; k < FMM_NLEVELS + 2; ++k) h->lvl_start[k] = next;
    if (next > t.cap_nodes) h->overflow |= OVF_NODES;
  }
  int run = t.hdr->lvl_start[l + 1] + before;
  for (int base = s; base < e; base += FMM_BLOCK) {
    int i = base + threadIdx.x;
    int nc = (i < e && i < t.cap_nodes) ? t.nnchild[i] : 0;
    sc[threadIdx.x] = nc;
    __syncthreads();
    for (int off = 1; off < FMM_BLOCK; off <<= 1) {
      int y = threadIdx.x >= off ? sc[threadIdx.x - off] : 0;
      __syncthreads();
      sc[threadIdx.x] += y;
      __syncthreads();
    }
    int first = run + sc[threadIdx.x] - nc;
    int total = sc[FMM_BLOCK - 1];
    __syncthreads();
    int leaves = 0;
    if (i < e && i < t.cap_nodes) leaves = emit_node(t, i, l, nc, first, leaf_size);
    if (leaves) atomicAdd((int *)&t.hdr->n_leaves, leaves);
    run += total;
  }
}

// ---------------------------------------------------------------------------
// Every split level at once (leaf_size <= TD_MAXLEAF): a fixed number of
// launches whatever the depth, and no host read of the split depth first.
//
// The cell of level l that holds sorted particle i (a run of keys sharing
// their first l octal digits) holds more than L = leaf_size particles exactly
// when some k in [i - L, i] of the same system has keys k and k + L sharing
// those digits (then k .. k + L, which contains i, lies in the run; and a run
// of more than L particles contains such a window around any of its
// particles).  With c(k) the common leading levels of keys k and k + L, the
// cells along i's path are split at levels 0 .. m, m the largest c(k) over
// that window, and i's leaf is at level d(i) = m + 1 (0 when no window fits
// in the system; at most FMM_MAXLEVEL).  A cell of level l >= 1 exists when
// its parent is split, i.e. l <= d(i) for its particles, and particle i
// starts one at every level l from cp(i) + 1 to d(i), cp(i) the common
// levels of keys i - 1 and i (0 at the first particle of a system); it ends
// the run of every level l from cp(i + 1) + 1 (0 at the system's last
// particle) to d(i).  Nodes are numbered level by level, in sorted order
// within a level, as the level-by-level split numbers them, so the two build
// the same tree bit for bit.
// ---------------------------------------------------------------------------
#define TD_THREADS 1024
#define TD_WAVES (TD_THREADS / 64)
#define TD_MAXLEAF 1024

__device__ __forceinline__ int common_levels(uint64_t a, uint64_t b) {
  const uint64_t x = a ^ b;
  return x == 0 ? FMM_MAXLEVEL : (__clzll(x) - 1) / 3;
}

// per-particle level data, packed: d | lo << 8 | lo2 << 16 (lo: first level
// >= 1 at which i starts a cell; lo2: first level at which i ends a run)
__device__ __forceinline__ void td_unpack(uint64_t v, int &d, int &lo, int &lo2) {
  d = (int)(v & 255u);
  lo = (int)((v >> 8) & 255u);
  lo2 = (int)((v >> 16) & 255u);
}

struct LevelLds {
  int cw[TD_THREADS + TD_MAXLEAF];  // c over [b0 - L, b0 + TD_THREADS), then window maxima
  int wcnt[TD_WAVES][FMM_MAXLEVEL];
  int wmax[TD_WAVES];
};

// Block blk of TD_THREADS sorted particles: d, lo, lo2 of each into key2, per
// level l >= 1 the number of cells of level l that start in the block into
// hist[(l - 1) * nblk + blk], and the split depth into the header.  The
// maximum over a window of L + 1 values comes from two overlapping windows of
// the largest power of two within it, formed by doubling in LDS.
__device__ __forceinline__ void tree_levels(const DevTree &t, int n, int L, int blk, int nblk,
                                            uint32_t *hist, LevelLds &S) {
  const int b0 = blk * TD_THREADS, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  for (int k = tid; k < TD_THREADS + L; k += TD_THREADS) {
    const int g = b0 - L + k;
    int c = -1;
    if (g >= 0 && g < n) {
      const int r = t.n_req > 1 ? upper_index(t.req_off, t.n_req, g) : 0;
      if (g + L < t.req_off[r + 1]) c = common_levels(t.key[g], t.key[g + L]);
    }
    S.cw[k] = c;
  }
  __syncthreads();
  int best = S.cw[L + tid];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) best = max(best, __shfl_xor(best, off, 64));
  if (lane == 0) S.wmax[w] = best;
  int span = 1;
  for (; 2 * span <= L + 1; span *= 2) {
    const int k1 = tid + TD_THREADS;
    const int v0 = max(S.cw[tid], S.cw[min(tid + span, TD_THREADS + L - 1)]);
    const int v1 = k1 < TD_THREADS + L ? max(S.cw[k1], S.cw[min(k1 + span, TD_THREADS + L - 1)]) : 0;
    __syncthreads();
    S.cw[tid] = v0;
    if (k1 < TD_THREADS + L) S.cw[k1] = v1;
    __syncthreads();
  }
  const int i = b0 + tid;
  int lo = 1, hi = 0;
  if (i < n) {
    const int r = t.n_req > 1 ? upper_index(t.req_off, t.n_req, i) : 0;
    const int rs = t.req_off[r], re = t.req_off[r + 1];
    // windows that start before the system do not fit in their own and hold -1
    const int m = max(S.cw[tid], S.cw[tid + L + 1 - span]);
    const int d = m < 0 ? 0 : min(FMM_MAXLEVEL, m + 1);
    const int cpi = i == rs ? 0 : common_levels(t.key[i - 1], t.key[i]);
    const int lo2 = i + 1 == re ? 0 : common_levels(t.key[i], t.key[i + 1]) + 1;
    lo = cpi + 1;
    hi = d;
    t.key2[i] = (uint64_t)d | ((uint64_t)lo << 8) | ((uint64_t)lo2 << 16);
  }
  for (int l = 1; l <= FMM_MAXLEVEL; ++l) {
    const unsigned long long b = __ballot(lo <= l && l <= hi);
    if (lane == 0) S.wcnt[w][l - 1] = __popcll(b);
  }
  __syncthreads();
  if (tid < FMM_MAXLEVEL) {
    int s = 0;
    for (int ww = 0; ww < TD_WAVES; ++ww) s += S.wcnt[ww][tid];
    hist[(size_t)tid * nblk + blk] = (uint32_t)s;
  }
  if (tid == 64) {
    for (int ww = 0; ww < TD_WAVES; ++ww) best = max(best, S.wmax[ww]);
    if (best > 0) atomicMax(&t.hdr->max_prefix, best);
  }
}

__global__ __launch_bounds__(TD_THREADS) void k_tree_levels(DevTree t, int n, int L, int nblk,
                                                            uint32_t *hist) {
  __shared__ LevelLds lds;
  tree_levels(t, n, L, blockIdx.x, nblk, hist, lds);
}

struct NodeLds {
  int wpre[TD_WAVES][FMM_MAXLEVEL];
  int boff[FMM_MAXLEVEL], btot[FMM_MAXLEVEL];
  int lvs[FMM_NLEVELS + 2];
  int leaves[TD_WAVES];
};

// The nodes of levels >= 1 that block blk's particles start, and the children
// of the roots.  tot = NULL (at most 64 blocks): hist holds the blocks' cells
// per level and the block adds up those before it; otherwise hist holds, per
// level, each block's exclusive offset among the level's cells, tot the level
// totals.  A split cell's child count is written first as the end of its
// children (by the particle that ends the cell) and turned into a count by
// k_node_info.
__device__ __forceinline__ void tree_nodes(const DevTree &t, int n, int blk, int nblk,
                                           const uint32_t *hist, const uint32_t *tot,
                                           int walk_levels, NodeLds &S) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if (tot) {
    if (tid < FMM_MAXLEVEL) {
      S.boff[tid] = (int)hist[(size_t)tid * nblk + blk];
      S.btot[tid] = (int)tot[tid];
    }
  } else {
    for (int l = w; l < FMM_MAXLEVEL; l += TD_WAVES) {
      const int v = lane < nblk ? (int)hist[(size_t)l * nblk + lane] : 0;
      const int all = wave_sum(v), before = wave_sum(lane < blk ? v : 0);
      if (lane == 0) {
        S.boff[l] = before;
        S.btot[l] = all;
      }
    }
  }
  const int i = blk * TD_THREADS + tid;
  int d = 0, lo = 1, lo2 = FMM_MAXLEVEL + 1, r = 0;
  uint64_t key = 0;
  if (i < n) {
    td_unpack(t.key2[i], d, lo, lo2);
    r = t.n_req > 1 ? upper_index(t.req_off, t.n_req, i) : 0;
    key = t.key[i];
  }
  const int hi = i < n ? d : 0;
  const unsigned long long below = lanes_below_mask();
  int rank[FMM_MAXLEVEL + 2];  // exclusive rank among the level's cell starts, levels 1..
#pragma unroll
  for (int l = 1; l <= FMM_MAXLEVEL; ++l) {
    const unsigned long long b = __ballot(lo <= l && l <= hi);
    rank[l] = __popcll(b & below);
    if (lane == 0) S.wpre[w][l - 1] = __popcll(b);
  }
  rank[0] = rank[FMM_MAXLEVEL + 1] = 0;
  __syncthreads();
  if (tid < FMM_MAXLEVEL) {  // exclusive prefix over the waves and the blocks before, in place
    int run = S.boff[tid];
    for (int ww = 0; ww < TD_WAVES; ++ww) {
      const int c = S.wpre[ww][tid];
      S.wpre[ww][tid] = run;
      run += c;
    }
  }
  if (tid == 64) {
    int at = t.n_req;
    S.lvs[0] = 0;
    S.lvs[1] = at;
    for (int l = 1; l <= FMM_NLEVELS; ++l) {
      at += l <= FMM_MAXLEVEL ? S.btot[l - 1] : 0;
      S.lvs[l + 1] = at;
    }
  }
  __syncthreads();
  const int64_t cap = t.cap_nodes;
  int leaves = 0;
  if (i < n) {
    const Box box = t.box[r];
#pragma unroll
    for (int l = 1; l <= FMM_MAXLEVEL; ++l) rank[l] += S.wpre[w][l - 1];
    // the root's children start at the system's first particle, its run ends at the last
    if (lo == 1 && i == t.req_off[r] && d > 0 && r < cap) t.nchild0[r] = S.lvs[1] + rank[1];
    if (lo2 == 0 && d > 0 && r < cap) t.nnchild[r] = S.lvs[1] + rank[1] + (lo <= 1 ? 1 : 0);
#pragma unroll
    for (int l = 1; l <= FMM_MAXLEVEL; ++l) {
      const bool starts = lo <= l && l <= hi, ends = lo2 <= l && l <= hi;
      if (!starts && !ends) continue;
      const bool split = l < d;
      if (starts) {  // a cell starts at i
        const int64_t k = (int64_t)S.lvs[l] + rank[l];
        leaves += !split;
        if (k < cap) {
          const bool ps = lo <= l - 1;  // i also starts its parent
          t.nbeg[k] = i;
          t.nlev[k] = l;
          t.nparent[k] = l == 1 ? r : S.lvs[l - 1] + rank[l - 1] + (ps ? 1 : 0) - 1;
          t.nchild0[k] = split ? S.lvs[l + 1] + rank[l + 1] : -1;
          if (!split) t.nnchild[k] = 0;
          t.nreq[k] = r;
          t.ngeo[k] = cell_geometry(box, key >> (3 * (FMM_MAXLEVEL - l)), l);
        }
      }
      if (ends) {  // a run ends at i
        const int64_t k = (int64_t)S.lvs[l] + rank[l] + (lo <= l ? 1 : 0) - 1;
        if (k < cap) {
          t.nend[k] = i + 1;
          if (split) t.nnchild[k] = S.lvs[l + 1] + rank[l + 1] + (lo <= l + 1 ? 1 : 0);
        }
      }
    }
  }
  leaves = wave_sum(leaves);
  if (lane == 0) S.leaves[w] = leaves;
  __syncthreads();
  if (tid == 0) {
    int s = 0;
    for (int ww = 0; ww < TD_WAVES; ++ww) s += S.leaves[ww];
    if (s) atomicAdd((int *)&t.hdr->n_leaves, s);
    if (blk == 0) {
      Header *h = t.hdr;
      for (int l = 0; l < FMM_NLEVELS + 2; ++l) h->lvl_start[l] = S.lvs[l];
      if (S.lvs[FMM_NLEVELS + 1] > cap) h->overflow |= OVF_NODES;
      int deepest = 0;
      for (int l = 1; l <= FMM_MAXLEVEL; ++l)
        if (S.lvs[l + 1] > S.lvs[l]) deepest = l;
      if (deepest > walk_levels) h->overflow |= OVF_DEPTH;
    }
  }
}

__global__ __launch_bounds__(TD_THREADS) void k_tree_nodes(DevTree t, int n, int nblk,
                                                           const uint32_t *hist,
                                                           const uint32_t *tot, int walk_levels) {
  __shared__ NodeLds lds;
  tree_nodes(t, n, blockIdx.x, nblk, hist, tot, walk_levels, lds);
}

// Walk record of cell k; turn_counts: nnchild of a split cell still holds
// the end of its children (tree_nodes) and becomes a count first.
__device__ __forceinline__ void node_info(const DevTree &t, int k, bool turn_counts) {
  const int c0 = t.nchild0[k];
  int nc = t.nnchild[k];
  if (turn_counts && c0 >= 0) {
    nc -= c0;
    t.nnchild[k] = nc;
  }
  t.ninfo[k] = make_int4(c0, nc, t.nbeg[k], t.nend[k]);
}

__global__ __launch_bounds__(FMM_BLOCK) void k_node_info(DevTree t, bool turn_counts) {
  const int total = min(t.hdr->lvl_start[FMM_NLEVELS + 1], (int)t.cap_nodes);
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < total; k += gridDim.x * blockDim.x)
    node_info(t, k, turn_counts);
}

// ---------------------------------------------------------------------------
// Small batches (at most SMALL_N active particles in all): the whole build up
// to the walk -- boxes, roots, keys, sort, sorted positions and every split
// level -- in one workgroup, one launch, with no host round trip: the steps of
// the multi-workgroup build on one tile and one block, so the tree is the same
// bit for bit.  1,000 particles: 155 -> 33 us (the split level by level
// and a radix sort of 8 wavefronts before).
// ---------------------------------------------------------------------------
static_assert(SMALL_N == MSORT_TILE && SMALL_N == TD_THREADS, "one tile, one block");

__global__ __launch_bounds__(SMALL_N) void k_build_small(DevTree t, int n, int leaf_size) {
  __shared__ union {
    TileLds tile;
    LevelLds level;
    NodeLds node;
  } lds;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  bool bad = false;
  for (int r = w; r < t.n_req; r += SMALL_N / 64) {  // root boxes: a wavefront per request
    const DevReq q = t.reqs[r];
    double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int i = lane; i < q.n; i += 64) {
      const int64_t g = q.active ? q.active[i] : i;
      for (int d = 0; d < 3; ++d) {
        const double x = q.pos[d * q.n_total + g];
        bad |= !isfinite(x);
        lo[d] = fmin(lo[d], x);
        hi[d] = fmax(hi[d], x);
      }
    }
    for (int off = 32; off > 0; off >>= 1)
      for (int d = 0; d < 3; ++d) {
        lo[d] = fmin(lo[d], __shfl_xor(lo[d], off, 64));
        hi[d] = fmax(hi[d], __shfl_xor(hi[d], off, 64));
      }
    if (lane == 0) finish_box(t.box[r], lo, hi, q.n == 0);
  }
  const int any = __syncthreads_or(bad);
  if (tid == 0) header_init(t, any != 0);
  __syncthreads();
  for (int r = tid; r < t.n_req; r += SMALL_N) root_init(t, r, leaf_size);
  sort_tile(t, n, 0, t.key, t.slot, true, lds.tile);
  __syncthreads();
  if (leaf_size >= n) {  // no cell is split: every window would reach past its system
    const int roots = min(t.n_req, (int)t.cap_nodes);  // empty systems have a root too
    for (int r = tid; r < roots; r += SMALL_N) node_info(t, r, true);
    return;
  }
  tree_levels(t, n, leaf_size, 0, 1, t.sort_hist, lds.level);
  __syncthreads();
  tree_nodes(t, n, 0, 1, t.sort_hist, nullptr, FMM_MAXLEVEL, lds.node);
  __syncthreads();
  const int total = min(lds.node.lvs[FMM_NLEVELS + 1], (int)t.cap_nodes);
  for (int k = tid; k < total; k += SMALL_N) node_info(t, k, true);
}

hipError_t launch_build_small(const DevTree &t, const BuildArgs &a, hipStream_t s) {
  if (a.tm) a.tm->start(PH_TREE, s);
  hipLaunchKernelGGL(k_build_small, dim3(1), dim3(SMALL_N), 0, s, t, a.n, a.leaf_size);
  if (a.tm) a.tm->stop(s);
  return hipGetLastError();
}

// Boxes, header, roots, keys, sort by (system, key, slot) and sorted positions.
hipError_t launch_sort(const DevTree &t, const BuildArgs &a, hipStream_t s) {
  const int n = a.n;
  const int nb = (n + FMM_BLOCK - 1) / FMM_BLOCK;
  if (a.tm) a.tm->start(PH_SORT, s);
  hipLaunchKernelGGL(k_bbox_partial, dim3(a.n_blk), dim3(FMM_BLOCK), 0, s, t);
  if (a.n_req <= INIT_WAVES) {
    hipLaunchKernelGGL(k_init, dim3(1), dim3(INIT_WAVES * 64), 0, s, t, a.leaf_size);
  } else {
    hipLaunchKernelGGL(k_header_init, dim3(1), dim3(1), 0, s, t);
    hipLaunchKernelGGL(k_boxes, dim3((a.n_req + 3) / 4), dim3(FMM_BLOCK), 0, s, t, a.leaf_size);
  }
  const int merges = sort_merges(n, a.n_max, a.n_req);
  if (n > 0 && merges >= 0) {
    // the result always lands in key / slot
    uint64_t *k0 = merges & 1 ? t.key2 : t.key, *k1 = merges & 1 ? t.key : t.key2;
    int32_t *s0 = merges & 1 ? t.slot2 : t.slot, *s1 = merges & 1 ? t.slot : t.slot2;
    hipLaunchKernelGGL(k_sort_tiles, dim3((n + MSORT_TILE - 1) / MSORT_TILE), dim3(MSORT_TILE), 0,
                       s, t, n, k0, s0, merges == 0);
    int R = MSORT_TILE;
    for (int m = 0; m < merges; ++m, R *= MSORT_FAN) {
      hipLaunchKernelGGL(k_sort_merge, dim3(nb), dim3(FMM_BLOCK), 0, s, t, n, R, k0, s0, k1, s1,
                         m + 1 == merges);
      std::swap(k0, k1);
      std::swap(s0, s1);
    }
  } else if (n > 0) {
    const int nblk = (n + SORT_TILE - 1) / SORT_TILE;
    // 8 passes over the 63-bit key, then (several requests) one pass per byte
    // of the largest request id; with an odd number of passes the keys start
    // in key2 / slot2, so that the result always lands in key / slot
    int req_passes = 0;
    if (a.n_req > 1) {
      req_passes = a.n_req > 65536 ? 4 : (a.n_req > 256 ? 2 : 1);
      hipLaunchKernelGGL(k_slot_req, dim3(nb), dim3(FMM_BLOCK), 0, s, t, n);
    }
    const int passes = 8 + req_passes;
    const int odd = passes & 1;
    hipLaunchKernelGGL(k_keys, dim3(nb), dim3(FMM_BLOCK), 0, s, t, n, odd);
    uint64_t *kin = odd ? t.key2 : t.key, *kout = odd ? t.key : t.key2;
    int32_t *sin = odd ? t.slot2 : t.slot, *sout = odd ? t.slot : t.slot2;
    for (int pass = 0; pass < passes; ++pass) {
      const int by_req = pass >= 8;
      const int shift = by_req ? (pass - 8) * 8 : pass * 8;
      hipLaunchKernelGGL(k_sort_hist, dim3(nblk), dim3(SORT_THREADS), 0, s, kin, sin, t.slot_req, n,
                         shift, by_req, t.sort_hist, nblk);
      hipLaunchKernelGGL(k_sort_digit_scan, dim3(256), dim3(FMM_BLOCK), 0, s, t.sort_hist, nblk,
                         t.sort_dtot);
      hipLaunchKernelGGL(k_sort_scatter, dim3(nblk), dim3(SORT_THREADS), 0, s, kin, sin, kout, sout,
                         t.slot_req, n, shift, by_req, t.sort_hist, nblk, t.sort_dtot);
      std::swap(kin, kout);
      std::swap(sin, sout);
    }
    hipLaunchKernelGGL(k_gather_sorted, dim3(nb), dim3(FMM_BLOCK), 0, s, t, n);
  }
  if (n > 0 && !build_tree_direct_ok(a.leaf_size))
    hipLaunchKernelGGL(k_split_depth, dim3(std::min(nb, 512)), dim3(FMM_BLOCK), 0, s, t, n,
                       a.leaf_size);
  if (a.tm) a.tm->stop(s);
  return hipGetLastError();
}

// Every level at once (see tree_levels); false when leaf_size is beyond the
// window that fits in LDS (then launch_build_tree builds level by level).
bool build_tree_direct_ok(int leaf_size) { return leaf_size >= 1 && leaf_size <= TD_MAXLEAF; }

// walk_levels: the levels the walk that follows covers (a deeper tree is
// flagged with OVF_DEPTH and not evaluated)
hipError_t launch_build_tree_direct(const DevTree &t, const BuildArgs &a, int walk_levels,
                                    hipStream_t s) {
  const int n = a.n;
  if (a.tm) a.tm->start(PH_TREE, s);
  if (n > 0) {
    const int nblk = (n + TD_THREADS - 1) / TD_THREADS;
    const bool scan = nblk > 64;  // more blocks than a wavefront adds up itself
    hipLaunchKernelGGL(k_tree_levels, dim3(nblk), dim3(TD_THREADS), 0, s, t, n, a.leaf_size, nblk,
                       t.sort_hist);
    if (scan)
      hipLaunchKernelGGL(k_sort_digit_scan, dim3(FMM_MAXLEVEL), dim3(FMM_BLOCK), 0, s, t.sort_hist,
                         nblk, t.sort_dtot);
    hipLaunchKernelGGL(k_tree_nodes, dim3(nblk), dim3(TD_THREADS), 0, s, t, n, nblk, t.sort_hist,
                       scan ? t.sort_dtot : nullptr, walk_levels);
    hipLaunchKernelGGL(k_node_info, dim3(std::min(1024, std::max(1, n / 256))), dim3(FMM_BLOCK), 0,
                       s, t, true);
  }
  if (a.tm) a.tm->stop(s);
  return hipGetLastError();
}

// levels 0 .. max_level-1 are split (cells of level max_level are leaves)
hipError_t launch_build_tree(const DevTree &t, const BuildArgs &a, int max_level, hipStream_t s) {
  const int n = a.n;
  if (a.tm) a.tm->start(PH_TREE, s);
  if (n > 0) {
    for (int l = 0; l < max_level && l < FMM_MAXLEVEL; ++l) {
      hipLaunchKernelGGL(k_tree_count, dim3(FMM_SCAN_BLOCKS), dim3(FMM_BLOCK), 0, s, t, l,
                         a.leaf_size);
      hipLaunchKernelGGL(k_tree_emit, dim3(FMM_SCAN_BLOCKS), dim3(FMM_BLOCK), 0, s, t, l,
                         a.leaf_size);
    }
    hipLaunchKernelGGL(k_node_info, dim3(std::min(1024, std::max(1, n / 256))), dim3(FMM_BLOCK), 0,
                       s, t, false);
  }
  if (a.tm) a.tm->stop(s);
  return hipGetLastError();
}


