// Internal declarations shared by the HIP translation units of libfmm355.
//
// Data layout in HBM (one context, capacities fixed at creation):
//   particles (Morton-sorted order, SoA):  keys u64, slot i32 (active slot of
//     the particle), positions f64 x3, cell-local offsets f32 x3, masses f64 and
//     f32, leaf id i32, near-field (P2P) results f64 x4;
//   nodes (level-major: all level-0 nodes, then level 1, ...; inside a level in
//     Morton order): begin/end/level/parent/first-child/child-count i32,
//     geometry double4 (centre xyz, half side), multipole and local
//     coefficient rows of K = C(p+3,3) reals (node-major);
//   interaction lists: per target node (offset, count) into flat i32 arrays of
//     source node ids (directed entries; the unordered pair {A,B} appears once
//     in A's list and once in B's list).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#define FMM_MAXLEVEL 21
#define FMM_NLEVELS (FMM_MAXLEVEL + 1)
#define FMM_BLOCK 256
#define FMM_SCAN_BLOCKS 256
#define FMM_BBOX_BLOCKS 256  // box-reduction blocks per request, at most
#define FMM_BBOX_COLS 7      // lower, upper corner, non-finite flag of a block
#define SORT_TILE 4096       // keys per radix-sort tile (one histogram column)
// single-workgroup ("small") build and level passes
#define SMALL_N 1024                  // active particles of a batch built in one workgroup
#define SMALL_TREE_LEAVES 400         // batches of at most this many times leaf_size particles
                                      // are queued without reading the tree's size back
#define SMALL_NODES 2048              // cells of a tree whose M2M / L2L levels run in one workgroup

// error bits latched in Header::overflow
#define OVF_NODES 1
#define OVF_M2L 2
#define OVF_P2P 4
#define OVF_OPEN 8
#define OVF_STACK 16
// the tree holds cells deeper than the levels the (predicted) walk covers: the
// cells below them have no lists, so nothing may be evaluated on it
#define OVF_DEPTH 32
// the P2P work items, or the partial sums of split leaves, did not fit
#define OVF_ITEMS 64
// an open list outgrew the walk's path form (the host walks by levels)
#define OVF_PATH 128
// an input position was not finite: what was queued behind the build does nothing
#define OVF_INPUT 256
#define OVF_ANY                                                                            \
  (OVF_NODES | OVF_M2L | OVF_P2P | OVF_OPEN | OVF_STACK | OVF_DEPTH | OVF_ITEMS | OVF_PATH | \
   OVF_INPUT)

// What a queued kernel heeds: only bits that are final when it runs.  The build's
// are final for the upward pass (which runs beside the walk), those of build and
// walk for M2L and L2L (beside the near-field plan), all for what follows the plan.
#define OVF_BUILD (OVF_NODES | OVF_DEPTH | OVF_INPUT)
#define OVF_WALK (OVF_ANY & ~OVF_ITEMS)

struct Header {
  int32_t lvl_start[FMM_NLEVELS + 2];  // nodes of level l: [lvl_start[l], lvl_start[l+1])
  // list entries written (or needed): counted in 64 bits, since lists that do not
  // fit are counted too, and some 50,000 leaves that all list each other already
  // need 2^31 (capacities stay below that: the lists' offsets are int32)
  unsigned long long m2l_cursor;               // ordered M2L entries
  unsigned long long p2p_cursor;               // ordered P2P entries
  unsigned long long open_cursor[FMM_NLEVELS]; // open-list entries per level
  int32_t overflow;                    // OVF_* bits
  int32_t nonfinite;                   // an input position was not finite (OVF_INPUT too)
  unsigned long long p2p_pairs;        // ordered particle interactions in P2P
  int32_t n_leaves;
  int32_t max_prefix;  // deepest level of a cell holding more than leaf_size particles
  uint32_t item_cursor;            // near-field work items of the tree
  unsigned long long part_cursor;  // partial-sum rows of its split leaves
};

// One wavefront's share of the near field: sinks tb .. tb + 63 of leaf A
// against the entries [q0, q1) of its P2P list and, when those are one chunk
// of 64, the windows [w0, w1) of that chunk's source stream.  grp counts the
// leaf's shares; the sums of share 0 go to near[], those of the others to row
// part + (sink of the leaf) of the partial sums.
struct P2PItem {
  int32_t A, tb, q0, q1, w0, w1, grp, part;
};

// Box: o[3] (origin), L (side), s = 2^21/L, lo[3], hi[3]
struct Box {
  double o[3];
  double L;
  double s;
  double lo[3];
  double hi[3];
};

// One independent particle system of a batched solve.  Its active particles
// occupy slots [off, off + n) of the batch; positions/masses are read through
// its own pointers, outputs written to its own acc/pot.
struct DevReq {
  const double *pos;      // 3 x n_total SoA
  const int32_t *active;  // n indices or NULL
  const double *mass;     // n_total
  double *acc;            // 3 x n SoA
  double *pot;            // n
  const uint8_t *sinks;   // n flags, or NULL: every particle is a sink
  int64_t n_total;
  int32_t off;
  int32_t n;
};

struct DevTree {
  // batch of requests (R = 1 for a plain solve)
  DevReq *reqs;       // [cap_req]
  int32_t *req_off;   // [cap_req + 1] slot offsets
  int32_t *blk_off;   // [cap_req + 1] first bbox block of each request
  int32_t *slot_req;  // [cap_n] request of each slot
  int32_t *nreq;      // [cap_nodes] request of each cell
  int n_req;
  int cap_req;
  // particles, sorted order
  uint64_t *key, *key2;
  int32_t *slot, *slot2;
  double *sx, *sy, *sz;
  double *sm;
  float *sm32;
  int32_t *leaf_of;
  double *near;  // [4][cap_n]: ax, ay, az, pot
  double4 *pak;  // [cap_n] positions packed per active slot by the key pass, so
                 // that the sorted gather reads one 32-byte record per particle
  // nodes
  int32_t *nbeg, *nend, *nlev, *nparent, *nchild0, *nnchild;
  double4 *ngeo;
  int4 *ninfo;  // first child (-1: leaf), child count, begin, end: what the walk
                // reads of a candidate beside its geometry, in one load
  int32_t *bounds;  // [cap_nodes][8]
  void *M, *L;      // [cap_nodes][Kmax] of float or double
  void *Mh;         // [cap_nodes][KHmax]: moments folded onto z-degree <= 1 (harmonic far field)
  // lists
  int32_t *m2l_off, *m2l_cnt, *m2l_src;
  int32_t *p2p_off, *p2p_cnt, *p2p_src;
  int32_t *open_off, *open_cnt;
  int32_t *open_buf0, *open_buf1;
  // near-field work items (k_p2p_plan) and the partial sums of split leaves:
  // shares 1 .. nshare of leaf A at rows part_off[A] + (share - 1) * (its
  // particles) + sink
  P2PItem *items;                // [cap_items]
  int32_t *nshare, *part_off;    // [cap_nodes]
  double4 *part;                 // [cap_part] ax, ay, az, pot
  // scratch
  int32_t *scan_part;          // [FMM_SCAN_BLOCKS]
  double *bbox_part;           // [bbox blocks][FMM_BBOX_COLS]
  uint32_t *sort_hist;         // [256][sort blocks]
  uint32_t *sort_dtot;         // [256] digit totals
  uint32_t *scan_blk;          // block sums of the generic scan
  Header *hdr;
  Box *box;  // [cap_req]
  int64_t cap_n, cap_nodes, cap_m2l, cap_p2p, cap_open, cap_items, cap_part;
  int p2p_src_window;  // sources of one staged P2P window (by precision)
  int uncut;  // no list is cut into shares: there was no memory for the partial sums
  int kmax, khmax;
};

// ---------------------------------------------------------------------------
// wavefront helpers (wave64)
// ---------------------------------------------------------------------------
// largest r in [0, m) with off[r] <= x (request of a slot, or of a sorted
// position: both lie in the request's [off[r], off[r + 1]))
__device__ __forceinline__ int upper_index(const int32_t *off, int m, int x) {
  int lo = 0, hi = m - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (off[mid] <= x)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

__device__ __forceinline__ int lane_id() { return __lane_id(); }

__device__ __forceinline__ unsigned long long lanes_below_mask() {
  int l = __lane_id();
  return l == 0 ? 0ull : (~0ull >> (64 - l));
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Workgroups are dealt to the 8 XCDs (each with its own L2) round-robin in
// blockIdx order.  xcd_block maps blockIdx to a logical block index so that
// each XCD runs chunks of C consecutive logical blocks (the chunks themselves
// dealt round-robin): neighbouring cells, which share most of their sources,
// meet in one L2, while every XCD still gets a mix of the whole range.  A
// bijection on [0, G): the blocks past the last whole round of 8 C keep their
// index.
#define FMM_XCDS 8
template <int C>
__device__ __forceinline__ int xcd_block(int b, int G) {
  const int full = G / (FMM_XCDS * C) * (FMM_XCDS * C);
  if (b >= full) return b;
  const int x = b % FMM_XCDS, k = b / FMM_XCDS;
  return ((k / C) * FMM_XCDS + x) * C + k % C;
}

// Exclusive prefix sum over the wavefront (all 64 lanes active): within each row
// of 16 lanes by row shifts, then lane 15 of rows 0 and 2 into the next row and
// lane 31 into the upper half.  DPP moves: no LDS round trips (six lane
// permutes had made this the longest step of a walk round beside its loads).
__device__ __forceinline__ int wave_excl_scan_int(int v, int *total) {
  int x = v;
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false);  // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false);  // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false);  // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false);  // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);  // row_bcast:15
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);  // row_bcast:31
  *total = __builtin_amdgcn_readlane(x, 63);
  return x - v;
}

// v of a lane, the same in every lane
__device__ __forceinline__ unsigned long long readlane_u64(unsigned long long v, int lane) {
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), lane);
  return (unsigned long long)hi << 32 | lo;
}

// ---------------------------------------------------------------------------
// per-phase HIP-event timing on the context's stream (off unless enabled)
// ---------------------------------------------------------------------------
enum {
  PH_SORT = 0,   // root box, keys, radix sort, sorted gather
  PH_TREE = 1,   // level-by-level split, leaf marking
  PH_WALK = 2,   // symmetric dual walk
  PH_UP = 3,     // mass gather, P2M, M2M
  PH_M2L = 4,
  PH_P2P = 5,
  PH_DOWN = 6,   // L2L, L2P
  PH_N = 7
};

struct PhaseTimer {
  static const int CAP = 512;
  bool on = false;
  bool ready = false;
  unsigned mask = ~0u;  // phases recorded (bit p for phase p)
  hipEvent_t a[CAP], b[CAP];
  int ph[CAP];
  int n = 0, cur = -1;
  double ms[PH_N] = {0};
  long long cnt[PH_N] = {0};
  // an interval of phase p on stream s (intervals on different streams may overlap)
  int begin(int p, hipStream_t s) {
    if (!on || !(mask >> p & 1u)) return -1;
    if (n == CAP) flush();
    hipEventRecord(a[n], s);
    ph[n] = p;
    return n++;
  }
  void end(int k, hipStream_t s) {
    if (on && k >= 0) hipEventRecord(b[k], s);
  }
  void start(int p, hipStream_t s) { cur = begin(p, s); }
  void stop(hipStream_t s) {
    end(cur, s);
    cur = -1;
  }
  void flush() {
    for (int i = 0; i < n; ++i) {
      float t = 0.f;
      hipEventSynchronize(b[i]);
      hipEventElapsedTime(&t, a[i], b[i]);
      ms[ph[i]] += t;
      cnt[ph[i]] += 1;
    }
    n = 0;
  }
};

// ---------------------------------------------------------------------------
// host-side launchers (one translation unit each)
// ---------------------------------------------------------------------------
struct BuildArgs {
  int n;          // active particles over all requests
  int n_max;      // most active particles of one request
  int n_req;      // requests (roots)
  int n_blk;      // bbox blocks over all requests
  int leaf_size;
  double eps;
  double theta;
  PhaseTimer *tm;
  const int32_t *lvl_host;  // level starts of the built tree (host copy), for the walk
  int depth;
};

// tree.hip
#define MSORT_TILE 1024  // slots of a tile of the merge sort
#define MSORT_FAN 16     // runs merged at a time
// Merges of the merge sort over a batch of n particles in n_req systems, the largest
// of n_max: until a run holds the largest system (one system starts at slot 0,
// others anywhere in a tile).  -1: the radix sort is the faster.  A merge reads 15
// searches a key, so what it costs grows with n and with the runs it joins; the
// radix passes are 27 launches that 500,000 keys do not fill.  `full`: merges
// without the one that joins two runs only, for systems that start within a tile.
// Sort of a build, us, merge and radix, in systems of the size given:
//   1: 4.2 M in 3,000 467 and 765, 16.8 M in 10,007 2505 and 3169, in 16,384 2647
//      and 3491;
//   2: 0.5 M in 131,072 143 and 193, 1.05 M 233 and 224, 4.2 M 895 and 676; 0.5 M
//      in 262,144 179 and 191, 1.05 M 301 and 223;
//   3: one of 300,007 146 and 153, 393,216 160 and 161, 430,000 185 and 162.
static inline int sort_merges(int n, int n_max, int n_req) {
  const int64_t reach = n_req == 1 ? n : (int64_t)n_max + MSORT_TILE - 1;
  int merges = 0, full = 0;
  for (int64_t R = MSORT_TILE; R < reach; R *= MSORT_FAN) {
    ++merges;
    full += R < n_max;
  }
  const int most = full <= 1 ? INT32_MAX
                   : full == 2 ? (n_max <= 131072 ? 917504 : 589824)
                   : full == 3 ? 393216 : 0;
  return n <= most ? merges : -1;
}
hipError_t launch_sort(const DevTree &t, const BuildArgs &a, hipStream_t s);
// whole build up to the walk in one workgroup (a.n <= SMALL_N)
hipError_t launch_build_small(const DevTree &t, const BuildArgs &a, hipStream_t s);
hipError_t launch_build_tree(const DevTree &t, const BuildArgs &a, int max_level, hipStream_t s);
// every split level in a fixed number of launches (no host read of the split
// depth first); only for leaf sizes up to the window kept in LDS
bool build_tree_direct_ok(int leaf_size);
hipError_t launch_build_tree_direct(const DevTree &t, const BuildArgs &a, int walk_levels,
                                    hipStream_t s);
// traverse.hip
hipError_t launch_traverse(const DevTree &t, const BuildArgs &a, hipStream_t s);
// levels 0..levels, level bounds read on the device (tree sizes not yet known)
hipError_t launch_traverse_dev(const DevTree &t, const BuildArgs &a, int levels, hipStream_t s);
// Trees of at most this many split cells are walked in the path form: at 1,590
// it took 175 us against some 280 by levels, at 2,769 (2^20 sphere) a
// workgroup per group takes longer than the wavefront form's 168.  Where between
// the two sizes the forms cross has not been measured.
#define WALK_PATH_GROUPS 1600
// Whether a tree of n particles, not yet built, is expected to have that few split
// cells: those of the last tree (of last_n) in proportion.
static inline bool walk_paths_expected(int64_t last_groups, int64_t last_n, int64_t n) {
  return last_n > 0 && (last_groups + 1) * n <= (int64_t)WALK_PATH_GROUPS * last_n;
}
#define PATH_HOLD 32  // builds that walk by levels after a path walk failed
// the whole walk in one launch (trees of few split cells), sizes read on the
// device; flags OVF_PATH when an open list is too long for it
hipError_t launch_traverse_paths(const DevTree &t, const BuildArgs &a, int cells, bool first,
                                 hipStream_t s);
hipError_t launch_reset_lists(const DevTree &t, hipStream_t s);
// near-field work items of the walk's lists: needed by P2P and L2P only
hipError_t launch_p2p_plan(const DevTree &t, const BuildArgs &a, hipStream_t s);
// eval.hip
struct EvalArgs {
  hipStream_t side;         // P2P runs here, concurrently with the multipole passes
  hipEvent_t fork, join;
  int n;
  int n_nodes;
  int p;
  int kernel;     // 0 Wendland, 1 Plummer
  int mixed;      // 0 FP64, 1 mixed
  double eps;
  const int32_t *lvl_start_host;  // host copy, FMM_NLEVELS+1 entries
  int depth;
  PhaseTimer *tm;
  // queued before the host read the tree header: n_nodes, lvl_start_host and
  // depth are estimates (grid sizes, loop bounds) and the kernels take the
  // tree's sizes from the header
  bool dev;
  // with dev: n_nodes, lvl_start_host and depth are the tree's exact sizes (the
  // tree is final, only the lists may have overflowed): grids are exact, and
  // the kernels still take the sizes from the header and skip an overflowed build
  bool exact;
  // mass gather, P2M and M2M already queued by launch_upward (on the side
  // stream, beside the walk); the main stream waits for up_done before M2L
  bool upward_done;
  hipEvent_t up_done;
  // a tree of unknown but small size: M2M and L2L in one workgroup each, the
  // levels read on the device
  bool small_tree;
  // queued behind the walk: the side stream plans the near field of this build
  // before P2P and copies the header to pin_hdr (hdr_ev), so that neither
  // delays the multipole passes
  const BuildArgs *plan;
  Header *pin_hdr;
  hipEvent_t hdr_ev;
};
hipError_t launch_evaluate(const DevTree &t, const EvalArgs &e, hipStream_t s);
// mass gather, P2M and M2M of an evaluation on stream s (exact tree sizes)
hipError_t launch_upward(const DevTree &t, const EvalArgs &e, hipStream_t s);
bool eval_order_supported(int p);
// Wavefronts for the near-field items of a tree of n particles and some
// n_nodes cells; their number is read on the device: about one to two per leaf
// of a large system, up to one per staged window of a small one of few leaves,
// and one per 64 particles where leaves are larger.  The wavefronts stride over the
// items, so more than GRID_WAVES (a launch holds less than 2^32 threads) are not
// needed, and one without an item costs 0.25 ns (100,000 particles in leaves of 4, 8
// for each of 68,350 cells: P2P 106 -> 219 us).
#define GRID_WAVES (1 << 24)
static inline int p2p_grid_items(int n, int n_nodes) {
  int64_t w = 2 * (int64_t)n_nodes;
  if (n <= 131072) w = n_nodes > 32768 ? n_nodes : n_nodes > 4096 ? 32768 : 8 * (int64_t)n_nodes;
  const int64_t uncut = (int64_t)n / 64 + n_nodes;
  if (w < uncut) w = uncut;
  return (int)(w < 1 ? 1 : w > GRID_WAVES ? GRID_WAVES : w);
}
// sources of one staged P2P window
int p2p_window_sources(bool mixed);
// Most shares of a leaf's near list in a system of n particles.  The lists of a
// concentrated system are long at a few leaves only (at most 39 shares of 12,526
// to 500,000 particles of a Plummer sphere); where the softening makes every pair
// near, all are, and each share of each particle takes a row of partial sums:
// 2^25 rows (1 GiB) in all up to 2^20 particles, 32 a particle beyond.
__host__ __device__ static inline int p2p_share_max(int n) {
  if (n <= 1 << 18) return 128;
  return n >= 1 << 20 ? 32 : (1 << 25) / n;
}
// Source windows of a share in a system of n particles (0: shares of whole chunks):
// small systems have too few leaves to fill the chip, so every window is a share;
// large ones have leaves enough and are cut only where a list is long (disk galaxy
// 2^22: solve 14.4 -> 13.1 ms).  Systems of at most 1024 particles have no list
// longer than a few windows and the multipole passes beside P2P take longer: not
// cut, which needs no look at the sources.
#define P2P_SHARE_FINE_N 524288  // largest system cut by windows
__host__ __device__ static inline int p2p_share_windows(int n) {
  if (n <= SMALL_N || n > P2P_SHARE_FINE_N) return 0;
  return n <= 32768 ? 1 : n <= 131072 ? 2 : 4;
}
// Chunks of 64 list entries in a share of whole chunks: P2P_SHARE_CHUNKS, or where
// g windows of `window` sources make a share, as many as hold them at half full
// leaves.  Two or more (small leaves): the shares are whole chunks then, since a
// share cut at windows ends with its chunk.  Fewer: cut at windows.
#define P2P_SHARE_CHUNKS 4
__host__ __device__ static inline int p2p_leaf_chunks(int g, int window, int leaf_size) {
  return g > 0 ? g * window / (32 * leaf_size) : P2P_SHARE_CHUNKS;
}
// at most share_max shares of a list of cnt entries, of at least `chunks` chunks
__host__ __device__ static inline int p2p_share_chunks(int cnt, int share_max, int chunks) {
  const int all = (cnt + 63) / 64;
  return all <= share_max * chunks ? chunks : (all + share_max - 1) / share_max;
}
// Strides of the cells' rows at maximum degree p, of coefficients and of folded
// moments: even, so that every FP64 row starts on 16 bytes, whatever the order
// evaluated (the staged M2L reads rows in 16-byte units; at p 8 a row holds 165).
static inline int coeff_row(int p) { return ((p + 1) * (p + 2) * (p + 3) / 6 + 1) & ~1; }
static inline int folded_row(int p) { return ((p + 1) * (p + 1) + 1) & ~1; }
// grad.hip: force gradient of one system's n active particles (SoA 6 x n) on
// the tree and local expansions of the evaluation just queued on stream s
hipError_t launch_force_gradient(const DevTree &t, int n_nodes, int n, int p, int kernel,
                                 bool mixed, double eps, double *stage, double *gpart,
                                 double *grad, hipStream_t s);
// vector-source pass (eval.hip): sources m_j v_j on the last build's tree (one
// system), vec SoA 3 x e.n in active order, dv scratch 3 x cap_n doubles;
// the request's acc receives +gradient of their potential, pot the potential
hipError_t launch_dipole(const DevTree &t, const EvalArgs &e, const double *vec, double *dv,
                         hipStream_t s);
// its near field (grad.hip): minus sum_j m_j H(x_i - x_j) v_j over the P2P
// partners into near[0..2], sum_j m_j v_j . grad psi(x_i - x_j) into near[3]
hipError_t launch_p2p_dipole(const DevTree &t, int n_nodes, int n, int kernel, bool mixed,
                             double eps, const double *dv, hipStream_t s);
// hhs.hip
hipError_t launch_gather_mask_mass(const double *mass, const int32_t *sys, int n_sys,
                                   const int32_t *flag_fast, int mask_fast, double *out,
                                   hipStream_t s);
