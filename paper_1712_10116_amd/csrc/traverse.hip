// Symmetric dual tree walk (Sec. 2.3, Algorithm 4 with "open both") on gfx950.
//
// The walk over cell pairs starting from (root, root) visits a pair (A, C)
// and then:  accepts it for M2L if it is well separated; makes it a P2P pair
// if both are leaves; opens the non-leaf cell if exactly one is a leaf; opens
// BOTH cells otherwise.  The rule is symmetric in A and C, so the set of
// visited ordered pairs is closed under swapping and every unordered
// interaction appears in both cells' lists.
//
// Target-centric form used here: a visited pair (A, C) with A not a leaf and
// not accepted is recorded in A's "open" list; the children of A then inherit
// the candidates {children of C} (or C itself if C is a leaf).  A leaf target
// that meets a non-leaf candidate descends into that candidate's children on
// an LDS stack.  The children of one cell (a group) are walked together: they
// share their candidates.  Entries are counted, the lists allocated with one
// atomic each, then the entries written, so each cell's lists are contiguous
// and their content and order are deterministic, and the same in all three
// forms of the walk:
//   path form    the whole walk in one launch, a workgroup per group, for trees
//                of at most WALK_PATH_GROUPS split cells;
//   level form   a launch per level, a workgroup per group, for the levels of
//                larger trees with at most WALK_GROUP_LEVEL groups;
//   wavefront    a launch per level, a wavefront per group, for the others.
// Measured, walk of one solve: 1,000 particles 237 -> 22 us, 12,526 371 -> 57,
// 100,003 117 -> 55, 300,007 (1,590 split cells) 357 -> 175, disk galaxy 2^22
// 2.75 -> 2.04 ms (the wavefront form alone did all of them before).
//
// Well-separation is Eq. (1) with R = half side, plus the softening rule of
// Sec. 2.3, written in IEEE double without contraction:
//   d2 = (dx*dx + dy*dy) + dz*dz,  S = hA + hB,
//   d2*(theta*theta) > S*S  and  d2 > (eps + sqrt(3)*S)^2.
#include <algorithm>

#include "common.h"

#define TRAV_CAND 512   // expanded candidates of one block of 64 open-list entries
#define TRAV_STACK 768  // descent items (target tag in the top 3 bits)
// Room kept free for single-item (depth-first) pops: each pops one item and
// pushes at most its 8 children, one level deeper, so a depth-first run from
// any state grows the stack by at most 7 per level below it.
#define TRAV_RESERVE (7 * (FMM_MAXLEVEL + 1))
#define TRAV_TAG 28

enum { CAT_NONE = 0, CAT_M2L = 1, CAT_P2P = 2, CAT_OPEN = 3, CAT_DEEPEN = 4 };

__device__ __forceinline__ bool well_separated(const double4 a, const double4 b, double th2,
                                               double eps) {
  double dx = a.x - b.x;
  double dy = a.y - b.y;
  double dz = a.z - b.z;
  double d2 = (dx * dx + dy * dy) + dz * dz;
  double S = a.w + b.w;
  bool mac = d2 * th2 > S * S;
  double e = eps + 1.7320508075688772 * S;
  bool sep = d2 > e * e;
  return mac && sep;
}

__device__ __forceinline__ int classify(int A, const double4 &gA, bool leafA, int C,
                                        const double4 &gC, bool leafC, double th2, double eps) {
  if (C == A) return leafA ? CAT_P2P : CAT_OPEN;
  if (well_separated(gA, gC, th2, eps)) return CAT_M2L;
  if (leafA) return leafC ? CAT_P2P : CAT_DEEPEN;
  return CAT_OPEN;
}

// A group (the children of one cell, the targets, at most 8) is walked by a
// workgroup of 8 wavefronts, wavefront w deciding for target w.  The candidates
// of 64 open-list entries (at most 512) are loaded once, a chunk of 64 by each
// wavefront, and shared through LDS; a target's categories stay in registers
// until its lists are allocated, so the usual group (one block of candidates,
// no long descents) reads and classifies everything once.  One wavefront per
// group had done all 8 targets in turn, twice (count, then write): 25 us for
// a level however few its groups, nearly all of it instruction latency.
//
// Leaf targets' descents go through one LDS stack for the whole group, LIFO in
// batches of up to 64 items whose children (again at most 512) are a chunk per
// wavefront.  Entries take their places in a fixed order (base candidates
// chunk by chunk; before a chunk that might not fit on the stack, and at the
// end, the descents batch by batch, chunk by chunk), so lists are the same on
// every run.  Entries found by descents are logged in LDS with their places
// and written when the lists are allocated; a group whose log overflows, or
// with several blocks of candidates, is walked a second time to write.
#define WALK_WAVES 8
#define WALK_LOG 2048
#define WALK_OPEN 1024  // open-list entries of a path cell, at most

struct GroupLds {
  union {
    struct { double x, y, z, w; } geo[TRAV_CAND];  // candidates' geometry
    uint2 log[WALK_LOG];  // descents' entries: cell, list (5 bits) << 27 | place
  };
  int4 info[TRAV_CAND];
  int cand[TRAV_CAND];     // candidates expanded from a block of open-list entries
  int dcand[TRAV_CAND];    // children of popped descent items
  int2 stack[TRAV_STACK];  // descent items: (target tag << TRAV_TAG) | first child, child count
  struct { double x, y, z, w; } tgeo[8];
  int tnp[8];                     // particles of each target
  int cpush[TRAV_CAND / 64][8];   // per chunk of base candidates and target: items pushed
  int run[2][24];                 // entries so far per target and list
  int wc[WALK_WAVES][24];         // entries of one chunk of descents, by wavefront
  int2 wsum[WALK_WAVES];          // its pushes, its entries
  int off[24];
  int fits;
  // path form: the open lists of a path cell and of its parent, as (first
  // child, child count) or (cell, 0) for a leaf
  int2 open[2][WALK_OPEN];
  int nopen[2][WALK_WAVES];  // entries found by each wavefront, by parity of the block
};

// Descent items taken by the next batch from a stack of sp: batches of at most
// (TRAV_STACK - TRAV_RESERVE - sp) / 7 keep the stack below TRAV_STACK -
// TRAV_RESERVE; once that room is used up, items are popped one at a time
// (depth first), which the reserve absorbs.
__device__ __forceinline__ int batch_items(int sp) {
  const int room = (TRAV_STACK - TRAV_RESERVE - sp) / 7;
  return min(sp, max(1, min(64, room)));
}
// a chunk of candidates pushes at most 64 items per target, 512 in all, and
// must leave the depth-first reserve free: with more on the stack the descents
// come first
#define TRAV_PUSH_ROOM (TRAV_STACK - TRAV_RESERVE - 512)

// ordered particle pairs of a P2P entry
__device__ __forceinline__ unsigned long long pair_count(int nA, int nC, bool self) {
  return (unsigned long long)nA * (unsigned long long)nC - (self ? (unsigned long long)nA : 0ull);
}

// v with the value of one lane replaced (a compare and select per lane index
// had its lane masks hoisted into scalar registers, which spilled)
__device__ __forceinline__ int set_lane(int v, int lane, int value) {
  asm("v_writelane_b32 %0, %1, %2"
      : "+v"(v)
      : "s"(__builtin_amdgcn_readfirstlane(value)), "i"(lane));
  return v;
}

// The group being walked: the same in every lane, but for the own target.
struct Group {
  int n, id0;      // targets id0 .. id0 + n - 1
  unsigned leafs;  // bit tg: target tg is a leaf
  int in_cnt;          // open-list entries of the parent
  const int *open_in;  // level form: the parent's entries, and where the targets' go
  int *open_out;
  const int2 *open;    // path form: the parent's entries in LDS
  double th2, eps;
};

template <bool WRITE>
__device__ __forceinline__ void walk_descents(const DevTree &t, const Group &G, GroupLds &L,
                                              int &sp, int &cur, int &nlog,
                                              unsigned long long &pairs) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const unsigned long long below = lanes_below_mask();
  while (sp > 0) {
    const int take = batch_items(sp);
    __syncthreads();  // pushes and running counts of the step before
    int2 item = make_int2(0, 0);
    if (lane < take) item = L.stack[sp - take + lane];
    const int tag = item.x & ~((1 << TRAV_TAG) - 1), c0 = item.x & ((1 << TRAV_TAG) - 1);
    int total;
    const int pos = wave_excl_scan_int(item.y, &total);
    // every wavefront lists the children that fall into its own chunk
    for (int q = 0; q < item.y; ++q)
      if ((pos + q) >> 6 == w) L.dcand[pos + q] = tag | (c0 + q);
    __builtin_amdgcn_wave_barrier();
    sp -= take;
    const bool valid = 64 * w + lane < total;
    const int it = valid ? L.dcand[64 * w + lane] : 0;
    const int tgl = it >> TRAV_TAG;
    const int C = it & ((1 << TRAV_TAG) - 1);
    int cat = CAT_NONE;
    int4 iC = make_int4(0, 0, 0, 0);
    if (valid) {
      const double4 gC = t.ngeo[C];
      iC = t.ninfo[C];
      const auto &a = L.tgeo[tgl];
      cat = classify(G.id0 + tgl, make_double4(a.x, a.y, a.z, a.w), true, C, gC, iC.y == 0, G.th2,
                     G.eps);
      if (!WRITE && cat == CAT_P2P) pairs += pair_count(L.tnp[tgl], iC.w - iC.z, C == G.id0 + tgl);
    }
    // the chunk's entries per target and list, and each lane's rank among its own
    int rank = 0, npush = 0, nent = 0, count = 0;
    if (64 * w < total) {
#pragma unroll
      for (int tg = 0; tg < 8; ++tg) {
        if (!(G.leafs >> tg & 1)) continue;
        const bool mine = valid && tgl == tg;
        if (__ballot(mine) == 0ull) continue;
        const unsigned long long bm = __ballot(mine && cat == CAT_M2L);
        const unsigned long long bp = __ballot(mine && cat == CAT_P2P);
        const unsigned long long bd = __ballot(mine && cat == CAT_DEEPEN);
        const unsigned long long b = cat == CAT_M2L ? bm : cat == CAT_P2P ? bp : bd;
        const int r = __popcll(b & below) + (cat == CAT_DEEPEN ? npush : 0);
        rank = mine ? r : rank;
        count = set_lane(count, 3 * tg, __popcll(bm));
        count = set_lane(count, 3 * tg + 1, __popcll(bp));
        npush += __popcll(bd);
        nent += __popcll(bm) + __popcll(bp);
      }
    }
    if (lane < 24) L.wc[w][lane] = count;
    if (lane == 0) L.wsum[w] = make_int2(npush, nent);
    __syncthreads();
    int push0 = sp, pushed = 0, ent0 = nlog, ents = 0;
#pragma unroll
    for (int ww = 0; ww < WALK_WAVES; ++ww) {
      const int2 c = L.wsum[ww];
      push0 += ww < w ? c.x : 0;
      pushed += c.x;
      ent0 += ww < w ? c.y : 0;
      ents += c.y;
    }
    if (cat == CAT_DEEPEN) {
      if (push0 + rank < TRAV_STACK)  // always (see batch_items)
        L.stack[push0 + rank] = make_int2((tgl << TRAV_TAG) | iC.x, iC.y);
      else
        atomicOr(&t.hdr->overflow, OVF_STACK);
    }
    const unsigned long long be = __ballot(cat == CAT_M2L || cat == CAT_P2P);
    if (cat == CAT_M2L || cat == CAT_P2P) {
      const int j = 3 * tgl + cat - 1;
      int at = L.run[cur][j] + rank;
#pragma unroll
      for (int ww = 0; ww < WALK_WAVES - 1; ++ww) at += ww < w ? L.wc[ww][j] : 0;
      if (WRITE) {
        (cat == CAT_M2L ? t.m2l_src : t.p2p_src)[L.off[j] + at] = C;
      } else {
        const int e = ent0 + __popcll(be & below);
        if (e < WALK_LOG) L.log[e] = make_uint2((unsigned)C, (unsigned)j << 27 | (unsigned)at);
      }
    }
    sp = min(sp + pushed, TRAV_STACK);
    nlog += ents;
    if (threadIdx.x < 24) {
      int s = L.run[cur][threadIdx.x];
#pragma unroll
      for (int ww = 0; ww < WALK_WAVES; ++ww) s += L.wc[ww][threadIdx.x];
      L.run[cur ^ 1][threadIdx.x] = s;
    }
    cur ^= 1;
  }
  __syncthreads();
}

// One pass over a group's candidates.  Counting: cnt gets the entries of the
// own target's three lists, and with a single block of candidates cat[c] the
// category and place (<< 3) of candidate 64 c + lane.  Writing: entries go to
// their lists.
template <bool WRITE, bool PATH>
__device__ __forceinline__ void walk_pass(const DevTree &t, int l, int P, const Group &G,
                                          GroupLds &L, const double4 &gA, int npA, int (&cnt)[3],
                                          int (&cat)[TRAV_CAND / 64], int &total, int &nlog,
                                          unsigned long long &pairs) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const unsigned long long below = lanes_below_mask();
  const bool mine = w < G.n, leafA = G.leafs >> w & 1;
  const int A = G.id0 + w;
  int sp = 0, cur = 0;
#pragma unroll
  for (int k = 0; k < 3; ++k) cnt[k] = 0;
  if (threadIdx.x < 24) L.run[0][threadIdx.x] = 0;
  // the own target's counts live in registers, and in run[] during descents
  auto descents = [&]() {
    if (lane < 3) L.run[cur][3 * w + lane] = lane == 0 ? cnt[0] : lane == 1 ? cnt[1] : cnt[2];
    walk_descents<WRITE>(t, G, L, sp, cur, nlog, pairs);
#pragma unroll
    for (int k = 0; k < 3; ++k)
      cnt[k] = __builtin_amdgcn_readfirstlane(L.run[cur][3 * w + k]);
  };
  for (int eb = 0; eb < G.in_cnt; eb += 64) {
    // expand 64 open-list entries into candidate cells (children, or the leaf itself)
    const int e = eb + lane;
    int ec = 0, c0 = 0;
    if (e < G.in_cnt) {
      if (PATH) {
        const int2 o = G.open[e];
        ec = max(o.y, 1);
        c0 = o.x;
      } else if (l == 0) {
        ec = 1;  // the pair (root, root) of this request's tree
        c0 = P;
      } else {
        const int B = G.open_in[e];
        const int4 ib = t.ninfo[B];
        ec = ib.y > 0 ? ib.y : 1;
        c0 = ib.y > 0 ? ib.x : B;
      }
    }
    const int pos = wave_excl_scan_int(ec, &total);
    __syncthreads();  // the block before is placed
    for (int q = 0; q < ec; ++q)
      if ((pos + q) >> 6 == w) L.cand[pos + q] = c0 + q;
    __builtin_amdgcn_wave_barrier();
    const int own = 64 * w + lane;
    if (own < total) {
      const int C = L.cand[own];
      const double4 g = t.ngeo[C];
      L.geo[own] = {g.x, g.y, g.z, g.w};
      L.info[own] = t.ninfo[C];
    }
    __syncthreads();
    if (mine) {
#pragma unroll
      for (int c = 0; c < TRAV_CAND / 64; ++c) {
        cat[c] = CAT_NONE;
        if (64 * c < total) {
          const int i = 64 * c + lane;
          if (i < total) {
            const int C = L.cand[i];
            const auto &g = L.geo[i];
            const int4 iC = L.info[i];
            cat[c] = classify(A, gA, leafA, C, make_double4(g.x, g.y, g.z, g.w), iC.y == 0, G.th2,
                              G.eps);
            if (!WRITE && cat[c] == CAT_P2P) pairs += pair_count(npA, iC.w - iC.z, C == A);
          }
          if (leafA) {
            const int d = __popcll(__ballot(cat[c] == CAT_DEEPEN));
            if (lane == 0) L.cpush[c][w] = d;
          }
        }
      }
    }
    if (G.leafs) __syncthreads();  // push counts; the geometry's space becomes the log's
#pragma unroll
    for (int c = 0; c < TRAV_CAND / 64; ++c) {
      if (64 * c >= total) break;
      if (sp > TRAV_PUSH_ROOM) descents();
      if (mine) {
        const int k = cat[c];
        const unsigned long long bm = __ballot(k == CAT_M2L);
        const unsigned long long bp = __ballot(k == CAT_P2P);
        const unsigned long long bo = __ballot(k == CAT_OPEN);
        const unsigned long long b = k == CAT_M2L ? bm : k == CAT_P2P ? bp : bo;
        const int at = __popcll(b & below) + (k == CAT_M2L ? cnt[0] : k == CAT_P2P ? cnt[1] : cnt[2]);
        if (WRITE) {
          if (k >= CAT_M2L && k <= (PATH ? CAT_P2P : CAT_OPEN))
            (k == CAT_M2L ? t.m2l_src : k == CAT_P2P ? t.p2p_src : G.open_out)
                [L.off[3 * w + k - 1] + at] = L.cand[64 * c + lane];
        } else {
          cat[c] = k | at << 3;
        }
        cnt[0] += __popcll(bm);
        cnt[1] += __popcll(bp);
        cnt[2] += __popcll(bo);
        if (leafA) {
          const unsigned long long bd = __ballot(k == CAT_DEEPEN);
          int s = sp;
#pragma unroll
          for (int tg = 0; tg < 8; ++tg)
            if (tg < w && (G.leafs >> tg & 1)) s += L.cpush[c][tg];
          if (k == CAT_DEEPEN) {
            s += __popcll(bd & below);
            const int4 iC = L.info[64 * c + lane];
            if (s < TRAV_STACK)  // always (see batch_items)
              L.stack[s] = make_int2((w << TRAV_TAG) | iC.x, iC.y);
            else
              atomicOr(&t.hdr->overflow, OVF_STACK);
          }
        }
      }
      if (G.leafs) {
        int pushed = 0;
#pragma unroll
        for (int tg = 0; tg < 8; ++tg)
          if (G.leafs >> tg & 1) pushed += L.cpush[c][tg];
        sp = min(sp + __builtin_amdgcn_readfirstlane(pushed), TRAV_STACK);
      }
    }
  }
  if (sp > 0) descents();
}

// Allocates the lists of a group's targets by its first wavefront (lane tg:
// target tg, with mine[k] entries of list k), one allocation per list, the
// targets' lists laid out in target order inside it: all groups of a level
// allocate at about the same time, and device-scope atomics on one address
// serialise.  If any list does not fit, none is written and every target gets
// empty lists, so that no count ever covers entries that were not written (the
// host regrows and rebuilds): false.
__device__ __forceinline__ bool allocate_lists(const DevTree &t, int l, const Group &G,
                                               const int (&mine)[3], int (&o)[3]) {
  const int lane = threadIdx.x & 63;
  Header *h = t.hdr;
  unsigned long long *const cur[3] = {&h->m2l_cursor, &h->p2p_cursor, &h->open_cursor[l]};
  const int64_t cap[3] = {t.cap_m2l, t.cap_p2p, t.cap_open};
  const int ovf_bit[3] = {OVF_M2L, OVF_P2P, OVF_OPEN};
  int bits = 0, incl[3], tot[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    incl[k] = mine[k];  // inclusive prefix over the target lanes 0..7
#pragma unroll
    for (int d = 1; d < 8; d <<= 1) {
      const int y = __shfl_up(incl[k], d, 64);
      if (lane >= d) incl[k] += y;
    }
    tot[k] = __builtin_amdgcn_readlane(incl[k], 7);
  }
  // lane k allocates list k: the three in one instruction, one round trip
  const int tk = lane == 0 ? tot[0] : lane == 1 ? tot[1] : tot[2];
  unsigned long long got = 0;
  if (lane < 3 && tk > 0)
    got = atomicAdd(lane == 0 ? cur[0] : lane == 1 ? cur[1] : cur[2], (unsigned long long)tk);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int64_t base = (int64_t)readlane_u64(got, k);
    o[k] = (int)base + incl[k] - mine[k];
    if (lane < G.n && base + tot[k] > cap[k]) bits |= ovf_bit[k];
  }
  const bool ovf = __ballot(bits != 0) != 0ull;
  if (lane < G.n) {
    const int A = G.id0 + lane;
    t.m2l_off[A] = o[0];
    t.m2l_cnt[A] = ovf ? 0 : mine[0];
    t.p2p_off[A] = o[1];
    t.p2p_cnt[A] = ovf ? 0 : mine[1];
    t.open_off[A] = o[2];
    t.open_cnt[A] = ovf ? 0 : mine[2];
    if (bits) atomicOr(&h->overflow, bits);
  }
  return !ovf;
}

// Group P with its parent's open list in G (in_cnt, open_in / open).
template <bool PATH>
__device__ __forceinline__ void walk_group(const DevTree &t, int l, int P, Group &G, GroupLds &L) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int4 ia = t.ninfo[G.id0 + (lane < G.n ? lane : 0)];
  G.leafs = (unsigned)__ballot(lane < G.n && ia.y == 0);
  const double4 gA = t.ngeo[G.id0 + min(w, G.n - 1)];
  if (lane == 0) L.tgeo[w] = {gA.x, gA.y, gA.z, gA.w};
  if (threadIdx.x < 8) L.tnp[threadIdx.x] = ia.w - ia.z;
  const int npA = __builtin_amdgcn_readlane(ia.w - ia.z, w);
  unsigned long long pairs = 0;
  int cnt[3], cat[TRAV_CAND / 64], total = 0, nlog = 0;
  walk_pass<false, PATH>(t, l, P, G, L, gA, npA, cnt, cat, total, nlog, pairs);
  if (PATH) cnt[2] = 0;  // the next level's groups form their open lists themselves
  if (lane < 3) L.run[0][3 * w + lane] = lane == 0 ? cnt[0] : lane == 1 ? cnt[1] : cnt[2];
  __syncthreads();
  if (w == 0) {
    int mine[3] = {0, 0, 0}, o[3];
    if (lane < G.n)
#pragma unroll
      for (int k = 0; k < 3; ++k) mine[k] = L.run[0][3 * lane + k];
    const bool fits = allocate_lists(t, l, G, mine, o);
    if (lane < 8)
#pragma unroll
      for (int k = 0; k < 3; ++k) L.off[3 * lane + k] = o[k];
    if (lane == 0) L.fits = fits;
  }
  __syncthreads();
  if (L.fits) {
    if (G.in_cnt <= 64 && nlog <= WALK_LOG) {
      if (w < G.n && G.in_cnt > 0)
#pragma unroll
        for (int c = 0; c < TRAV_CAND / 64; ++c) {
          if (64 * c >= total) break;
          const int k = cat[c] & 7, at = cat[c] >> 3;
          if (k >= CAT_M2L && k <= (PATH ? CAT_P2P : CAT_OPEN))
            (k == CAT_M2L ? t.m2l_src : k == CAT_P2P ? t.p2p_src : G.open_out)
                [L.off[3 * w + k - 1] + at] = L.cand[64 * c + lane];
        }
      for (int e = threadIdx.x; e < nlog; e += WALK_WAVES * 64) {
        const uint2 v = L.log[e];
        const int j = (int)(v.y >> 27);
        (j % 3 == 0 ? t.m2l_src : t.p2p_src)[L.off[j] + (int)(v.y & ((1u << 27) - 1))] = (int)v.x;
      }
    } else {
      unsigned long long none = 0;
      walk_pass<true, PATH>(t, l, P, G, L, gA, npA, cnt, cat, total, nlog, none);
    }
    pairs = wave_sum(pairs);
    if (lane == 0 && pairs) atomicAdd(&t.hdr->p2p_pairs, pairs);
  }
}

// Level form.  Level l >= 1: group P is cell P of level l-1, its children are
// the targets.  Level 0: one group per request root, whose only candidate is
// itself, so cells of different requests never meet.
__device__ __forceinline__ void walk_level_group(const DevTree &t, int l, int P, double th2,
                                                 double eps, GroupLds &L) {
  Group G;
  G.n = 1;
  G.id0 = P;
  G.in_cnt = 1;
  G.open_in = nullptr;
  G.open = nullptr;
  if (l > 0) {
    const int4 ip = t.ninfo[P];
    if (ip.y == 0) return;
    G.n = ip.y;
    G.id0 = ip.x;
    G.in_cnt = t.open_cnt[P];
    G.open_in = ((l & 1) ? t.open_buf0 : t.open_buf1) + t.open_off[P];
  }
  G.open_out = (l & 1) ? t.open_buf1 : t.open_buf0;
  G.th2 = th2;
  G.eps = eps;
  walk_group<false>(t, l, P, G, L);
}

// ---------------------------------------------------------------------------
// Wavefront form, for levels with groups enough to fill the chip with a
// wavefront each (more than WALK_GROUP_LEVEL): half the instructions of the
// workgroup form and four groups in flight per SIMD, so what a level costs is
// its instructions, not their latency (4,096 groups: 62 us, 238 in the
// workgroup form).  Same entries in the same places.
// ---------------------------------------------------------------------------
#define TRAV_WAVES 2
#define WALK_GROUP_LEVEL 1024

// Per-wavefront state of the sibling targets (children of one parent cell).
struct Sibs {
  int n;          // number of targets, 1..8
  int id[8];
  bool leaf[8];
  int np[8];      // particles per target
  int cnt[8][3];  // M2L / P2P / OPEN entries counted (pass 0) or written (pass 1)
  int off[8][3];  // list offsets (pass 1)
};

struct WaveLds {
  int cand[TRAV_CAND];   // candidates expanded from a block of open-list entries
  int ccat[TRAV_CAND];   // their categories against the 8 targets (3 bits each), kept
                         // from the counting pass for the writing pass
  int dcand[TRAV_CAND];  // children of popped descent items
  int stack[TRAV_STACK]; // descent items: (target tag << TRAV_TAG) | cell
  double4 geo[8];
  int sid[8];            // target cells and their leaf flags, for per-lane lookup
  int sleaf[8];
};

template <bool WRITE>
__device__ __forceinline__ void emit(const DevTree &t, Sibs &S, int tg, int cat, bool mine, int C,
                                     int npC, int *open_out, unsigned long long &pairs) {
  const unsigned long long below = lanes_below_mask();
  const unsigned long long bm = __ballot(mine && cat == CAT_M2L);
  const unsigned long long bp = __ballot(mine && cat == CAT_P2P);
  const unsigned long long bo = __ballot(mine && cat == CAT_OPEN);
  if (WRITE) {
    if (mine && cat == CAT_M2L) t.m2l_src[S.off[tg][0] + S.cnt[tg][0] + __popcll(bm & below)] = C;
    if (mine && cat == CAT_P2P) t.p2p_src[S.off[tg][1] + S.cnt[tg][1] + __popcll(bp & below)] = C;
    if (mine && cat == CAT_OPEN) open_out[S.off[tg][2] + S.cnt[tg][2] + __popcll(bo & below)] = C;
  } else if (mine && cat == CAT_P2P) {  // particle pairs, counted once (counting pass)
    pairs += pair_count(S.np[tg], npC, C == S.id[tg]);
  }
  S.cnt[tg][0] += __popcll(bm);
  S.cnt[tg][1] += __popcll(bp);
  S.cnt[tg][2] += __popcll(bo);
}

// push (tg, C) for every lane whose leaf target descends into C
__device__ __forceinline__ void push_item(const DevTree &t, WaveLds &L, int &sp, bool push, int tg,
                                          int C) {
  const unsigned long long m = __ballot(push);
  const int k = __popcll(m);
  if (sp + k > TRAV_STACK) {  // cannot happen (see batch_items); kept as a guard
    if (__lane_id() == 0) atomicOr(&t.hdr->overflow, OVF_STACK);
    return;
  }
  if (push) L.stack[sp + __popcll(m & lanes_below_mask())] = (tg << TRAV_TAG) | C;
  sp += k;
}

// Descents of leaf targets into non-leaf cells, LIFO.  A popped item (tg, C)
// makes the children of C candidates of target tg; each may push one item.
// Batches of take <= (TRAV_STACK - TRAV_RESERVE - sp) / 7 items keep sp below
// TRAV_STACK - TRAV_RESERVE; once that room is used up, items are popped one
// at a time (depth first), which the reserve absorbs.
template <bool WRITE>
__device__ __forceinline__ void wave_drain(const DevTree &t, Sibs &S, WaveLds &L, int &sp, int *open_out, double th2,
                      double eps, unsigned long long &pairs) {
  const int lane = __lane_id();
  while (sp > 0) {
    const int take = batch_items(sp);
    const bool vp = lane < take;
    const int item = vp ? L.stack[sp - take + lane] : 0;
    __builtin_amdgcn_wave_barrier();
    sp -= take;
    const int tgi = item >> TRAV_TAG;
    const int Ci = item & ((1 << TRAV_TAG) - 1);
    const int4 ii = vp ? t.ninfo[Ci] : make_int4(0, 0, 0, 0);
    int total;
    const int pos = wave_excl_scan_int(ii.y, &total);
    for (int q = 0; q < ii.y; ++q) L.dcand[pos + q] = (tgi << TRAV_TAG) | (ii.x + q);
    __builtin_amdgcn_wave_barrier();
    for (int cb = 0; cb < total; cb += 64) {
      const bool valid = cb + lane < total;
      const int it = valid ? L.dcand[cb + lane] : 0;
      const int tgl = it >> TRAV_TAG;
      const int C = it & ((1 << TRAV_TAG) - 1);
      double4 gC = make_double4(0, 0, 0, 0);
      int nC = 0, npC = 0;
      if (valid) {
        gC = t.ngeo[C];
        const int4 iC = t.ninfo[C];
        nC = iC.y;
        npC = iC.w - iC.z;
      }
      // each lane's item belongs to one target: classify once against it
      const int lcat = valid ? classify(L.sid[tgl], L.geo[tgl], L.sleaf[tgl] != 0, C, gC,
                                        nC == 0, th2, eps)
                             : CAT_NONE;
#pragma unroll
      for (int tg = 0; tg < 8; ++tg) {
        if (tg < S.n) {
          const bool mine = valid && tgl == tg;
          if (__ballot(mine) == 0ull) continue;  // no item of this target in the chunk
          const int cat = mine ? lcat : CAT_NONE;
          emit<WRITE>(t, S, tg, cat, mine, C, npC, open_out, pairs);
          push_item(t, L, sp, cat == CAT_DEEPEN, tg, C);
        }
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// One pass over the candidates of a sibling group (pass 0 counts, pass 1 writes).
// With at most 64 open-list entries (one block of candidates, the usual
// case) the counting pass keeps every candidate's categories in LDS and the
// writing pass replays them: it reads no cell data for these candidates (its
// only global accesses are the list stores and the descents).  ncand: the
// number of cached candidates, set by the counting pass (0 when it expanded
// none, e.g. an open list emptied by an overflow) and read by the writing pass.
template <bool WRITE>
__device__ __forceinline__ void wave_group(const DevTree &t, int l, int P, Sibs &S, WaveLds &L,
                           const int *open_in, int *open_out, double th2, double eps,
                           unsigned long long &pairs, int &ncand) {
  const int lane = __lane_id();
#pragma unroll
  for (int tg = 0; tg < 8; ++tg) S.cnt[tg][0] = S.cnt[tg][1] = S.cnt[tg][2] = 0;
  int sp = 0;
  int in_off = 0, in_cnt = 1;
  if (l > 0) {
    in_off = t.open_off[P];
    in_cnt = t.open_cnt[P];
  }
  const bool cached = in_cnt <= 64;
  if (!WRITE) ncand = 0;
  if (WRITE && cached) {
    const int total = min(ncand, TRAV_CAND);
    for (int cb = 0; cb < total; cb += 64) {
      if (sp > TRAV_PUSH_ROOM) wave_drain<WRITE>(t, S, L, sp, open_out, th2, eps, pairs);
      const bool valid = cb + lane < total;
      const int C = valid ? L.cand[cb + lane] : 0;
      const int code = valid ? L.ccat[cb + lane] : 0;
#pragma unroll
      for (int tg = 0; tg < 8; ++tg) {
        if (tg < S.n) {
          const int cat = (code >> (3 * tg)) & 7;
          emit<WRITE>(t, S, tg, cat, valid, C, 0, open_out, pairs);
          if (S.leaf[tg]) push_item(t, L, sp, cat == CAT_DEEPEN, tg, C);
        }
      }
    }
    wave_drain<WRITE>(t, S, L, sp, open_out, th2, eps, pairs);
    return;
  }
  for (int eb = 0; eb < in_cnt; eb += 64) {
    // expand 64 open-list entries into candidate cells (children, or the leaf itself)
    const int e = eb + lane;
    int ec = 0, c0 = 0;
    if (e < in_cnt) {
      if (l == 0) {
        ec = 1;  // the pair (root, root) of this request's tree
        c0 = P;
      } else {
        const int B = open_in[in_off + e];
        const int4 iB = t.ninfo[B];
        ec = iB.y > 0 ? iB.y : 1;
        c0 = iB.y > 0 ? iB.x : B;
      }
    }
    int total;
    const int pos = wave_excl_scan_int(ec, &total);
    for (int q = 0; q < ec; ++q) L.cand[pos + q] = c0 + q;
    if (!WRITE && cached) ncand = total;
    __builtin_amdgcn_wave_barrier();
    for (int cb = 0; cb < total; cb += 64) {
      // a chunk pushes at most 64 items per target, 512 in all, and must leave
      // the depth-first reserve free
      if (sp > TRAV_PUSH_ROOM) wave_drain<WRITE>(t, S, L, sp, open_out, th2, eps, pairs);
      const bool valid = cb + lane < total;
      const int C = valid ? L.cand[cb + lane] : 0;
      double4 gC = make_double4(0, 0, 0, 0);
      int nC = 0, npC = 0;
      if (valid) {
        gC = t.ngeo[C];
        const int4 iC = t.ninfo[C];
        nC = iC.y;
        npC = iC.w - iC.z;
      }
      int code = 0;
#pragma unroll
      for (int tg = 0; tg < 8; ++tg) {
        if (tg < S.n) {
          const int cat = valid ? classify(S.id[tg], L.geo[tg], S.leaf[tg], C, gC, nC == 0, th2,
                                           eps)
                                : CAT_NONE;
          code |= cat << (3 * tg);
          emit<WRITE>(t, S, tg, cat, valid, C, npC, open_out, pairs);
          if (S.leaf[tg]) push_item(t, L, sp, cat == CAT_DEEPEN, tg, C);
        }
      }
      if (!WRITE && cached && valid) L.ccat[cb + lane] = code;
    }
    __builtin_amdgcn_wave_barrier();
  }
  wave_drain<WRITE>(t, S, L, sp, open_out, th2, eps, pairs);
}

// Level l >= 1: one wavefront per cell P of level l-1 with children; the
// children are the targets.  Level 0: one wavefront per request root, whose
// only candidate is itself, so cells of different requests never meet.
__device__ __forceinline__ void wave_parent(const DevTree &t, int l, int P, double th2, double eps, WaveLds &L) {
  const int lane = threadIdx.x & 63;
  Header *h = t.hdr;
  Sibs S;
  if (l == 0) {
    // a request's root is the only target of its group; every sibling slot
    // must hold a valid id because the slots are read below before the S.n
    // guard applies
    S.n = 1;
#pragma unroll
    for (int tg = 0; tg < 8; ++tg) S.id[tg] = P;
  } else {
    const int4 iP = t.ninfo[P];
    const int nc = iP.y, c0 = iP.x;
    if (nc == 0) return;
    S.n = nc;
#pragma unroll
    for (int tg = 0; tg < 8; ++tg) S.id[tg] = c0 + (tg < nc ? tg : 0);
  }
#pragma unroll
  for (int tg = 0; tg < 8; ++tg) {
    const int A = S.id[tg];
    const int4 iA = t.ninfo[A];
    S.leaf[tg] = iA.y == 0;
    S.np[tg] = iA.w - iA.z;
  }
  if (lane < 8) {
    int A = S.id[0];
    bool lf = S.leaf[0];
#pragma unroll
    for (int tg = 1; tg < 8; ++tg)
      if (lane == tg) {
        A = S.id[tg];
        lf = S.leaf[tg];
      }
    L.geo[lane] = t.ngeo[A];
    L.sid[lane] = A;
    L.sleaf[lane] = lf ? 1 : 0;
  }
  __builtin_amdgcn_wave_barrier();
  const int *open_in = (l & 1) ? t.open_buf0 : t.open_buf1;
  int *open_out = (l & 1) ? t.open_buf1 : t.open_buf0;
  unsigned long long pairs = 0;
  int ncand = 0;
  wave_group<false>(t, l, P, S, L, open_in, open_out, th2, eps, pairs, ncand);
  // allocate every target's lists (lane tg handles target tg)
  int mine[3] = {0, 0, 0};
#pragma unroll
  for (int tg = 0; tg < 8; ++tg)
    if (lane == tg)
#pragma unroll
      for (int k = 0; k < 3; ++k) mine[k] = S.cnt[tg][k];
  // one allocation per wavefront and list (the targets' lists laid out in
  // target order inside it): all wavefronts of a level allocate at about the
  // same time, and device-scope atomics on one address serialise
  int o[3] = {0, 0, 0};
  int bits = 0;
  {
    unsigned long long *const cur[3] = {&h->m2l_cursor, &h->p2p_cursor, &h->open_cursor[l]};
    const int64_t cap[3] = {t.cap_m2l, t.cap_p2p, t.cap_open};
    const int ovf_bit[3] = {OVF_M2L, OVF_P2P, OVF_OPEN};
    int incl[3], tot[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      incl[k] = mine[k];  // inclusive prefix over the target lanes 0..7
#pragma unroll
      for (int d = 1; d < 8; d <<= 1) {
        const int y = __shfl_up(incl[k], d, 64);
        if (lane >= d) incl[k] += y;
      }
      tot[k] = __shfl(incl[k], 7, 64);
    }
    // lane k allocates list k: the three in one instruction, one round trip
    const int tk = lane == 0 ? tot[0] : lane == 1 ? tot[1] : tot[2];
    unsigned long long got = 0;
    if (lane < 3 && tk > 0)
      got = atomicAdd(lane == 0 ? cur[0] : lane == 1 ? cur[1] : cur[2], (unsigned long long)tk);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int64_t base = (int64_t)readlane_u64(got, k);
      o[k] = (int)base + incl[k] - mine[k];
      if (lane < S.n && base + tot[k] > cap[k]) bits |= ovf_bit[k];
    }
  }
  // if any target's lists do not fit, the wavefront writes none of them and
  // every one of its targets gets empty lists: no count ever covers entries
  // that were not written (the host regrows and rebuilds)
  const bool ovf = __ballot(bits != 0) != 0ull;
  if (lane < S.n) {
    int A = S.id[0];
#pragma unroll
    for (int tg = 1; tg < 8; ++tg)
      if (lane == tg) A = S.id[tg];
    t.m2l_off[A] = o[0];
    t.m2l_cnt[A] = ovf ? 0 : mine[0];
    t.p2p_off[A] = o[1];
    t.p2p_cnt[A] = ovf ? 0 : mine[1];
    t.open_off[A] = o[2];
    t.open_cnt[A] = ovf ? 0 : mine[2];
    if (bits) atomicOr(&h->overflow, bits);
  }
  if (ovf) return;
#pragma unroll
  for (int tg = 0; tg < 8; ++tg)
#pragma unroll
    for (int k = 0; k < 3; ++k) S.off[tg][k] = __shfl(o[k], tg, 64);
  wave_group<true>(t, l, P, S, L, open_in, open_out, th2, eps, pairs, ncand);
  pairs = wave_sum(pairs);
  if (lane == 0 && pairs) atomicAdd(&h->p2p_pairs, pairs);
}

__global__ __launch_bounds__(TRAV_WAVES * 64) void k_walk_waves(DevTree t, int l, int ps, int pe,
                                                                double th2, double eps) {
  __shared__ WaveLds lds[TRAV_WAVES];
  const int w = threadIdx.x >> 6;
  const int P = ps + xcd_block<32>(blockIdx.x, gridDim.x) * TRAV_WAVES + w;
  if (P >= pe) return;
  wave_parent(t, l, P, th2, eps, lds[w]);
}

// Level l with its bounds read from the tree header (queued before the
// level sizes are known on the host): the waves of the grid stride over the
// parents; nothing is done on a tree whose node workspace overflowed, nor of
// positions that are not finite.
__global__ __launch_bounds__(TRAV_WAVES * 64) void k_walk_waves_dev(DevTree t, int l, double th2,
                                                                    double eps) {
  __shared__ WaveLds lds[TRAV_WAVES];
  const Header *h = t.hdr;
  if (h->overflow & (OVF_NODES | OVF_INPUT)) return;
  const int ps = l == 0 ? 0 : h->lvl_start[l - 1];
  const int pe = l == 0 ? t.n_req : h->lvl_start[l];
  const int w = threadIdx.x >> 6;
  const int nw = gridDim.x * TRAV_WAVES;
  for (int P = ps + xcd_block<32>(blockIdx.x, gridDim.x) * TRAV_WAVES + w; P < pe; P += nw)
    wave_parent(t, l, P, th2, eps, lds[w]);
}

// ---------------------------------------------------------------------------
// Path form: the whole walk in one launch.  A group needs its parent's open
// list, which depends on nothing but the parent's ancestors: the open list of
// a path cell is those of its candidates (children of its parent's open cells)
// that it neither accepts nor ends at, in order.  So every workgroup forms the
// open lists along the path from the root to its own cell P in LDS (one
// candidate per thread and level: about 2 us a level) and no level waits for
// another: 9 launches of 15-40 us of a 12,526-particle solve became one.  The
// levels above are redone by every group below them, so trees of many groups
// keep the level form.  A path cell with more than WALK_OPEN open cells
// flags OVF_PATH and the host walks by levels.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double lane_value(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, lane);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// The open list of cell P (level lev, particles from begin on) of the tree
// under root; its buffer in ob, its length (-1: too long) returned.
__device__ __forceinline__ int path_open_list(const DevTree &t, int root, int lev, int begin,
                                              double th2, double eps, GroupLds &L, int &ob) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const unsigned long long below = lanes_below_mask();
  int4 ip = t.ninfo[root];
  ob = 0;
  int nopen = 1, par = 0;
  if (threadIdx.x == 0) L.open[0][0] = make_int2(ip.x, ip.y);  // (root, root) is opened
  __syncthreads();
  for (int k = 1; k <= lev; ++k) {
    // the path cell: the child of the last one that holds P's particles
    const int ch = ip.x + (lane < ip.y ? lane : 0);
    const int4 ic = t.ninfo[ch];
    const double4 gc = t.ngeo[ch];
    int A = 0, next = 0;
    double4 gA = make_double4(0, 0, 0, 0);
    for (int eb = 0; eb < nopen; eb += 64) {
      int2 o = make_int2(0, 0);
      const bool ve = eb + lane < nopen;
      if (ve) o = L.open[ob][eb + lane];
      const int ec = ve ? max(o.y, 1) : 0;
      int total;
      const int pos = wave_excl_scan_int(ec, &total);
      for (int q = 0; q < ec; ++q)
        if ((pos + q) >> 6 == w) L.cand[pos + q] = o.x + q;
      __builtin_amdgcn_wave_barrier();
      const int i = 64 * w + lane;
      const bool valid = i < total;
      const int C = valid ? L.cand[i] : root;
      const double4 gC = t.ngeo[C];
      const int4 iC = t.ninfo[C];
      if (eb == 0) {
        const int j = (int)__ffsll((long long)__ballot(lane < ip.y && ic.z <= begin &&
                                                       begin < ic.w)) - 1;
        A = ip.x + j;
        gA = make_double4(lane_value(gc.x, j), lane_value(gc.y, j), lane_value(gc.z, j),
                          lane_value(gc.w, j));
        ip = make_int4(__builtin_amdgcn_readlane(ic.x, j), __builtin_amdgcn_readlane(ic.y, j), 0,
                       0);
      }
      const bool open = valid && classify(A, gA, false, C, gC, iC.y == 0, th2, eps) == CAT_OPEN;
      const unsigned long long b = __ballot(open);
      if (lane == 0) L.nopen[par][w] = __popcll(b);
      __syncthreads();
      int at = next + __popcll(b & below);
#pragma unroll
      for (int ww = 0; ww < WALK_WAVES; ++ww) {
        const int c = L.nopen[par][ww];
        at += ww < w ? c : 0;
        next += c;
      }
      par ^= 1;
      if (open && at < WALK_OPEN)
        L.open[ob ^ 1][at] = iC.y > 0 ? make_int2(iC.x, iC.y) : make_int2(C, 0);
    }
    __syncthreads();
    nopen = __builtin_amdgcn_readfirstlane(next);
    if (nopen > WALK_OPEN) return -1;
    ob ^= 1;
  }
  return nopen;
}

__global__ __launch_bounds__(WALK_WAVES * 64, 4) void k_walk_paths(DevTree t, double th2,
                                                                   double eps) {
  __shared__ GroupLds lds;
  Header *h = t.hdr;
  if (h->overflow & (OVF_NODES | OVF_INPUT)) return;
  const int nn = min(h->lvl_start[FMM_NLEVELS], (int)t.cap_nodes);
  for (int P = blockIdx.x; P < nn; P += gridDim.x) {
    const int4 ip = t.ninfo[P];
    if (P < t.n_req && threadIdx.x == 0) {  // a root: itself its only candidate
      const bool leaf = ip.y == 0;
      const int64_t at = leaf ? (int64_t)atomicAdd(&h->p2p_cursor, 1ull) : 0;
      const bool fits = at < t.cap_p2p;
      if (leaf && !fits) atomicOr(&h->overflow, OVF_P2P);
      if (leaf && fits) t.p2p_src[at] = P;
      t.m2l_off[P] = 0;
      t.m2l_cnt[P] = 0;
      t.p2p_off[P] = (int)at;
      t.p2p_cnt[P] = leaf && fits ? 1 : 0;
      if (leaf) atomicAdd(&h->p2p_pairs, pair_count(ip.w - ip.z, ip.w - ip.z, true));
    }
    if (ip.y == 0) continue;
    Group G;
    G.n = ip.y;
    G.id0 = ip.x;
    G.open_in = nullptr;
    G.open_out = nullptr;
    G.th2 = th2;
    G.eps = eps;
    int ob;
    G.in_cnt = path_open_list(t, t.nreq[P], t.nlev[P], ip.z, th2, eps, lds, ob);
    if (G.in_cnt < 0) {
      if (threadIdx.x == 0) atomicOr(&h->overflow, OVF_PATH);
      return;
    }
    G.open = lds.open[ob];
    walk_group<true>(t, 0, P, G, lds);
    __syncthreads();
  }
}

// One level: groups ps .. pe - 1, a workgroup each.
__global__ __launch_bounds__(WALK_WAVES * 64, 4) void k_walk_level(DevTree t, int l, int ps,
                                                                   int pe, double th2, double eps) {
  __shared__ GroupLds lds;
  const int P = ps + blockIdx.x;
  if (P < pe) walk_level_group(t, l, P, th2, eps, lds);
}

// ---------------------------------------------------------------------------
// Near-field work items.  With one wavefront per leaf the near field waited
// for its longest list: a sparse outer leaf of a concentrated system lists a
// large part of all leaves (12,526-particle Plummer sphere, leaf 64: one leaf
// of 785 kept P2P running for 540 us, now 34).  A leaf's list is therefore cut
// into shares, each summed by a wavefront of its own and added up in share
// order when L2P reads them; the groups of 64 sinks of a leaf are separate
// items too (they had been taken in turn by one wavefront).
//
// The cut depends on the leaf, its list and the size of its own system only,
// so a system's sums do not depend on what it is batched with, nor on the
// sinks asked for.  Shares consist of whole windows of the source stream, so
// the FP32 partial sums of the mixed form are those of the uncut list.
//
// How many windows or chunks a share has: p2p_share_windows, p2p_leaf_chunks.  A
// list that would be cut into more than p2p_share_max shares takes twice or four
// times the windows a share, or whole chunks, as many as it needs.
#define P2P_SHARE_MAX_LEAF 4096  // larger leaves (coincident particles) are cut by sinks only
#define P2P_SHARE_STEPS 3        // windows per share tried: g, 2 g, 4 g

__device__ __forceinline__ void emit_whole_chunks(const DevTree &t, int A, int nA, int cnt, int per,
                                                  int groups, int64_t i0, int64_t r0) {
  const int T = (nA + 63) >> 6;
  for (int k = 0; k < groups; ++k)
    for (int q = 0; q < T; ++q)
      t.items[i0 + (int64_t)k * T + q] =
          P2PItem{A, q * 64, k * per, min(cnt, (k + 1) * per), 0, 1 << 30, k,
                  k ? (int32_t)(r0 + (int64_t)(k - 1) * nA) : -1};
}

#define PLAN_WAVES 4
#define PLAN_CHUNKS 256  // window counts of list chunks a wavefront keeps

// Source windows of the four chunks of 64 list entries from qb on, summed over
// the wavefront (0 past the list's end); their loads are independent.
__device__ __forceinline__ void chunk_windows(const DevTree &t, int off, int cnt, int qb,
                                              int (&nw)[4]) {
  const int lane = threadIdx.x & 63;
  int B[4], nb[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int q = qb + 64 * k + lane;
    B[k] = q < cnt ? t.p2p_src[off + q] : -1;
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) nb[k] = B[k] >= 0 ? t.nend[B[k]] - t.nbeg[B[k]] : 0;
#pragma unroll
  for (int k = 0; k < 4; ++k)
    nw[k] = (wave_sum(nb[k]) + t.p2p_src_window - 1) / t.p2p_src_window;
}

// Each wavefront plans npw consecutive cells, 64 at a time: a lane per cell,
// and for systems cut by windows the whole wavefront on one leaf after the
// other (it adds up the source counts of the leaf's chunks).  A workgroup
// allocates its items and rows with one atomic each.
// chunks: p2p_leaf_chunks of 1, 2 and 4 windows a share (the same in every lane).
__global__ __launch_bounds__(PLAN_WAVES * 64) void k_p2p_plan(DevTree t, int npw_min, int3 chunks) {
  __shared__ int s_items[PLAN_WAVES];
  __shared__ unsigned long long s_rows[PLAN_WAVES];
  __shared__ unsigned s_item0;
  __shared__ unsigned long long s_row0;
  __shared__ uint16_t s_nw[PLAN_WAVES][PLAN_CHUNKS];
  Header *h = t.hdr;
  if (h->overflow & OVF_WALK) return;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int nn = min(h->lvl_start[FMM_NLEVELS], (int)t.cap_nodes);
  const int nwaves = gridDim.x * PLAN_WAVES;
  const int npw = max((nn + nwaves - 1) / nwaves, npw_min);
  const int64_t first = (int64_t)(blockIdx.x * PLAN_WAVES + w) * npw;
  for (int b = 0; b < npw; b += 64) {
    const int64_t id = first + b + lane;
    const bool leaf = b + lane < npw && id < nn && t.nnchild[id] == 0;
    const int A = leaf ? (int)id : 0;
    int nA = 0, cnt = 0, off = 0, g = 0, groups = 0, share_max = 1, per = 1;
    if (leaf) {
      const int n = t.reqs[t.nreq[A]].n;
      nA = t.nend[A] - t.nbeg[A];
      cnt = t.p2p_cnt[A];
      off = t.p2p_off[A];
      g = p2p_share_windows(n);
      const int whole = g == 0 ? P2P_SHARE_CHUNKS : g == 1 ? chunks.x : g == 2 ? chunks.y : chunks.z;
      if (whole > 1 || t.uncut) g = 0;
      share_max = p2p_share_max(n);
      // list entries of a share of whole chunks
      per = nA > P2P_SHARE_MAX_LEAF || t.uncut
                ? max(cnt, 1)
                : 64 * p2p_share_chunks(cnt, share_max, max(whole, 1));
      groups = cnt <= per ? 1 : (cnt + per - 1) / per;
    }
    // leaves whose chunks are counted, and those cut by windows
    const unsigned long long counted =
        __ballot(leaf && g > 0 && nA <= P2P_SHARE_MAX_LEAF && cnt > 0);
    unsigned long long fine = counted;
    int used = 0;  // chunks counted so far in this batch (kept up to PLAN_CHUNKS)
    for (unsigned long long m = counted; m; m &= m - 1) {
      const int l = (int)__ffsll((long long)m) - 1;  // the same in every lane
      const int c = __builtin_amdgcn_readlane(cnt, l), o = __builtin_amdgcn_readlane(off, l);
      const int gl = __builtin_amdgcn_readlane(g, l);
      const int most = __builtin_amdgcn_readlane(share_max, l), gs = 31 - __clz(gl);  // gl: a power of two
      const int kept = used;
      int step = 0, shares = 0;
      for (;; ++step) {  // a second round at lists of more than p2p_share_max shares only
        shares = 0;
        used = kept;
        for (int qb = 0; qb < c; qb += 256) {
          int nw[4];
          chunk_windows(t, o, c, qb, nw);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            if (qb + 64 * k < c) {
              if (lane == 0 && used < PLAN_CHUNKS) s_nw[w][used] = (uint16_t)nw[k];
              ++used;
            }
            shares += (nw[k] + (gl << step) - 1) >> (gs + step);
          }
        }
        if (shares <= most || step == P2P_SHARE_STEPS - 1) break;
      }
      if (shares > most) {
        fine &= ~(1ull << l);
      } else if (lane == l) {
        g = gl << step;
        groups = max(1, shares);
      }
    }
    const int T = (nA + 63) >> 6;
    const int items = leaf ? groups * T : 0;
    const int rows = leaf ? (groups - 1) * nA : 0;
    int itot, rtot;
    const int ipos = wave_excl_scan_int(items, &itot);
    const int rpos = wave_excl_scan_int(rows, &rtot);
    if (lane == 0) {
      s_items[w] = itot;
      s_rows[w] = (unsigned long long)rtot;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      unsigned it = 0;
      unsigned long long r = 0;
      for (int k = 0; k < PLAN_WAVES; ++k) {
        it += (unsigned)s_items[k];
        r += s_rows[k];
      }
      s_item0 = it ? atomicAdd(&h->item_cursor, it) : 0u;
      s_row0 = r ? atomicAdd(&h->part_cursor, r) : 0ull;
      if ((int64_t)s_item0 + it > t.cap_items || (int64_t)(s_row0 + r) > t.cap_part) {
        atomicOr(&h->overflow, OVF_ITEMS);
        s_item0 = 0xffffffffu;
      }
    }
    __syncthreads();
    int64_t i0 = s_item0, r0 = (int64_t)s_row0;
    const bool fits = s_item0 != 0xffffffffu;
    for (int k = 0; k < w; ++k) {
      i0 += s_items[k];
      r0 += (int64_t)s_rows[k];
    }
    __syncthreads();  // the totals are rewritten by the next batch
    if (!fits) continue;  // uniform over the workgroup
    i0 += ipos;
    r0 += rpos;
    if (leaf) {
      t.nshare[A] = groups - 1;
      t.part_off[A] = (int32_t)r0;
      if (!(fine >> lane & 1)) emit_whole_chunks(t, A, nA, cnt, per, groups, i0, r0);
    }
    int at = 0;  // the batch's chunks in the order counted
    for (unsigned long long m = counted; m; m &= m - 1) {
      const int l = (int)__ffsll((long long)m) - 1;  // the same in every lane
      const int c = __builtin_amdgcn_readlane(cnt, l), o = __builtin_amdgcn_readlane(off, l);
      const int gl = __builtin_amdgcn_readlane(g, l);
      if (!(fine >> l & 1)) {
        at += (c + 63) >> 6;
        continue;
      }
      const int Al = __builtin_amdgcn_readlane(A, l), nl = __builtin_amdgcn_readlane(nA, l);
      const int Tl = __builtin_amdgcn_readlane(T, l);
      const int64_t il = (int64_t)readlane_u64((unsigned long long)i0, l);
      const int64_t rl = (int64_t)readlane_u64((unsigned long long)r0, l);
      int done = 0;  // shares of the chunks before
      for (int qb = 0; qb < c; qb += 64, ++at) {
        int nw;
        if (at < PLAN_CHUNKS) {
          nw = s_nw[w][at];
        } else {
          int n4[4];
          chunk_windows(t, o, min(c, qb + 64), qb, n4);
          nw = n4[0];
        }
        const int ng = (nw + gl - 1) / gl;
        for (int k = lane; k < ng * Tl; k += 64) {
          const int gk = done + k / Tl, q = k % Tl;
          t.items[il + (int64_t)gk * Tl + q] =
              P2PItem{Al, q * 64, qb, min(c, qb + 64), (k / Tl) * gl, (k / Tl + 1) * gl, gk,
                      gk ? (int32_t)(rl + (int64_t)(gk - 1) * nl) : -1};
        }
        done += ng;
      }
      if (done == 0)  // no sources
        for (int q = lane; q < Tl; q += 64)
          t.items[il + q] = P2PItem{Al, q * 64, 0, 0, 0, 0, 0, -1};
    }
  }
}

hipError_t launch_p2p_plan(const DevTree &t, const BuildArgs &a, hipStream_t s) {
  if (a.n <= 0) return hipSuccess;
  // a wavefront per cell where the systems are cut by windows (8 n / leaf_size
  // bounds the cells a context holds), a lane per cell where they are not: a
  // workgroup's items then follow 1024 cells in order, and so the XCDs' shares
  const int64_t cells = std::min<int64_t>(t.cap_nodes, (int64_t)a.n + 1024);
  int3 chunks;
  chunks.x = p2p_leaf_chunks(1, t.p2p_src_window, a.leaf_size);
  chunks.y = p2p_leaf_chunks(2, t.p2p_src_window, a.leaf_size);
  chunks.z = p2p_leaf_chunks(4, t.p2p_src_window, a.leaf_size);
  const int g = a.n_req == 1 ? p2p_share_windows(a.n_max) : 1;  // 1: of the smallest cut by windows
  const bool whole = a.n_max > P2P_SHARE_FINE_N || g == 0 ||
                     (g == 1 ? chunks.x : g == 2 ? chunks.y : chunks.z) > 1;
  const int npw = whole ? 64 : 1;
  const int blocks = (int)std::min<int64_t>(1024, (cells + npw * PLAN_WAVES - 1) / (npw * PLAN_WAVES));
  hipLaunchKernelGGL(k_p2p_plan, dim3(std::max(blocks, 1)), dim3(PLAN_WAVES * 64), 0, s, t, npw,
                     chunks);
  return hipGetLastError();
}

__global__ void k_reset_lists(Header *h) {
  int i = threadIdx.x;
  if (i == 0) {
    h->m2l_cursor = 0;
    h->p2p_cursor = 0;
    h->p2p_pairs = 0;
    h->overflow &= OVF_BUILD;
    h->item_cursor = 0;
    h->part_cursor = 0;
  }
  if (i < FMM_NLEVELS) h->open_cursor[i] = 0;
}

hipError_t launch_reset_lists(const DevTree &t, hipStream_t s) {
  hipLaunchKernelGGL(k_reset_lists, dim3(1), dim3(64), 0, s, t.hdr);
  return hipGetLastError();
}

// the whole walk in one launch; cells: an estimate (or bound) of the tree's
// cells, for the grid; first: the header is as the build left it
hipError_t launch_traverse_paths(const DevTree &t, const BuildArgs &a, int cells, bool first,
                                 hipStream_t s) {
  if (!first) launch_reset_lists(t, s);
  if (a.n <= 0) return hipGetLastError();
  if (a.tm) a.tm->start(PH_WALK, s);
  const int blocks = std::min(std::max(cells, 1), GRID_WAVES / WALK_WAVES);
  hipLaunchKernelGGL(k_walk_paths, dim3(blocks), dim3(WALK_WAVES * 64), 0, s, t,
                     a.theta * a.theta, a.eps);
  if (a.tm) a.tm->stop(s);
  return hipGetLastError();
}

hipError_t launch_traverse(const DevTree &t, const BuildArgs &a, hipStream_t s) {
  launch_reset_lists(t, s);
  if (a.n <= 0) return hipGetLastError();
  const double th2 = a.theta * a.theta;
  if (a.tm) a.tm->start(PH_WALK, s);
  for (int l = 0; l <= a.depth; ++l) {
    int ps = l == 0 ? 0 : a.lvl_host[l - 1];
    int pe = l == 0 ? a.n_req : a.lvl_host[l];
    int nw = pe - ps;
    if (nw <= 0) continue;
    if (nw <= WALK_GROUP_LEVEL)
      hipLaunchKernelGGL(k_walk_level, dim3(nw), dim3(WALK_WAVES * 64), 0, s, t, l, ps, pe, th2,
                         a.eps);
    else
      hipLaunchKernelGGL(k_walk_waves, dim3((nw + TRAV_WAVES - 1) / TRAV_WAVES),
                         dim3(TRAV_WAVES * 64), 0, s, t, l, ps, pe, th2, a.eps);
  }
  if (a.tm) a.tm->stop(s);
  return hipGetLastError();
}

// Levels 0..levels with the bounds of each read on the device; the grid fills
// the chip for large trees.
hipError_t launch_traverse_dev(const DevTree &t, const BuildArgs &a, int levels, hipStream_t s) {
  launch_reset_lists(t, s);
  if (a.n <= 0) return hipGetLastError();
  const double th2 = a.theta * a.theta;
  const int blocks = std::min(2048, std::max(16, a.n / 512));
  if (a.tm) a.tm->start(PH_WALK, s);
  for (int l = 0; l <= levels && l <= FMM_MAXLEVEL; ++l)
    hipLaunchKernelGGL(k_walk_waves_dev, dim3(blocks), dim3(TRAV_WAVES * 64), 0, s, t, l, th2,
                       a.eps);
  if (a.tm) a.tm->stop(s);
  return hipGetLastError();
}
