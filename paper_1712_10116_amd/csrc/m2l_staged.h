// M2L with the sources' rows staged in LDS (included by eval.hip).
#pragma once
#include <utility>

#include "common.h"
#include "expansion.h"

// M2L in FP64 at p >= 5: the same sums, a wavefront per target cell and lanes
// over its sources, with the sources' rows staged in LDS.  A source's row is 288
// to 672 bytes, a lane each, so reading the rows lane by lane looks up 64 cache
// lines per load instruction: at p 6 that took longer than the arithmetic, and
// the row, the derivatives and the sums together overflowed 256 registers, so
// that half of the instructions moved values between register files.  Here four
// lanes read 64 consecutive bytes of a row, straight into LDS (16 rows per
// instruction), while the derivatives are formed; moments are read from LDS as
// they are used.  The factors (-beta)^|m| enter as a Horner scheme in beta, so
// that moments are used as stored.
//
// Slot c of a row's 64-byte piece holds its 16-byte unit c ^ (row / 4 mod 4), so
// that the 16 rows of a group lie on different banks.  For p 6 with softening the
// last degree (a third of the row) is read directly, and used once: with it the
// row would exceed the LDS of four workgroups per CU.
// M2L alone, lane-per-row -> staged: 300,007 particles, leaf 40, p 6, 250 -> 155
// us; 65,536, leaf 64, p 6, softened, 345 -> 150 (VALU issuing 64%, was 42%, of
// it a third moves between register files, was half).
template <int P, bool HARM>
struct M2LRow {
  static constexpr int N = HARM ? HI<P>::KH : MI<P>::K;  // moments of a row
  static constexpr int DEG = !HARM && P > 5 ? P - 1 : P;  // highest degree staged
  static constexpr int STAGED = HARM ? HI<P>::KH : MI<DEG>::K;
  static constexpr int UNITS = (STAGED + 1) / 2;
  static constexpr int PIECES = (UNITS + 3) / 4;
};

// The operations for the outputs of degree NLO .. NHI, in order (compile time):
// s[n] *= -beta before each lower degree of moments, then s[n] += M[j] D[nm].
template <int P, bool HARM, int NLO, int NHI>
struct M2LOps {
  enum { SCALE, FIRST, ADD };
  static constexpr int walk(M2LOps *o) {
    constexpr MI<P> mi{};
    constexpr HI<P> hi{};
    int c = 0;
    for (int dm = P - NLO; dm >= 0; --dm) {
      for (int n = 0; n < MI<P>::K; ++n)
        if (mi.deg[n] >= NLO && mi.deg[n] <= NHI && (!HARM || mi.z[n] <= 1) &&
            dm < P - mi.deg[n]) {
          if (o) {
            o->kind[c] = SCALE;
            o->n[c] = n;
          }
          ++c;
        }
      bool first = true;
      for (int j = 0; j < M2LRow<P, HARM>::N; ++j) {
        const int m = HARM ? hi.full[j] : j;
        if (mi.deg[m] != dm) continue;
        for (int n = 0; n < MI<P>::K; ++n) {
          if (mi.deg[n] < NLO || mi.deg[n] > NHI || mi.deg[n] + dm > P || (HARM && mi.z[n] > 1))
            continue;
          if (o) {
            o->kind[c] = first && dm == P - mi.deg[n] ? FIRST : ADD;
            o->n[c] = n;
            o->j[c] = j;
            o->nm[c] = mi.at(mi.x[n] + mi.x[m], mi.y[n] + mi.y[m], mi.z[n] + mi.z[m]);
          }
          ++c;
        }
        first = false;
      }
    }
    return c;
  }
  static constexpr int N = 2048;
  int kind[N], n[N], j[N], nm[N], count;
  constexpr M2LOps() : kind(), n(), j(), nm(), count() { count = walk(this); }
};

template <int P, bool HARM, int NLO, int NHI>
inline constexpr M2LOps<P, HARM, NLO, NHI> m2l_op_list{};

template <int P, bool HARM, int NLO, int NHI, int C>
__device__ __forceinline__ void m2l_op(const double2 *const (&rb)[4], const double *direct,
                                       double mbeta, const double (&D)[MI<P>::K],
                                       double (&s)[MI<P>::K]) {
  typedef M2LRow<P, HARM> Row;
  typedef M2LOps<P, HARM, NLO, NHI> Ops;
  constexpr const Ops &ops = m2l_op_list<P, HARM, NLO, NHI>;
  constexpr int kind = ops.kind[C], n = ops.n[C], j = ops.j[C], nm = ops.nm[C];
  if constexpr (kind == Ops::SCALE) {
    s[n] *= mbeta;
  } else {
    double M;
    if constexpr (j < Row::STAGED) {
      const double2 v = rb[(j >> 1) & 3][(j >> 3) * 64];
      M = (j & 1) ? v.y : v.x;
    } else {
      M = direct[j - Row::STAGED];
    }
    s[n] = kind == Ops::FIRST ? M * D[nm] : fma(M, D[nm], s[n]);
  }
}

// every operation expanded by the front end: loops of this length are not
// unrolled in full
template <int P, bool HARM, int NLO, int NHI, int... C>
__device__ __forceinline__ void m2l_ops(std::integer_sequence<int, C...>,
                                        const double2 *const (&rb)[4], const double *direct,
                                        double mbeta, const double (&D)[MI<P>::K],
                                        double (&s)[MI<P>::K]) {
  const int done[] = {(m2l_op<P, HARM, NLO, NHI, C>(rb, direct, mbeta, D, s), 0)...};
  (void)done;
}

template <int P, bool HARM, int NLO, int NHI>
__device__ __forceinline__ void m2l_degrees(const double2 *const (&rb)[4], const double *direct,
                                            double mbeta, const double (&D)[MI<P>::K],
                                            double (&acc)[MI<P>::K]) {
  constexpr MI<P> mi{};
  double s[MI<P>::K];
  m2l_ops<P, HARM, NLO, NHI>(
      std::make_integer_sequence<int, m2l_op_list<P, HARM, NLO, NHI>.count>{}, rb, direct, mbeta,
      D, s);
#pragma unroll
  for (int n = 0; n < MI<P>::K; ++n)
    if (mi.deg[n] >= NLO && mi.deg[n] <= NHI && (!HARM || mi.z[n] <= 1)) acc[n] += s[n];
}

template <int P, int KERNEL>
__global__ __launch_bounds__(64) void k_m2l_staged(DevTree t, int n_nodes, double eps) {
  constexpr bool HARM = KERNEL == 0;
  constexpr int K = MI<P>::K;
  constexpr MI<P> mi{};
  typedef M2LRow<P, HARM> Row;
  constexpr int ND = Row::N - Row::STAGED;  // moments read directly
  __shared__ double2 rows[4 * Row::PIECES * 64];  // [group of 16 rows][piece][lane]
  const int lane = threadIdx.x;
  const double *M = (const double *)(HARM ? t.Mh : t.M);
  const int stride = HARM ? t.khmax : t.kmax;
  double *L = (double *)t.L;
  const double2 *rb[4];
#pragma unroll
  for (int c = 0; c < 4; ++c)
    rb[c] = rows + (lane >> 4) * (Row::PIECES * 64) + (lane & 15) * 4 +
            (c ^ ((lane >> 2) & 3));
  n_nodes = node_count<OVF_WALK>(t, n_nodes);
  for (int A = xcd_block<128>(blockIdx.x, gridDim.x); A < n_nodes; A += gridDim.x) {
    if (skipped(t, A)) continue;
    const double4 gA = t.ngeo[A];
    const double ih = 1.0 / gA.w;
    const double e2 = KERNEL == 1 ? (eps * ih) * (eps * ih) : 0.0;
    const int off = t.m2l_off[A], cnt = t.m2l_cnt[A];
    double acc[K];
#pragma unroll
    for (int k = 0; k < K; ++k) acc[k] = 0.0;
    // a lane without a source takes the last one's place, and its sums are not
    // used; the next source's index is read one iteration ahead
    int Bn = cnt > 0 ? t.m2l_src[off + min(lane, cnt - 1)] : 0;
    for (int q0 = 0; q0 < cnt; q0 += 64) {
      const int B = Bn;
      if (q0 + 64 < cnt) Bn = t.m2l_src[off + min(q0 + 64 + lane, cnt - 1)];
      const double4 gB = t.ngeo[B];
      double direct[ND > 0 ? ND : 1];
      if (ND > 0) {
        const double *row = M + (size_t)B * stride + Row::STAGED;
#pragma unroll
        for (int j = 0; j < ND; ++j) direct[j] = row[j];
      }
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        // this lane's row of the group, and the unit of it that it reads
        const int Br = __shfl(B, g * 16 + (lane >> 2), 64);
        const double *row = M + (size_t)Br * stride;
        const int c = (lane & 3) ^ (lane >> 4);
#pragma unroll
        for (int s = 0; s < Row::PIECES; ++s) {
          const int u = min(4 * s + c, Row::UNITS - 1);
          __builtin_amdgcn_global_load_lds(
              (const __attribute__((address_space(1))) void *)(row + 2 * u),
              (__attribute__((address_space(3))) void *)(rows + (g * Row::PIECES + s) * 64), 16,
              0, 0);
        }
      }
      const double X = (gA.x - gB.x) * ih, Y = (gA.y - gB.y) * ih, Z = (gA.z - gB.z) * ih;
      double D[K];
      derivatives_in_place<P, HARM ? 1 : P>(X, Y, Z, e2, D);
      if (HARM) {
#pragma unroll
        for (int k = 0; k < K; ++k)
          if (mi.z[k] == 2)
            D[k] = -D[mi.at(mi.x[k] + 2, mi.y[k], 0)] - D[mi.at(mi.x[k], mi.y[k] + 2, 0)];
      }
      const double mbeta = -(gB.w * ih);
      __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the rows are in LDS
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      if (q0 + lane < cnt) {
        m2l_degrees<P, HARM, 0, 1>(rb, direct, mbeta, D, acc);
        asm volatile("" ::: "memory");  // moments read again rather than held
        m2l_degrees<P, HARM, 2, P>(rb, direct, mbeta, D, acc);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the rows have been read
      __builtin_amdgcn_wave_barrier();
    }
    // The sums over the lanes, through LDS: a lane per coefficient, PART at a time
    double *buf = (double *)rows;
    constexpr int PART = 32;
    double mine[(K + 63) / 64];
#pragma unroll
    for (int i = 0; i < (K + 63) / 64; ++i) mine[i] = 0.0;
#pragma unroll
    for (int k0 = 0; k0 < K; k0 += PART) {
#pragma unroll
      for (int k = k0; k < k0 + PART && k < K; ++k)
        if (!HARM || mi.z[k] <= 1) buf[(k - k0) * 65 + lane] = acc[k];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      // lanes l and l + 32: the two halves of coefficient k0 + l mod 32
      double v = 0.0;
      const double *b = buf + (lane & 31) * 65 + (lane >> 5) * 32;
      if (k0 + (lane & 31) < K) {
#pragma unroll 8
        for (int i = 0; i < 32; ++i) v += b[i];
      }
      v += __shfl_xor(v, 32, 64);
      if ((lane >> 5) == ((k0 / PART) & 1)) mine[k0 / 64] = v * ih;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    if (HARM) {  // the coefficients with n_z >= 2, by one lane
#pragma unroll
      for (int i = 0; i < (K + 63) / 64; ++i)
        if (64 * i + lane < K) buf[64 * i + lane] = mine[i];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      if (lane == 0) {
        double l[K];
#pragma unroll
        for (int k = 0; k < K; ++k) l[k] = mi.z[k] <= 1 ? buf[k] : 0.0;
        unfold_locals<double, P>(l);
#pragma unroll
        for (int k = 0; k < K; ++k)
          if (mi.z[k] > 1) buf[k] = l[k];
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int i = 0; i < (K + 63) / 64; ++i)
        if (64 * i + lane < K) mine[i] = buf[64 * i + lane];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
#pragma unroll
    for (int i = 0; i < (K + 63) / 64; ++i)
      if (64 * i + lane < K) L[(size_t)A * t.kmax + 64 * i + lane] = mine[i];
    __builtin_amdgcn_s_waitcnt(0xC07F);
    __builtin_amdgcn_wave_barrier();
  }
}
