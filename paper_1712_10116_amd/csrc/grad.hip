// Force gradient d a_i / d x_i (the tidal tensor) of every active particle,
// the quantity the forward fourth-order integrator of Sec. 4.1 needs from the
// FMM, computed on the tree, lists and local expansions of the evaluation
// just made: minus the Hessian of the leaf's local expansion, plus for every
// particle of every leaf in the sink leaf's P2P list the derivative of
// m g(r) d (d = x_j - x_i) with respect to x_i, -m (g I + (dg/dr)/r d d^T).
// Output SoA, 6 rows of n: xx, yy, zz, xy, xz, yz, in active order.
//
// Both parts run in the evaluation's precision (the near part's pair terms
// on offsets from the sink leaf's centre, summed into FP64 per source leaf).
#include "common.h"
#include "expansion.h"

#include <type_traits>

namespace {

constexpr int CA[6] = {0, 1, 2, 0, 0, 1}, CB[6] = {0, 1, 2, 1, 2, 2};

// g = psi'(r)/r and h = (dg/dr)/r of the pair kernel.  Wendland C2 (Eq. 8):
// inside the radius g = (21u^5 - 90u^4 + 140u^3 - 84u^2 + 14)/eps^3 and h =
// (105u^3 - 360u^2 + 420u - 168)/eps^5 (u = r/eps), outside 1/r^3 and
// -3/r^5; Plummer: s^(-3/2) and -3 s^(-5/2), s = r^2 + eps^2.
template <typename R, int KERNEL>
__device__ __forceinline__ void pair_gh(R r2, R eps, R ie, R &g, R &h) {
  if (KERNEL == 1) {
    const R rs = fast_rsqrt<R>(r2 + eps * eps), is = rs * rs;
    g = is * rs;
    h = R(-3) * g * is;
  } else {
    const R ir = fast_rsqrt<R>(r2);
    if (r2 >= eps * eps) {
      const R ir2 = ir * ir;
      g = ir2 * ir;
      h = R(-3) * g * ir2;
    } else {
      const R u = r2 > R(0) ? r2 * ir * ie : R(0), ie3 = ie * ie * ie;
      g = ((((R(21) * u - R(90)) * u + R(140)) * u - R(84)) * u * u + R(14)) * ie3;
      h = (((R(105) * u - R(360)) * u + R(420)) * u - R(168)) * ie3 * ie * ie;
    }
  }
}

// A staged source: its offset from the sink leaf's centre and its mass, in R.
template <typename R>
struct alignas(4 * sizeof(R)) SrcR {
  R x, y, z, m;
};

// What fills the slots past a leaf's end: no mass, so far away that the pair
// kernel stays finite (and its products with the mass zero) in R.
template <typename R>
__device__ __forceinline__ SrcR<R> far_source() {
  const R far = sizeof(R) == 4 ? R(1e15) : R(1e150);  // as P2P pads
  return SrcR<R>{far, far, far, R(0)};
}

// The entries of its leaf's P2P list that a near-field work item covers here.
// The items are those of P2P (groups of 64 sinks, shares of the list), but the
// sums below run leaf by leaf, so share grp of ng takes the grp-th part of the
// list's entries.
struct ItemRange {
  int A, tb, q0, q1, grp, part;
};
__device__ __forceinline__ ItemRange item_range(const DevTree &t, int it) {
  const P2PItem im = t.items[it];
  const int64_t cnt = t.p2p_cnt[im.A];
  const int ng = t.nshare[im.A] + 1;
  return {im.A, im.tb, (int)(cnt * im.grp / ng), (int)(cnt * (im.grp + 1) / ng), im.grp, im.part};
}

// near part: one wavefront (and workgroup) per work item, lanes over its sinks
// (and, for 32 sinks or fewer, over 2-16 phases of the sources), each source
// leaf staged through LDS 64 particles at a time as offsets from the sink
// leaf's centre in R (FP32 in the mixed form: cell-local offsets, as in the
// forces' P2P); pair terms in R, summed in R over one source leaf and then into
// FP64.  Per pair: m h d (3 products) and six FMAs of it with d for the h d d^T
// part; the g I part is one sum of m g per source leaf.  The self pair (d = 0)
// is masked by a select, so an infinite g or h there never reaches a sum; only
// the leaf itself, which alone holds it, runs the form with the select (seven of
// 41 instructions a pair in FP64: 65,536 particles, this kernel and the
// vector-source one 364 -> 339 us at most, solve and field 1656 -> 1567).
// Written in sorted order to stage (6 rows of stride cap_n), shares past the
// first to gpart (6 values a row); k_l2p_grad adds them and the far part and
// writes each particle's tensor once in active order.  One wavefront per leaf
// had left the kernel waiting for the longest lists (65,536-particle Plummer
// sphere, leaf 64, FP64, this kernel and the vector-source one together: 2.6 ->
// 0.75 ms).
template <typename R, int KERNEL>
__global__ __launch_bounds__(64) void k_p2p_grad(DevTree t, double eps,
                                                 double *__restrict__ stage,
                                                 double *__restrict__ gpart) {
  const int lane = threadIdx.x;
  // neighbouring leaves, which share most of their sources, on one XCD
  const int first = __builtin_amdgcn_readfirstlane(xcd_block<128>(blockIdx.x, gridDim.x));
  const R reps = (R)eps, ie = eps > 0 ? (R)(1.0 / eps) : R(0);
  __shared__ SrcR<R> st[64];
  const int n_items = (int)t.hdr->item_cursor;
  for (int it = first; it < n_items; it += gridDim.x) {
    const ItemRange im = item_range(t, it);
    const int A = im.A, tb = im.tb;
    const int bA = t.nbeg[A], nA = t.nend[A] - bA;
    const int loff = t.p2p_off[A];
    const double4 gA = t.ngeo[A];
    {
      // lanes = (sink, phase): nph phases share each sink and take every
      // nph-th source, so a leaf of fewer than 64 sinks still fills the wave
      const int ns = min(64, nA - tb);
      const int nph = ns <= 4 ? 16 : ns <= 8 ? 8 : ns <= 16 ? 4 : ns <= 32 ? 2 : 1;
      const int ti = lane / nph, ph = lane % nph;
      const bool valid = ti < ns;
      const int i = bA + tb + (valid ? ti : 0);
      // the sink's offset, formed exactly as a staged source's
      const R xi = (R)(t.sx[i] - gA.x), yi = (R)(t.sy[i] - gA.y), zi = (R)(t.sz[i] - gA.z);
      double G[6] = {0, 0, 0, 0, 0, 0};
      for (int q = im.q0; q < im.q1; ++q) {
        const int B = t.p2p_src[loff + q];
        const int eB = t.nend[B];
        R Gs[6] = {0, 0, 0, 0, 0, 0};
        R Gg = 0;
        for (int jb = t.nbeg[B]; jb < eB; jb += 64) {
          // up to 64 sources of leaf B staged in LDS by the wave's lanes
          const int nj = min(64, eB - jb);
          SrcR<R> e = far_source<R>();
          if (lane < nj)
            e = SrcR<R>{(R)(t.sx[jb + lane] - gA.x), (R)(t.sy[jb + lane] - gA.y),
                        (R)(t.sz[jb + lane] - gA.z), (R)t.sm[jb + lane]};
          st[lane] = e;
          __builtin_amdgcn_wave_barrier();
          // every lane takes the same number of steps: slot ph + k, k = 0, nph,
          // ..., stays below 64 (nph divides 64); slots past nj hold no mass
          auto pairs = [&](auto own) {
            const int si = i - jb - ph;
            for (int k = 0; k < nj; k += nph) {
              const SrcR<R> sv = st[ph + k];
              const R dx = sv.x - xi, dy = sv.y - yi, dz = sv.z - zi;
              const R r2 = fma(dz, dz, fma(dy, dy, dx * dx));
              R g, h;
              pair_gh<R, KERNEL>(r2, reps, ie, g, h);
              const bool skip = own && k == si;
              const R mg = skip ? R(0) : sv.m * g;
              const R mh = skip ? R(0) : sv.m * h;
              const R hx = mh * dx, hy = mh * dy, hz = mh * dz;
              Gg += mg;
              Gs[0] = fma(-hx, dx, Gs[0]);
              Gs[1] = fma(-hy, dy, Gs[1]);
              Gs[2] = fma(-hz, dz, Gs[2]);
              Gs[3] = fma(-hx, dy, Gs[3]);
              Gs[4] = fma(-hx, dz, Gs[4]);
              Gs[5] = fma(-hy, dz, Gs[5]);
            }
          };
          if (B == A)
            pairs(std::true_type{});
          else
            pairs(std::false_type{});
          __builtin_amdgcn_wave_barrier();
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) G[c] += (double)(Gs[c] - Gg);
#pragma unroll
        for (int c = 3; c < 6; ++c) G[c] += (double)Gs[c];
      }
      // the phases of a sink are consecutive lanes: fold them onto phase 0
      for (int o = nph >> 1; o > 0; o >>= 1)
#pragma unroll
        for (int c = 0; c < 6; ++c) G[c] += __shfl_xor(G[c], o, 64);
      if (valid && ph == 0) {
        const int64_t cap = t.cap_n;
        double *out = im.grp == 0 ? stage + i : gpart + 6 * (int64_t)(im.part + (i - bA));
        const int64_t stride = im.grp == 0 ? cap : 1;
#pragma unroll
        for (int c = 0; c < 6; ++c) out[c * stride] = G[c];
      }
    }
  }
}

// minus the Hessian of the leaf's local expansion (coefficients scaled by
// h^|n|, so the second derivatives carry 1/h^2) added to the near part staged
// in sorted order, written to grad in active order (zero for p = 1: the
// Hessian of a degree-1 expansion vanishes)
template <typename T, int P>
__global__ __launch_bounds__(FMM_BLOCK) void k_l2p_grad(DevTree t, int n,
                                                        const double *__restrict__ stage,
                                                        const double *__restrict__ gpart,
                                                        double *__restrict__ grad, int64_t nq,
                                                        int32_t off) {
  constexpr MI<P> mi{};
  constexpr int K = MI<P>::K;
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  const int leaf = t.leaf_of[j];
  const double4 g = t.ngeo[leaf];
  const double ih = 1.0 / g.w;
  T mono[K], Lt[K];
  monomials<T, P>((T)((t.sx[j] - g.x) * ih), (T)((t.sy[j] - g.y) * ih),
                  (T)((t.sz[j] - g.z) * ih), mono);
  const T *row = (const T *)t.L + (size_t)leaf * t.kmax;
#pragma unroll
  for (int k = 0; k < K; ++k) Lt[k] = row[k];
  T H[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int k = 0; k < K; ++k) {
    if (mi.deg[k] + 2 > P) continue;
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      const int a = mi.x[k] + (CA[c] == 0) + (CB[c] == 0);
      const int b = mi.y[k] + (CA[c] == 1) + (CB[c] == 1);
      const int e = mi.z[k] + (CA[c] == 2) + (CB[c] == 2);
      H[c] = fma(Lt[mi.at(a, b, e)], mono[k], H[c]);
    }
  }
  const int64_t k = t.slot[j] - off, cap = t.cap_n;
  const double s2 = ih * ih;
  double G[6];
#pragma unroll
  for (int c = 0; c < 6; ++c) G[c] = stage[c * cap + j];
  const int ne = t.nshare[leaf];
  if (ne > 0) {  // the near part's further shares, in share order
    const int b = t.nbeg[leaf], na = t.nend[leaf] - b;
    const double *row = gpart + 6 * (int64_t)(t.part_off[leaf] + (j - b));
    for (int e = 0; e < ne; ++e)
#pragma unroll
      for (int c = 0; c < 6; ++c) G[c] += row[6 * (int64_t)e * na + c];
  }
#pragma unroll
  for (int c = 0; c < 6; ++c) grad[c * nq + k] = G[c] - (double)H[c] * s2;
}

template <typename T, int P>
void launch_l2p_grad(const DevTree &t, int n, const double *stage, const double *gpart,
                     double *grad, hipStream_t s) {
  hipLaunchKernelGGL((k_l2p_grad<T, P>), dim3((n + FMM_BLOCK - 1) / FMM_BLOCK), dim3(FMM_BLOCK),
                     0, s, t, n, stage, gpart, grad, (int64_t)n, 0);
}

template <typename T, int KERNEL>
bool dispatch_grad(const DevTree &t, int n_nodes, int n, int p, double eps, double *stage,
                   double *gpart, double *grad, hipStream_t s) {
  hipLaunchKernelGGL((k_p2p_grad<T, KERNEL>), dim3(p2p_grid_items(n, n_nodes)), dim3(64), 0, s, t,
                     eps, stage, gpart);
  switch (p) {
    case 1: launch_l2p_grad<T, 1>(t, n, stage, gpart, grad, s); return true;
    case 2: launch_l2p_grad<T, 2>(t, n, stage, gpart, grad, s); return true;
    case 3: launch_l2p_grad<T, 3>(t, n, stage, gpart, grad, s); return true;
    case 4: launch_l2p_grad<T, 4>(t, n, stage, gpart, grad, s); return true;
    case 5: launch_l2p_grad<T, 5>(t, n, stage, gpart, grad, s); return true;
    case 6: launch_l2p_grad<T, 6>(t, n, stage, gpart, grad, s); return true;
    default: return false;
  }
}

// Near field of the vector-source pass: for every sink i the sum over the
// particles j of its leaf's P2P partners (j != i) of m_j H(x_i - x_j) v_j,
// H = g I + h d d^T the pair Hessian, and of m_j v_j . grad psi(x_i - x_j)
// = -m_j g (v_j . d), d = x_j - x_i.  Written to near[] in sorted order with
// the sign of an acceleration (minus the field) so that L2P adds the far
// field's gradient the same way (shares past the first to the partial rows, as
// P2P's).  Layout as k_p2p_grad: one wavefront per work item, (sink, phase)
// lanes, each source leaf staged through LDS 64 particles at a time (offsets
// from the sink leaf's centre, mass and vector in R), pair terms in R, summed
// in R over one source leaf and then into FP64.
template <typename R, int KERNEL>
__global__ __launch_bounds__(64) void k_p2p_dip(DevTree t, double eps,
                                                const double *__restrict__ dv) {
  const int lane = threadIdx.x;
  // neighbouring leaves, which share most of their sources, on one XCD
  const int first = __builtin_amdgcn_readfirstlane(xcd_block<128>(blockIdx.x, gridDim.x));
  const R reps = (R)eps, ie = eps > 0 ? (R)(1.0 / eps) : R(0);
  const int64_t cap = t.cap_n;
  __shared__ SrcR<R> sx[64], sv[64];
  const int n_items = (int)t.hdr->item_cursor;
  for (int it = first; it < n_items; it += gridDim.x) {
    const ItemRange im = item_range(t, it);
    const int A = im.A, tb = im.tb;
    const int bA = t.nbeg[A], nA = t.nend[A] - bA;
    const int loff = t.p2p_off[A];
    const double4 gA = t.ngeo[A];
    {
      const int ns = min(64, nA - tb);
      const int nph = ns <= 4 ? 16 : ns <= 8 ? 8 : ns <= 16 ? 4 : ns <= 32 ? 2 : 1;
      const int ti = lane / nph, ph = lane % nph;
      const bool valid = ti < ns;
      const int i = bA + tb + (valid ? ti : 0);
      const R xi = (R)(t.sx[i] - gA.x), yi = (R)(t.sy[i] - gA.y), zi = (R)(t.sz[i] - gA.z);
      double U[4] = {0, 0, 0, 0};
      for (int q = im.q0; q < im.q1; ++q) {
        const int B = t.p2p_src[loff + q];
        const int eB = t.nend[B];
        R Us[4] = {0, 0, 0, 0};
        for (int jb = t.nbeg[B]; jb < eB; jb += 64) {
          const int nj = min(64, eB - jb);
          SrcR<R> ex = far_source<R>(), ev{R(0), R(0), R(0), R(0)};
          if (lane < nj) {
            const int j = jb + lane;
            ex = SrcR<R>{(R)(t.sx[j] - gA.x), (R)(t.sy[j] - gA.y), (R)(t.sz[j] - gA.z),
                         (R)t.sm[j]};
            ev = SrcR<R>{(R)dv[j], (R)dv[cap + j], (R)dv[2 * cap + j], R(0)};
          }
          sx[lane] = ex;
          sv[lane] = ev;
          __builtin_amdgcn_wave_barrier();
          // same number of steps on every lane, as in k_p2p_grad
          auto pairs = [&](auto own) {
            const int si = i - jb - ph;
            for (int k = 0; k < nj; k += nph) {
              const SrcR<R> p = sx[ph + k], v = sv[ph + k];
              const R dx = p.x - xi, dy = p.y - yi, dz = p.z - zi;
              const R r2 = fma(dz, dz, fma(dy, dy, dx * dx));
              R g, h;
              pair_gh<R, KERNEL>(r2, reps, ie, g, h);
              const bool skip = own && k == si;
              const R mg = skip ? R(0) : p.m * g;
              const R mh = skip ? R(0) : p.m * h;
              const R dvv = fma(dz, v.z, fma(dy, v.y, dx * v.x));
              const R mhd = mh * dvv;
              Us[0] = fma(mg, v.x, fma(mhd, dx, Us[0]));
              Us[1] = fma(mg, v.y, fma(mhd, dy, Us[1]));
              Us[2] = fma(mg, v.z, fma(mhd, dz, Us[2]));
              Us[3] = fma(-mg, dvv, Us[3]);
            }
          };
          if (B == A)
            pairs(std::true_type{});
          else
            pairs(std::false_type{});
          __builtin_amdgcn_wave_barrier();
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) U[c] += (double)Us[c];
      }
      for (int o = nph >> 1; o > 0; o >>= 1)
#pragma unroll
        for (int c = 0; c < 4; ++c) U[c] += __shfl_xor(U[c], o, 64);
      if (valid && ph == 0) {
        if (im.grp == 0) {
          t.near[i] = -U[0];
          t.near[cap + i] = -U[1];
          t.near[2 * cap + i] = -U[2];
          t.near[3 * cap + i] = U[3];
        } else {
          t.part[im.part + (i - bA)] = make_double4(-U[0], -U[1], -U[2], U[3]);
        }
      }
    }
  }
}

}  // namespace

hipError_t launch_p2p_dipole(const DevTree &t, int n_nodes, int n, int kernel, bool mixed,
                             double eps, const double *dv, hipStream_t s) {
  const dim3 grid(p2p_grid_items(n, n_nodes)), blk(64);
  if (mixed) {
    if (kernel == 1)
      hipLaunchKernelGGL((k_p2p_dip<float, 1>), grid, blk, 0, s, t, eps, dv);
    else
      hipLaunchKernelGGL((k_p2p_dip<float, 0>), grid, blk, 0, s, t, eps, dv);
  } else {
    if (kernel == 1)
      hipLaunchKernelGGL((k_p2p_dip<double, 1>), grid, blk, 0, s, t, eps, dv);
    else
      hipLaunchKernelGGL((k_p2p_dip<double, 0>), grid, blk, 0, s, t, eps, dv);
  }
  return hipGetLastError();
}

// One system's tree (request 0 at slot offset 0), n active particles.
hipError_t launch_force_gradient(const DevTree &t, int n_nodes, int n, int p, int kernel,
                                 bool mixed, double eps, double *stage, double *gpart,
                                 double *grad, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  bool ok;
  if (mixed)
    ok = kernel == 1 ? dispatch_grad<float, 1>(t, n_nodes, n, p, eps, stage, gpart, grad, s)
                     : dispatch_grad<float, 0>(t, n_nodes, n, p, eps, stage, gpart, grad, s);
  else
    ok = kernel == 1 ? dispatch_grad<double, 1>(t, n_nodes, n, p, eps, stage, gpart, grad, s)
                     : dispatch_grad<double, 0>(t, n_nodes, n, p, eps, stage, gpart, grad, s);
  if (!ok) return hipErrorInvalidValue;
  return hipGetLastError();
}
