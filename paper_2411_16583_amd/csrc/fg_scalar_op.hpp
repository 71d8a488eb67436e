// Operators of the scalar problems in real space: the phase-field operator of
// eq. (32) and the Fick operator of eq. (43), by the 7-point and the forward /
// backward difference stencils.
#pragma once
#include "fg_launch.hpp"

namespace fg {

// Voxel neighbours along each axis (periodic) as offsets within the field.
struct Nbr {
  long c;         // the voxel
  long p[3], m[3];  // + e_j, - e_j relative to it
};
__device__ __forceinline__ Nbr neighbours(const Grid3& g, int i0, int i1, int i2) {
  const long s0 = (long)g.n1 * g.n2, s1 = g.n2;
  Nbr n;
  n.c = i0 * s0 + i1 * s1 + i2;
  n.p[0] = (i0 + 1 == g.n0) ? s0 - s0 * g.n0 : s0;
  n.m[0] = (i0 == 0) ? s0 * g.n0 - s0 : -s0;
  n.p[1] = (i1 + 1 == g.n1) ? s1 - s0 : s1;
  n.m[1] = (i1 == 0) ? s0 - s1 : -s1;
  n.p[2] = (i2 + 1 == g.n2) ? 1 - s1 : 1;
  n.m[2] = (i2 == 0) ? s1 - 1 : -1;
  return n;
}

// L(v) = grad+^T ( Aplus grad+ v ) at a voxel (forward differences, their
// adjoint for the divergence).  With div = -grad+^T and Aplus = -M c(1-c) C^-1
// this is div[ M c(1-c) C^-1 grad v ], the operator of eq. (43).
__device__ __forceinline__ double fick_L(const double* __restrict__ v, const double* __restrict__ A6, const Grid3& g,
                                         long N, const Nbr& n) {
  const double ih[3] = {g.ih0, g.ih1, g.ih2};
  // Aplus component index for (j, k)
  constexpr int aidx[9] = {0, 5, 4, 5, 1, 3, 4, 3, 2};
  const double* vc = v + n.c;
  const double* ac = A6 + n.c;
  double gr[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) gr[k] = (vc[n.p[k]] - vc[0]) * ih[k];
  double out = 0.0;
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    // flux_j at the voxel and at its lower neighbour x - e_j
    const double* vm = vc + n.m[j];
    double fx = 0.0, fm = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      fx += ac[aidx[3 * j + k] * N] * gr[k];
      const double gm = ((k == j ? vc[0] : vm[n.p[k]]) - vm[0]) * ih[k];
      fm += ac[aidx[3 * j + k] * N + n.m[j]] * gm;
    }
    // grad+^T w = sum_j (w_j(x - e_j) - w_j(x)) / h_j
    out += (fm - fx) * ih[j];
  }
  return out;
}

// Operator of a scalar PCG on p fused with the N2 transform of its result:
//   OP = 0  q = a p - k Lap_h p (phase field, 7-point),
//   OP = 1  q = p / w + dt L(p) (Fick; kdiff = dt),
//   OP = 2  q = p (the right-hand side),
// and the partial sums of p.q (OP 0, 1), into the line layout or (planes) the
// plane layout.  A workgroup owns LPB lines (i0, i1): its
// threads evaluate the stencil voxel by voxel along the lines into LDS, then
// T threads per line transform it there; q itself never goes to memory.
// Bound by HBM: 128^3 Fick 35 us for its 9 words per voxel (4.3 TB/s), phase
// field 17 us for 3.  The Fick PCG iteration went from 153 to 97 us with this
// and the residual kept in the spectrum.
constexpr int kScalarThreads = 256;
template <int M> constexpr int scalar_lines() {
  constexpr int n = kScalarThreads / 2 / Line<M>::T, cap = 4096 / (2 * M);
  return n < cap ? n : (cap > 0 ? cap : 1);
}

template <int M, int OP>
__global__ void __launch_bounds__(kScalarThreads)
k_scalar_op(const double* __restrict__ p, const double* __restrict__ coef, const double* __restrict__ A6, double kdiff,
            Grid3 g, double2* __restrict__ out, double* __restrict__ partials, SpecTables<double> tb, Gate gate, int planes) {
  using C = double2;
  using LS = Line<M>;
  constexpr int LPB = scalar_lines<M>(), N2 = 2 * M;
  constexpr int PAD = (M >= 16) ? 1 : 0;
  __shared__ C lds[LPB * (M + PAD)];
  __shared__ double red[16];
  if (gate(0)) return;
  const long nlines = (long)g.n0 * g.n1, N = nlines * N2;
  const long line0 = (long)blockIdx.x * LPB;
  double acc = 0.0;
  for (int v = threadIdx.x; v < LPB * N2; v += kScalarThreads) {
    const int ll = v / N2, i2 = v - ll * N2;
    const long line = line0 + ll;
    double qv = 0.0;
    if (line < nlines) {
      const int i0 = (int)(line / g.n1), i1 = (int)(line - (long)i0 * g.n1);
      const Nbr n = neighbours(g, i0, i1, i2);
      const double* pc = p + n.c;
      const double p0 = pc[0];
      if constexpr (OP == 0) {
        const double l0 = (2.0 * p0 - pc[n.p[0]] - pc[n.m[0]]) * g.ih0 * g.ih0;
        const double l1 = (2.0 * p0 - pc[n.p[1]] - pc[n.m[1]]) * g.ih1 * g.ih1;
        const double l2 = (2.0 * p0 - pc[n.p[2]] - pc[n.m[2]]) * g.ih2 * g.ih2;
        qv = coef[n.c] * p0 + kdiff * (l0 + l1 + l2);
      } else if constexpr (OP == 2) {
        qv = p0;
      } else {
        qv = p0 / coef[n.c] + kdiff * fick_L(p, A6, g, N, n);
      }
      acc += p0 * qv;
    }
    reinterpret_cast<double*>(lds + ll * (M + PAD))[i2] = qv;
  }
  __syncthreads();
  const int t = threadIdx.x % LS::T;
  const int lt = threadIdx.x / LS::T;
  const int ll = lt < LPB ? lt : LPB - 1;  // idle threads only take part in the barriers
  const bool mine = lt < LPB;
  const bool active = mine && line0 + ll < nlines;
  C* my = lds + ll * (M + PAD);
  C v[LS::E];
  if (mine) {
#pragma unroll
    for (int e = 0; e < LS::E; ++e) v[e] = my[LS::idxA(t, e)];
    // a line's threads sit in one wave (T divides 64)
    static_assert(64 % LS::T == 0, "lines within one wave");
    lds_sync<true>();
    line_fft_AB<M, false, C, true>(v, my, 1, t, tb.twM);
#pragma unroll
    for (int e = 0; e < LS::E; ++e) my[LS::idxB(t, e)] = v[e];
    lds_sync<true>();
    if (active && !planes) {
#pragma unroll
      for (int e = 0; e < LS::E; ++e) {
        const int k = LS::idxB(t, e);
        out[(line0 + ll) * M + k] = r2c_post(my, k, M, tb.post[k]);
      }
    }
  }
  if (planes) {
    __syncthreads();
    for (int i = threadIdx.x; i < LPB * M; i += kScalarThreads) {
      const int k = i / LPB, j = i - k * LPB;
      if (line0 + j < nlines) out[(long)k * nlines + line0 + j] = r2c_post(lds + j * (M + PAD), k, M, tb.post[k]);
    }
  }
  if constexpr (OP == 2) return;
  const double s = block_sum(acc, red);
  if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

}  // namespace fg
