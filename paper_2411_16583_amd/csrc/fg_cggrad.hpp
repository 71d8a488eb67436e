// Real-space stencil kernels around the CG in divergence form (fg_cg3.hpp):
//   k_grad_store  Z = D U as a 9-component field (the projection itself);
//   k_cg_result   the CG solution x = D (xi + alpha pi) in double precision
//                 (the steps that xi has not taken yet included), stored or added
//                 to a 9-component field.
#pragma once
#include "fg_fft.hpp"
#include "fg_launch.hpp"
#include "fg_potential.hpp"

namespace fg {

// Z = D U: component 3 c + j of Z (N values apart, zis per item) is D_j of
// component c of U (ucs apart, uis per item), evaluated in TO precision.
template <typename TI, typename TO, int W>
__global__ void __launch_bounds__(256)
k_grad_store(const TI* __restrict__ U, long ucs, long uis, TO* __restrict__ Z, long zis, const int* __restrict__ idle,
             int n0, int n1, int n2, TO q0, TO q1, TO q2) {
  using VO = typename VecW<TO, W>::type;
  const int item = blockIdx.y;
  if (idle && idle[item]) return;
  const long N = (long)n0 * n1 * n2;
  U += (long)item * uis;
  Z += (long)item * zis;
  const int G = n2 / W;
  const long g = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= N / W) return;
  const long line = g / G;
  const StencilLines sl = stencil_lines(line, W * (int)(g - line * G), n0, n1, n2);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    TI ui[2][2][W + 1];
    load_corners<TI, W>(U + c * ucs, sl, ui);
    TO u[2][2][W + 1];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int q = 0; q <= W; ++q) u[a][b][q] = (TO)ui[a][b][q];
    TO D[3][W];
    corner_grad<TO, W>(u, q0, q1, q2, D);
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      VO w;
#pragma unroll
      for (int v = 0; v < W; ++v) reinterpret_cast<TO*>(&w)[v] = D[j][v];
      reinterpret_cast<VO*>(Z + (3 * c + j) * N)[g] = w;
    }
  }
}

// Two doubles of a caller's field, which is aligned to 8 bytes and no more.
typedef double Pair8 __attribute__((ext_vector_type(2), aligned(8)));

// x = D (xi + alpha pi) of every item not idle, evaluated in double
// precision (a discrete gradient: compatible to rounding whatever the
// precision of xi), added to Z (ADD) or stored there.  The deferred step
// alpha pi is left out after a breakdown (the direction pass had already
// applied the last valid one); a solve that never iterated has x = 0.
// xi, pi: 3 N values per item (pi2: distance of the buffer that odd iterations
// write); pairs: xi takes its steps two at a time.  Z: 9 N.
template <typename T, bool ADD>
__global__ void __launch_bounds__(256)
k_cg_result(const T* __restrict__ xi, const T* __restrict__ pi, long pi2, int pairs,
            const KrylovScalars* __restrict__ ksb,
            double* __restrict__ Z, const int* __restrict__ idle, int n0, int n1, int n2, double q0, double q1,
            double q2) {
  const int item = blockIdx.y;
  if (idle && idle[item]) return;
  const KrylovScalars* ks = ksb + item;
  // n steps; the direction pass of iteration `run` was the last, and xi has the
  // steps before `have` (every step before its own, or, two at a time, before
  // the last even iteration)
  const int n = ks->iter, run = ks->flag == 1 ? n : n - 1, have = pairs ? run & ~1 : run;
  const bool none = n == 0;
  if (ADD && none) return;
  const int left = n - have;  // steps still to be taken: 0, 1 or (pairs) 2
  const bool empty = pairs && have == 0;
  const T alpha = (T)ks->alpha, alpha1 = (T)ks->alpha1;
  const long N = (long)n0 * n1 * n2;
  xi += (long)item * 3 * N;
  pi += (long)item * 3 * N;
  const T *pl = pi + ((n + 1) & 1) * pi2, *pb = pi + (n & 1) * pi2;  // pi_{n-1}, pi_{n-2}
  Z += (long)item * 9 * N;
  const int G = n2 / 2;
  const long g = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= N / 2) return;
  const long line = g / G;
  const StencilLines sl = stencil_lines(line, 2 * (int)(g - line * G), n0, n1, n2);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    double u[2][2][3] = {};
    if (!none) {
      T x[2][2][3] = {}, p[2][2][3];
      if (!empty) load_corners<T, 2>(xi + c * N, sl, x);
      auto add = [&](const T* f, T al) {
        load_corners<T, 2>(f + c * N, sl, p);
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int q = 0; q < 3; ++q) x[a][b][q] = x[a][b][q] + al * p[a][b][q];
      };
      if (left == 2) add(pb, alpha1);
      if (left >= 1) add(pl, alpha);
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int q = 0; q < 3; ++q) u[a][b][q] = (double)x[a][b][q];
    }
    double D[3][2];
    corner_grad<double, 2>(u, q0, q1, q2, D);
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      Pair8* z = reinterpret_cast<Pair8*>(Z + (3 * c + j) * N) + g;
      const Pair8 d = {D[j][0], D[j][1]};
      if constexpr (ADD)
        *z = *z + d;
      else
        *z = d;
    }
  }
}

// Z = D U over all items (two voxels per thread).
template <typename TI, typename TO>
void launch_grad_store(const TI* U, long ucs, long uis, TO* Z, long zis, const int* idle, int n0, int n1, int n2,
                       int nitems, const double h[3], hipStream_t s) {
  const long N = (long)n0 * n1 * n2;
  const TO q0 = (TO)(0.25 / h[0]), q1 = (TO)(0.25 / h[1]), q2 = (TO)(0.25 / h[2]);
  const dim3 grid((unsigned)((N / 2 + 255) / 256), (unsigned)nitems);
  hipLaunchKernelGGL((k_grad_store<TI, TO, 2>), grid, dim3(256), 0, s, U, ucs, uis, Z, zis, idle, n0, n1, n2, q0, q1,
                     q2);
}

template <typename T, bool ADD>
void launch_cg_result(const T* xi, const T* pi, long pi2, int pairs, const KrylovScalars* ks, double* Z, const int* idle, int n0, int n1,
                      int n2, int nitems, const double h[3], hipStream_t s) {
  const long N = (long)n0 * n1 * n2;
  hipLaunchKernelGGL((k_cg_result<T, ADD>), dim3((unsigned)((N / 2 + 255) / 256), (unsigned)nitems), dim3(256), 0, s, xi,
                     pi, pi2, pairs, ks, Z, idle, n0, n1, n2, 0.25 / h[0], 0.25 / h[1], 0.25 / h[2]);
}

}  // namespace fg
