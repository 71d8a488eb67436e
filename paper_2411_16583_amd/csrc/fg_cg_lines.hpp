// One kernel for the real-space half of a CG iteration on small grids: the
// inverse N2 pass with the CG vectors (k_c2r_dir), q = D^T K : (D pi)
// (k_cg_op) and the N2 pass of q (k_r2c_edges).
//
// A workgroup takes L node lines of one node plane, whole along N2: it forms
// pi on the three planes and L + 2 lines that their stencils touch (9 (L + 2)
// short transforms; the lines it owns are stored), the tangent on two voxel
// planes of L + 1 lines, and transforms its 3 L lines of q, with nothing but
// LDS in between.  The neighbours' lines are transformed again by their own
// workgroups, so pi is kept in two buffers (iteration k writes buffer k mod 2).
// Bound by latency, a launch and half a dozen dependent waits: 16^3 FP64 11.6 us
// where the three passes took 8.0 + 5.6 + 6.3 and two more launches.
#pragma once
#include "fg_cg3.hpp"

namespace fg {

template <typename R> struct LinesArgs {
  const cplx<R>* z;  // spectrum of z, plane layout
  cplx<R>* q;        // of q, plane layout (not z)
  R *pi, *xi;        // pi: two buffers pi2 values apart
  long pi2;
  const R* st;
  KrylovScalars* ks;
  const double* prr;  // partial sums of r.r of the iteration before, np per item
  int np;
  double* partials;  // p.Kp per workgroup
  int n0, n1, L, nb, groups;  // nb blocks of lines per plane, groups = n0 nb workgroups per item
  SpecTables<R> tb;
  R q0, q1, q2;
};

constexpr int kLinesThreads = 256;
// LDS of a workgroup: pi, the tangent's Y, the exchange rows of the transforms
// (a spare row for the idle threads) and their tables; real: bytes of a real.
inline size_t lines_lds(size_t real, int M, int L) {
  const size_t reals = (size_t)2 * M * (9 * (L + 2) + 18 * (L + 1));
  return (reals + 2 * ((size_t)(9 * (L + 2) + 1) * (M + 1) + 2 * M)) * real;
}

template <typename R, int M, int LAW>
__global__ void __launch_bounds__(kLinesThreads) k_cg_lines(LinesArgs<R> a) {
  using C = cplx<R>;
  using LS = Line<M>;
  constexpr int N2 = 2 * M, LPB = kLinesThreads / LS::T, ROW = M + 1;
  constexpr int NS = LAW == kLawSVK ? 17 : 12;
  extern __shared__ __align__(16) char smem_raw[];
  __shared__ double red[16];
  const int L = a.L, n0 = a.n0, n1 = a.n1, nl1 = 9 * (L + 2);
  C* stw = reinterpret_cast<C*>(smem_raw);
  C* spost = stw + M;
  C* lds = spost + M;
  R* pib = reinterpret_cast<R*>(lds + (nl1 + 1) * ROW);  // [plane][component][line][N2]
  R* yb = pib + nl1 * N2;                                 // [plane][9][line][N2]
  const int item = (int)(blockIdx.x / (unsigned)a.groups), g = (int)blockIdx.x - item * a.groups;
  const int v = g / a.nb, i1b = (g - v * a.nb) * L;  // node plane and first node line
  const long nlines = (long)n0 * n1, N = nlines * N2;
  KrylovScalars* ks = a.ks + item;
  const C* z = a.z + (long)item * 3 * nlines * M;
  C* q = a.q + (long)item * 3 * nlines * M;
  const R* st = a.st + (long)item * state_words(LAW) * N;
  auto wrap = [](int i, int n) { return i < 0 ? i + n : i % n; };
  // voxel of a task of the tangent
  const int lv = (L + 1) * N2;
  auto voxel = [&](int task, int& pl, int& l, int& x) {
    pl = task >= lv ? 1 : 0;
    const int r = task - pl * lv;
    l = r / N2;
    x = r - l * N2;
  };
  R A[NS];
  auto state = [&](int task) {
    int pl, l, x;
    voxel(task, pl, l, x);
    const R* s = st + ((long)wrap(v + pl, n0) * n1 + wrap(i1b + l, n1)) * N2 + x;
#pragma unroll
    for (int k = 0; k < NS; ++k) A[k] = s[k * N];
  };
  // read ahead of the transforms
  if ((int)threadIdx.x < 2 * lv) state(threadIdx.x);
  double rr = thread_partials(a.prr + (long)item * a.np, a.np);
  for (int k = threadIdx.x; k < M; k += kLinesThreads) {
    stw[k] = a.tb.twM[k];
    spost[k] = a.tb.post[k];
  }
  if (ks->done) return;
  const bool pending = !ks->fresh;
  const int idx = ks->iter + (pending ? 1 : 0);  // this iteration
  const bool first = idx == 0;
  const R alpha = first ? R(0) : (R)ks->alpha;
  R beta = first ? R(0) : (R)ks->beta;
  rr = block_sum_all(rr, red);
  if (pending) {
    const KrylovTest kt = krylov_test(ks, rr, 0.0, 0);
    if (g == 0 && threadIdx.x == 0) {
      ks->run_rr = rr;
      ks->run_iter = kt.iter;
      ks->stop = kt.done;
    }
    if (kt.done) return;
    beta = (R)kt.beta;
  }
  const R* po = a.pi + (first ? 0 : (idx - 1) & 1) * a.pi2 + (long)item * 3 * N;
  R* pn = a.pi + (idx & 1) * a.pi2 + (long)item * 3 * N;
  R* xi = a.xi + (long)item * 3 * N;
  const int t = threadIdx.x % LS::T, ll = threadIdx.x / LS::T;
  C* my = lds + min(ll, nl1) * ROW;
  // pi on the planes v - 1, v, v + 1 and the lines i1b - 1 ... i1b + L
  for (int base = 0; base < nl1; base += LPB) {
    const int line = base + ll;
    const bool act = line < nl1;
    const int lm = act ? line % (L + 2) : 0, r = act ? line / (L + 2) : 0;
    const int c = r % 3, pl = r / 3;
    const long gl = (long)wrap(v - 1 + pl, n0) * n1 + wrap(i1b - 1 + lm, n1);
    const bool own = act && pl == 1 && lm >= 1 && lm <= L && i1b + lm - 1 < n1;
    const long off = c * N / 2 + gl * M;  // in pairs of reals
    C w[LS::E], p[LS::E], x[LS::E];
#pragma unroll
    for (int e = 0; e < LS::E; ++e) {
      w[e] = p[e] = x[e] = mk<C>(R(0), R(0));
      if (act) w[e] = z[((long)c * M + LS::idxA(t, e)) * nlines + gl];
    }
    if (act && !first) {
#pragma unroll
      for (int e = 0; e < LS::E; ++e) {
        p[e] = reinterpret_cast<const C*>(po)[off + LS::idxB(t, e)];
        if (own) x[e] = reinterpret_cast<const C*>(xi)[off + LS::idxB(t, e)];
      }
    }
#pragma unroll
    for (int e = 0; e < LS::E; ++e) my[LS::idxA(t, e)] = w[e];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < LS::E; ++e) {
      const int k = LS::idxA(t, e);
      const C xk = w[e];
      if (k == 0) {
        w[e] = mk<C>(xk.x + xk.y, xk.x - xk.y);
      } else {
        const C xm = my[M - k];
        const C s = cadd(xk, cconj(xm));
        const C d = cmulc(csub(xk, cconj(xm)), spost[k]);
        w[e] = cadd(s, mul_pi(d));
      }
    }
    __syncthreads();
    line_fft_AB<M, true>(w, my, 1, t, stw);
#pragma unroll
    for (int e = 0; e < LS::E; ++e) {
      const int n = LS::idxB(t, e);
      const C o = first ? w[e] : mk<C>(w[e].x + beta * p[e].x, w[e].y + beta * p[e].y);
      if (act) reinterpret_cast<C*>(pib + line * N2)[n] = o;
      if (own) {
        reinterpret_cast<C*>(pn)[off + n] = o;
        reinterpret_cast<C*>(xi)[off + n] =
            first ? mk<C>(R(0), R(0)) : mk<C>(x[e].x + alpha * p[e].x, x[e].y + alpha * p[e].y);
      }
    }
  }
  __syncthreads();
  // Y = K : (D pi) on the voxel planes v, v + 1 and the lines i1b ... i1b + L
  double acc = 0.0;
  for (int task = threadIdx.x; task < 2 * lv;) {
    int pl, l, x;
    voxel(task, pl, l, x);
    const int xm = x == 0 ? N2 - 1 : x - 1;
    R X[9], Y[9];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      R cs[2][3];
#pragma unroll
      for (int s = 0; s < 2; ++s) {  // planes before and behind
        const R* u1 = pib + (((pl + s) * 3 + c) * (L + 2) + l) * N2;  // line i1 - 1
        const R* u0 = u1 + N2;
        const R a0 = u0[x] + u0[xm], a1 = u1[x] + u1[xm];
        cs[s][0] = a0 + a1;
        cs[s][1] = a0 - a1;
        cs[s][2] = (u0[x] + u1[x]) - (u0[xm] + u1[xm]);
      }
      X[3 * c] = a.q0 * (cs[1][0] - cs[0][0]);
      X[3 * c + 1] = a.q1 * (cs[1][1] + cs[0][1]);
      X[3 * c + 2] = a.q2 * (cs[1][2] + cs[0][2]);
    }
    R F[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) F[k] = A[k];
    if constexpr (LAW == kLawSVK) {
      R S[6];
#pragma unroll
      for (int k = 0; k < 6; ++k) S[k] = A[9 + k];
      svk_apply<R>(F, S, A[15], A[16], X, Y);
    } else {
      tangent_apply<R>(F, A[9], A[10], A[11], X, Y);
    }
    double d = 0.0;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      d += (double)X[k] * (double)Y[k];
      yb[((pl * 9 + k) * (L + 1) + l) * N2 + x] = Y[k];
    }
    if (pl == 0 && l < L && i1b + l < n1) acc += d;  // each voxel once
    task += kLinesThreads;
    if (task < 2 * lv) state(task);
  }
  __syncthreads();
  // q on the node lines and its N2 transform
  for (int base = 0; base < 3 * L; base += LPB) {
    const int line = base + ll;
    const bool act = line < 3 * L && i1b + line % L < n1;
    const int c = act ? line / L : 0, l = act ? line % L : 0;
    // what voxel (l, x) gives its two nodes on the line l (s = 0: node x, node
    // x - 1) or on the line before it (s = 1)
    auto give = [&](int l_, int x, int s, R& f, R& b) {
#pragma clang fp contract(off)
      const R* y = yb + (3 * c * (L + 1) + l_) * N2 + x;
      const int comp = (L + 1) * N2, plane = 9 * comp;
      const R d0 = a.q0 * (y[0] - y[plane]);
      const R s1 = a.q1 * (y[comp] + y[plane + comp]);
      const R s2 = a.q2 * (y[2 * comp] + y[plane + 2 * comp]);
      const R u = s == 0 ? d0 + s1 : d0 - s1;
      f = u + s2;
      b = u - s2;
    };
    auto node = [&](int x) {
      const int xp = x + 1 == N2 ? 0 : x + 1;
      R f0, f1, c0, c1, o;
      give(l, x, 0, f0, o);
      give(l, xp, 0, o, c0);
      give(l + 1, x, 1, f1, o);
      give(l + 1, xp, 1, o, c1);
      return (f0 + c0) + (f1 + c1);
    };
    C w[LS::E];
#pragma unroll
    for (int e = 0; e < LS::E; ++e) {
      const int n = LS::idxA(t, e);
      w[e] = act ? mk<C>(node(2 * n), node(2 * n + 1)) : mk<C>(R(0), R(0));
    }
    line_fft_AB<M, false>(w, my, 1, t, stw);
#pragma unroll
    for (int e = 0; e < LS::E; ++e) my[LS::idxB(t, e)] = w[e];
    __syncthreads();
    if (act) {
      const long gl = (long)v * n1 + i1b + l;
#pragma unroll
      for (int e = 0; e < LS::E; ++e) {
        const int k = LS::idxB(t, e);
        q[((long)c * M + k) * nlines + gl] = r2c_post(my, k, M, spost[k]);
      }
    }
    __syncthreads();
  }
  const double s = block_sum(acc, red);
  if (threadIdx.x == 0) a.partials[(long)item * a.groups + g] = s;
}

}  // namespace fg
