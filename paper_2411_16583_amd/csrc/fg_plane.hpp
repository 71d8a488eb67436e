// The N1 and N0 passes of a component's spectrum in one kernel, for grids whose
// (N0, N1) plane of one kx fits in LDS: forward N1 and N0 transforms, the CG
// update of the spectral residual, the norm and the symbol of k_n0, and the
// inverse transforms, one plane per kx: 12 words per voxel and one launch
// instead of 24 and three.
//
// Plane layout: component, kx, then the plane contiguous, (i0, i1); the N2
// passes write and read it through LDS, whole runs of lines per kx.  A line
// (N1 or N0) is transformed by the T threads of its line shape, all in one
// wave, from registers with its exchange in its own row or column of the LDS
// plane; the plane passes through LDS only between the N1 and N0 lines, with
// one workgroup barrier there and one on the way back.  The residual is kept
// in the order (kz, ky), read ahead of the N0 transform.
//
// Bound by its chain of LDS passes and barriers, with one plane per workgroup
// on 96 (64^3) to 144 (96^3) of 256 CUs: 16.3 and 39 us in double precision.
// The iteration with the three passes instead takes 54 / 112 us, with this
// 50 / 110 (other grids: plane_fits).
#pragma once
#include "fg_cg3.hpp"

namespace fg {

// Division of a small non-negative integer by a constant (n d < 2^32).
struct FastDiv {
  unsigned d, m;
  __host__ __device__ FastDiv(unsigned d_ = 1) : d(d_), m(d_ > 1 ? (unsigned)((0x100000000ull + d_ - 1) / d_) : 0u) {}
  __device__ __forceinline__ unsigned div(unsigned n) const { return d == 1 ? n : __umulhi(n, m); }
  __device__ __forceinline__ void divmod(unsigned n, unsigned& q, unsigned& r) const {
    q = div(n);
    r = n - q * d;
  }
};

template <typename R, typename RO> struct PlaneArgs {
  const cplx<R>* q;  // planes
  cplx<RO>* z;       // planes (may be q)
  cplx<RO>* s;       // spectral residual, planes (kz, ky)
  int n0, n1, M, P;  // P planes per workgroup (a power of two dividing M)
  int groups;        // workgroups per item
  FastDiv dn1;
  SpecTables<R> tb;
  R scale;
  double sa0, sa1;  // kSymLap
  Gate gate;
  KrylovScalars* ks;
  const double* pap;  // partial sums of p.Kp of an item (kN0Cg)
  int npap, pcg;
  double *partials, *partials2;  // one per workgroup, items consecutive
};

// Most dynamic LDS that a workgroup takes: 160 KiB, with a margin for the
// kernel's static LDS.
constexpr size_t kPlaneLds = 160 * 1024 - 1024;
// LDS: the planes (odd line stride), the stage twiddles and the symbol tables.
template <typename R> inline size_t plane_lds(int n0, int n1, int P) {
  return ((size_t)P * n0 * (n1 | 1) + n0 + n1) * sizeof(cplx<R>) + 2 * (size_t)(n0 + n1) * sizeof(R);
}

#define FG_PLANE_LINES(X) X(1) X(4) X(6) X(8) X(12) X(16) X(24) X(32) X(48) X(64) X(96) X(128) X(256) X(512)

// Forward N1 lines: global rows -> LDS rows (natural ky).
template <int L, typename C>
__device__ __forceinline__ void plane_rows_fwd(const C* __restrict__ src, C* x, int nl, const C* tw) {
  using LS = ZLine<L>;
  static_assert(64 % LS::T == 0, "lines within one wave");
  constexpr int LD = L | 1;
  for (int task = threadIdx.x; task < nl * LS::T; task += blockDim.x) {
    const int line = task / LS::T, t = task % LS::T;
    C v[LS::E];
#pragma unroll
    for (int e = 0; e < LS::E; ++e) v[e] = src[line * L + LS::idxA(t, e)];
    LS::template fwd<false, C, true>(v, x + line * LD, 1, t, tw);
#pragma unroll
    for (int e = 0; e < LS::E; ++e) x[line * LD + LS::idxB(t, e)] = v[e];
  }
}

// Inverse N1 lines: LDS rows -> global rows.
template <int L, typename C, typename CO>
__device__ __forceinline__ void plane_rows_inv(C* x, CO* __restrict__ dst, int nl, const C* tw) {
  using LS = ZLine<L>;
  using RO = decltype(CO::x);
  constexpr int LD = L | 1;
  for (int task = threadIdx.x; task < nl * LS::T; task += blockDim.x) {
    const int line = task / LS::T, t = task % LS::T;
    C v[LS::E];
#pragma unroll
    for (int e = 0; e < LS::E; ++e) v[e] = x[line * LD + LS::idxB(t, e)];
    lds_sync<true>();
    LS::template inv<C, true>(v, x + line * LD, 1, t, tw);
#pragma unroll
    for (int e = 0; e < LS::E; ++e) dst[line * L + LS::idxA(t, e)] = mk<CO>((RO)v[e].x, (RO)v[e].y);
  }
}

// Column and thread of a task of the N0 lines: 64 / T columns of a wave side
// by side.
template <int T> __device__ __forceinline__ void plane_col(int task, int& col, int& t) {
  constexpr int CW = 64 / T;
  const int w = task >> 6, lane = task & 63;
  col = w * CW + lane % CW;
  t = lane / CW;
}

// N0 lines of all columns: forward, op(v, e-th element's kz, column, s) on the
// spectrum (s: the residual there), and (INV) inverse; without INV the
// spectrum is left in LDS, natural kz.
template <int L, bool LOADS, bool INV, typename C, typename CO, typename F>
__device__ __forceinline__ void plane_cols(C* x, int LD, int n1, FastDiv dn1, int P, const CO* __restrict__ s,
                                           const C* tw, F op) {
  using LS = ZLine<L>;
  const int ncol = P * n1, tasks = (ncol * LS::T + 63) / 64 * 64;
  for (int task = threadIdx.x; task < tasks; task += blockDim.x) {
    int col, t;
    plane_col<LS::T>(task, col, t);
    const bool on = col < ncol;
    unsigned pl, ky;
    dn1.divmod(on ? col : 0, pl, ky);
    C* c = x + pl * L * LD + ky;
    const CO* sp = s + pl * L * n1 + ky;
    C v[LS::E];
    CO r[LOADS ? LS::E : 1];
    if constexpr (LOADS) {
#pragma unroll
      for (int e = 0; e < LS::E; ++e) r[e] = sp[LS::idxB(t, e) * n1];
    }
#pragma unroll
    for (int e = 0; e < LS::E; ++e) v[e] = c[LS::idxA(t, e) * LD];
    if (!on) continue;  // (whole tail lanes of the last wave; their line is not theirs)
    lds_sync<true>();
    LS::template fwd<false, C, true>(v, c, LD, t, tw);
#pragma unroll
    for (int e = 0; e < LS::E; ++e) op(v[e], LS::idxB(t, e), (int)pl, (int)ky, LOADS ? r[LOADS ? e : 0] : CO{});
    if constexpr (INV) {
      LS::template inv<C, true>(v, c, LD, t, tw);
#pragma unroll
      for (int e = 0; e < LS::E; ++e) c[LS::idxA(t, e) * LD] = v[e];
    } else {
#pragma unroll
      for (int e = 0; e < LS::E; ++e) c[LS::idxB(t, e) * LD] = v[e];
    }
  }
}

// Inverse N0 lines alone (natural kz in LDS).
template <int L, typename C>
__device__ __forceinline__ void plane_cols_inv(C* x, int LD, int n1, FastDiv dn1, int P, const C* tw) {
  using LS = ZLine<L>;
  const int ncol = P * n1, tasks = (ncol * LS::T + 63) / 64 * 64;
  for (int task = threadIdx.x; task < tasks; task += blockDim.x) {
    int col, t;
    plane_col<LS::T>(task, col, t);
    if (col >= ncol) continue;
    unsigned pl, ky;
    dn1.divmod(col, pl, ky);
    C* c = x + pl * L * LD + ky;
    C v[LS::E];
#pragma unroll
    for (int e = 0; e < LS::E; ++e) v[e] = c[LS::idxB(t, e) * LD];
    lds_sync<true>();
    LS::template inv<C, true>(v, c, LD, t, tw);
#pragma unroll
    for (int e = 0; e < LS::E; ++e) c[LS::idxA(t, e) * LD] = v[e];
  }
}

// TH bounds the registers: 512 threads (256 registers) in double precision;
// single precision takes a thread per line task up to 768, or, where there are
// more workgroups than CUs, at most 512 of a build with 128 registers, so that
// two workgroups share a CU instead of a second round with few of them.
// (FP32, 512-thread build / chosen, us: 96^3 30.3 / 27.5, 24 x 256 x 64 20.6 /
// 19.5, 48 x 96 x 192 29.0 / 24.1.)
template <typename R, typename RO, int MODE, int SYM, int TH>
__global__ void __launch_bounds__(TH) k_plane(PlaneArgs<R, RO> a) {
  using C = cplx<R>;
  using CO = cplx<RO>;
  extern __shared__ __align__(16) char smem_raw[];
  __shared__ double red[16];
  const int item = (int)(blockIdx.x / (unsigned)a.groups);
  const int g = (int)blockIdx.x - item * a.groups;
  if (a.gate(item)) return;
  const int n0 = a.n0, n1 = a.n1, LD = n1 | 1, nl = a.P * n0;
  C* x = reinterpret_cast<C*>(smem_raw);
  C* tw0 = x + nl * LD;
  C* tw1 = tw0 + n0;
  R* fz = reinterpret_cast<R*>(tw1 + n1);  // scaled sin and cos of the half frequencies
  R* cz = fz + n0;
  R* fy = cz + n0;
  R* cy = fy + n1;
  const long base = ((long)item * a.groups + g) * (long)nl * n1;
  const C* src = a.q + base;
  CO* dst = a.z + base;
  CO* res = a.s + base;
  for (int i = threadIdx.x; i < n0; i += blockDim.x) {
    tw0[i] = a.tb.tw0[i];
    fz[i] = a.tb.sz[i];
    cz[i] = a.tb.cz[i];
  }
  for (int i = threadIdx.x; i < n1; i += blockDim.x) {
    tw1[i] = a.tb.tw1[i];
    fy[i] = a.tb.sy[i];
    cy[i] = a.tb.cy[i];
  }
  // every workgroup adds the partial sums of p.Kp itself (in the same order),
  // its share read ahead of the transforms; one of them records the step length
  double pap = 0.0;
  if constexpr (MODE == kN0Cg) pap = thread_partials(a.pap + (long)item * a.npap, a.npap);
  __syncthreads();
  switch (n1) {
#define FG_CASE(L_) \
  case L_: plane_rows_fwd<L_>(src, x, nl, tw1); break;
    FG_PLANE_LINES(FG_CASE)
#undef FG_CASE
  }
  R alpha = R(0);
  if constexpr (MODE == kN0Cg) {
    const double s = block_sum_all(pap, red);
    KrylovScalars* ks = a.ks + item;
    const double rn = a.pcg ? ks->run_rz : ks->run_rr;
    if (g == 0 && threadIdx.x == 0) krylov_alpha(ks, s, a.pcg);
    if (!(s > 0.0)) return;  // p.Kp <= 0: breakdown
    alpha = (R)(rn / s);
  } else {
    __syncthreads();
  }
  double acc = 0.0, acc2 = 0.0;
  auto symbol = [&](int kz, int ky, R cx, R sx) {
    if constexpr (SYM == kSymProj) {
      const R ra = fz[kz] * cy[ky] * cx, rb = cz[kz] * fy[ky] * cx, rc = cz[kz] * cy[ky] * sx;
      const R r2 = ra * ra + rb * rb + rc * rc;
      return r2 > R(0) ? a.scale / r2 : R(0);
    } else {
      const double la = (double)(fz[kz] * fz[kz] + fy[ky] * fy[ky] + sx * sx);
      return (R)((double)a.scale / (a.sa0 + a.sa1 * la));
    }
  };
  auto norm = [&](C v, R f, double w) {
    const double d = (double)v.x * (double)v.x + (double)v.y * (double)v.y;
    if constexpr (SYM == kSymProj) {
      acc += w * (double)f * d;
    } else {
      acc += w * (double)a.scale * d;
      acc2 += w * (double)f * d;
    }
  };
  // CG update of the residual at one position
  auto update = [&](C& v, int kz, int pl, int ky, CO r) {
    if constexpr (MODE == kN0Cg)
      v = mk<C>((R)r.x - alpha * v.x, (R)r.y - alpha * v.y);
    res[(pl * n0 + kz) * n1 + ky] = mk<CO>((RO)v.x, (RO)v.y);
  };
  const int pid0 = g * a.P;             // first plane (component, kx) of the workgroup
  const bool packed = pid0 % a.M == 0;  // its kx is 0
  constexpr bool kLoads = MODE == kN0Cg;
  if (!packed) {
    auto op = [&](C& v, int kz, int pl, int ky, CO r) {
      update(v, kz, pl, ky, r);
      const int kx = (pid0 + pl) % a.M;
      const R f = symbol(kz, ky, a.tb.cx[kx], a.tb.sx[kx]);
      norm(v, f, 2.0);
      v = cscale(v, f);
    };
    switch (n0) {
#define FG_CASE(L_) \
  case L_: plane_cols<L_, kLoads, true>(x, LD, n1, a.dn1, a.P, (const CO*)res, tw0, op); break;
      FG_PLANE_LINES(FG_CASE)
#undef FG_CASE
    }
  } else {
    // kx = 0 holds A + i B (the real planes kx = 0 and kx = N2/2): each pair
    // of opposite frequencies is separated, scaled and recombined by one thread
    auto op = [&](C& v, int kz, int pl, int ky, CO r) {
      update(v, kz, pl, ky, r);
      if (pl > 0) {
        const int kx = (pid0 + pl) % a.M;
        const R f = symbol(kz, ky, a.tb.cx[kx], a.tb.sx[kx]);
        norm(v, f, 2.0);
        v = cscale(v, f);
      }
    };
    switch (n0) {
#define FG_CASE(L_) \
  case L_: plane_cols<L_, kLoads, false>(x, LD, n1, a.dn1, a.P, (const CO*)res, tw0, op); break;
      FG_PLANE_LINES(FG_CASE)
#undef FG_CASE
    }
    __syncthreads();
    const R cA = a.tb.cx[0], sA = a.tb.sx[0], cB = a.tb.cx[a.M], sB = a.tb.sx[a.M];
    for (int i = threadIdx.x; i < n0 * n1; i += blockDim.x) {
      unsigned kz, ky;
      a.dn1.divmod(i, kz, ky);
      const int q0 = kz == 0 ? 0 : n0 - (int)kz, q1 = ky == 0 ? 0 : n1 - (int)ky;
      const int ip = q0 * n1 + q1;
      if (ip < i) continue;
      const C u = x[kz * LD + ky], um = x[q0 * LD + q1];
      const C A = cscale(cadd(u, cconj(um)), R(0.5));
      const C B = cscale(mul_mi(csub(u, cconj(um))), R(0.5));
      const R fa = symbol((int)kz, (int)ky, cA, sA), fb = symbol((int)kz, (int)ky, cB, sB);
      const double w = ip == i ? 1.0 : 2.0;
      norm(A, fa, w);
      norm(B, fb, w);
      const C ta = cscale(A, fa), tb = cscale(B, fb);
      x[kz * LD + ky] = cadd(ta, mul_pi(tb));
      if (ip != i) x[q0 * LD + q1] = cadd(cconj(ta), mul_pi(cconj(tb)));
    }
    __syncthreads();
    switch (n0) {
#define FG_CASE(L_) \
  case L_: plane_cols_inv<L_>(x, LD, n1, a.dn1, a.P, tw0); break;
      FG_PLANE_LINES(FG_CASE)
#undef FG_CASE
    }
  }
  __syncthreads();
  switch (n1) {
#define FG_CASE(L_) \
  case L_: plane_rows_inv<L_>(x, dst, nl, tw1); break;
    FG_PLANE_LINES(FG_CASE)
#undef FG_CASE
  }
  double s = block_sum(acc, red);
  if (threadIdx.x == 0) a.partials[blockIdx.x] = s;
  if constexpr (SYM == kSymLap) {
    s = block_sum(acc2, red);
    if (threadIdx.x == 0) a.partials2[blockIdx.x] = s;
  }
}

}  // namespace fg
