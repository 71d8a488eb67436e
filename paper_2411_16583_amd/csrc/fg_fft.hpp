// Batched 1-D FFTs of one line length L inside a workgroup, and the three
// axis passes of the 3-D real transform used by the Fourier-Galerkin
// operator (Sec. 3.2 "FFT resolution algorithms", eq. (30)).
//
// Line algorithm: two-stage Cooley-Tukey with L = R1 * R2.  T threads share a
// line (T = gcd(R1, R2)); each thread keeps E = L / T elements in registers
// and the only exchange between the stages goes through LDS:
//   layout A (natural): thread t holds x[(t + T u) + R2 n1], e = u R1 + n1
//   layout B (spectral): thread t holds X[(t + T v) + R1 k2], e = v R2 + k2
// fwd: A -> B (stage 1 radix R1 over n1, twiddle W_L^{b k1}, stage 2 radix R2)
// inv: B -> A (the mirror image), so a spectrum produced by fwd can be
// multiplied pointwise and transformed back without any reordering.
//
// 3-D real layout: (C, N0, N1, N2) with N2 fastest.  The half spectrum is
// stored "packed" in exactly the same bytes, (C, N0, N1, M) complex with
// M = N2 / 2: along N2 the DC and Nyquist coefficients of a real line are
// both real, and X[0] holds (Re X_0, Re X_M).  After the N1 and N0 passes
// the kx = 0 column therefore carries A + i B, A and B being the 2-D spectra
// of the kx = 0 and kx = M planes; the pointwise operator separates them with
// the partner column at (-kz, -ky) (kernel k_fft_z_dc).
#pragma once
#include "fg_complex.hpp"

namespace fg {

// Device-side scalars of one Krylov solve (FP64, in the workspace).
struct KrylovScalars {
  double rr;     // current r.r
  double rr0;    // b.b
  double rz;     // r.z (preconditioned solves)
  double pAp;
  double alpha;
  double alpha1;  // of the iteration before
  double beta;
  double tol2;   // tol^2 (0: run to maxit)
  int iter;
  int maxit;
  int done;      // 1 when converged, broken down or out of iterations
  int flag;      // 0 running/converged, 1 breakdown, 2 max iterations
  // Where the partial sums of an iteration are few, its direction pass
  // (k_c2r_dir) adds them up in every workgroup instead of waiting for a
  // kernel of its own.  What it finds is kept apart from what its other
  // workgroups still read, and taken over by the pass that forms alpha.
  double run_rr, run_rz;
  int run_iter;
  int stop;    // the passes of the running iteration skip the item (set with done, or by the direction pass)
  int fresh;   // rr ... flag above are those of the last iteration; 0: its partial sums are still to be added up
  int pad_;

  // rr ... flag are what the next iteration starts from
  __host__ __device__ __forceinline__ void publish() {
    run_rr = rr;
    run_rz = rz;
    run_iter = iter;
    stop = done;
    fresh = 1;
  }
};

// Which batch item a workgroup belongs to and whether that item is masked
// off; workgroups of masked items return at once.  The mask is one int word
// per item (nonzero: skip), either the done flag of the item's Krylov
// scalars or a separate per-item flag array.  A plan is a batch of one item.
struct Skip {
  const int* gate = nullptr;  // nullptr: never skip
  int stride = 0;             // ints between the words of consecutive items
  long per_item = 1L << 62;   // grid units (lines, planes or rows) per item
  __host__ __device__ int item(long unit) const { return (int)(unit / per_item); }
  __device__ __forceinline__ bool operator()(long unit) const {
    return gate && gate[(long)item(unit) * stride] != 0;
  }
  Skip unit(long per) const {
    Skip s = *this;
    s.per_item = per;
    return s;
  }
  __device__ __forceinline__ bool masked(int item) const { return gate && gate[(long)item * stride] != 0; }
  // Workgroups of lpb lines over nlines lines (per_item lines per item) that
  // never straddle two items: ceil(lines per item / lpb) workgroups per item.
  __host__ __device__ long item_lines(long nlines) const { return per_item < nlines ? per_item : nlines; }
  __host__ __device__ long line_blocks(long nlines, int lpb) const {
    const long lpi = item_lines(nlines);
    return (nlines / lpi) * ((lpi + lpb - 1) / lpb);
  }
};

// Line of thread row ll of this workgroup under the item-aligned split.
struct LineMap {
  long line;    // global line index
  bool active;  // inside its item
  int item;
};
__device__ __forceinline__ LineMap map_line(const Skip& sk, long nlines, int lpb, int ll) {
  const long lpi = sk.item_lines(nlines);
  const long bpi = (lpi + lpb - 1) / lpb;
  const long it = (long)blockIdx.x / bpi;
  const long lin = ((long)blockIdx.x - it * bpi) * lpb + ll;
  return LineMap{it * lpi + lin, lin < lpi, (int)it};
}
static_assert(sizeof(KrylovScalars) % sizeof(int) == 0, "gate stride");

template <int L> struct LineShape;
#define FG_LINE_SHAPE(L_, R1_, R2_) \
  template <> struct LineShape<L_> { static constexpr int R1 = R1_, R2 = R2_; };
FG_LINE_SHAPE(1, 1, 1)
FG_LINE_SHAPE(2, 2, 1)
FG_LINE_SHAPE(3, 3, 1)
FG_LINE_SHAPE(4, 4, 1)
FG_LINE_SHAPE(6, 6, 1)
FG_LINE_SHAPE(8, 8, 1)
FG_LINE_SHAPE(12, 12, 1)
FG_LINE_SHAPE(16, 4, 4)
FG_LINE_SHAPE(24, 6, 4)
FG_LINE_SHAPE(32, 8, 4)
FG_LINE_SHAPE(48, 12, 4)
FG_LINE_SHAPE(64, 8, 8)
FG_LINE_SHAPE(96, 12, 8)
FG_LINE_SHAPE(128, 16, 8)
FG_LINE_SHAPE(256, 16, 16)
FG_LINE_SHAPE(512, 32, 16)
#undef FG_LINE_SHAPE

constexpr int cgcd(int a, int b) { return b == 0 ? a : cgcd(b, a % b); }

template <int L> struct Line {
  static constexpr int R1 = LineShape<L>::R1;
  static constexpr int R2 = LineShape<L>::R2;
  static constexpr int T = (R2 == 1) ? 1 : cgcd(R1, R2);
  static constexpr int U = R2 / T;
  static constexpr int V = R1 / T;
  static constexpr int E = L / T;
  __device__ __forceinline__ static int idxA(int t, int e) {
    return t + T * (e / R1) + R2 * (e % R1);
  }
  __device__ __forceinline__ static int idxB(int t, int e) {
    return t + T * (e / R2) + R1 * (e % R2);
  }
};

// Multiply by the stage twiddle W_L^{j} (table tw[j] = e^{-2 pi i j / L}).
template <bool INV, typename C>
__device__ __forceinline__ C twiddle_tab(C a, const C* __restrict__ tw, int j) {
  C w = tw[j];
  return INV ? cmulc(a, w) : cmul(a, w);
}

// Forward (or, with INV, inverse) DFT of a line, layout A -> layout B.
// lds: the line's exchange buffer, element i at lds[i * ls].  Ends with a
// barrier so that the caller may reuse the buffer immediately.
// Order LDS accesses: across the workgroup, or (WAVE) within the wave only,
// for lines that no other wave touches.
template <bool WAVE> __device__ __forceinline__ void lds_sync() {
  if constexpr (WAVE) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

template <int L, bool INV, typename C, bool WAVE = false>
__device__ __forceinline__ void line_fft_AB(C (&v)[Line<L>::E], C* lds, int ls, int t,
                                            const C* __restrict__ tw) {
  using LS = Line<L>;
  if constexpr (LS::R2 == 1) {
    Dft<LS::R1, 1, INV, C>::run(v);
  } else {
#pragma unroll
    for (int u = 0; u < LS::U; ++u) {
      const int b = t + LS::T * u;
      Dft<LS::R1, 1, INV, C>::run(v + u * LS::R1);
#pragma unroll
      for (int k1 = 1; k1 < LS::R1; ++k1)
        v[u * LS::R1 + k1] = twiddle_tab<INV>(v[u * LS::R1 + k1], tw, (b * k1) % L);
#pragma unroll
      for (int k1 = 0; k1 < LS::R1; ++k1) lds[(k1 * LS::R2 + b) * ls] = v[u * LS::R1 + k1];
    }
    lds_sync<WAVE>();
#pragma unroll
    for (int w = 0; w < LS::V; ++w) {
      const int k1 = t + LS::T * w;
#pragma unroll
      for (int n2 = 0; n2 < LS::R2; ++n2) v[w * LS::R2 + n2] = lds[(k1 * LS::R2 + n2) * ls];
      Dft<LS::R2, 1, INV, C>::run(v + w * LS::R2);
    }
    lds_sync<WAVE>();
  }
}

// Inverse DFT of a line, layout B -> layout A (mirror of line_fft_AB).
template <int L, typename C, bool WAVE = false>
__device__ __forceinline__ void line_ifft_BA(C (&v)[Line<L>::E], C* lds, int ls, int t,
                                             const C* __restrict__ tw) {
  using LS = Line<L>;
  if constexpr (LS::R2 == 1) {
    Dft<LS::R1, 1, true, C>::run(v);
  } else {
#pragma unroll
    for (int w = 0; w < LS::V; ++w) {
      const int k1 = t + LS::T * w;
      Dft<LS::R2, 1, true, C>::run(v + w * LS::R2);
#pragma unroll
      for (int n2 = 1; n2 < LS::R2; ++n2)
        v[w * LS::R2 + n2] = twiddle_tab<true>(v[w * LS::R2 + n2], tw, (n2 * k1) % L);
#pragma unroll
      for (int n2 = 0; n2 < LS::R2; ++n2) lds[(n2 * LS::R1 + k1) * ls] = v[w * LS::R2 + n2];
    }
    lds_sync<WAVE>();
#pragma unroll
    for (int u = 0; u < LS::U; ++u) {
      const int n2 = t + LS::T * u;
#pragma unroll
      for (int k1 = 0; k1 < LS::R1; ++k1) v[u * LS::R1 + k1] = lds[(n2 * LS::R1 + k1) * ls];
      Dft<LS::R1, 1, true, C>::run(v + u * LS::R1);
    }
    lds_sync<WAVE>();
  }
}

// ----------------------------------------------------------------------------
// Deterministic block reduction of one double per thread.  Fixed shuffle tree
// within a wave, then wave partials summed in order by thread 0.
__device__ __forceinline__ double block_sum(double v, double* red /*>= 16 doubles in LDS*/) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int nw = (blockDim.x + 63) >> 6;
  __syncthreads();
  if (lane == 0) red[wid] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int k = 0; k < nw; ++k) s += red[k];
  return s;  // valid in thread 0 only
}
// The same, for every thread.
__device__ __forceinline__ double block_sum_all(double v, double* red) {
  block_sum(v, red);
  double s = 0.0;
  for (int k = 0; k < (int)((blockDim.x + 63) >> 6); ++k) s += red[k];
  return s;
}

// Sum of nparts partials in a fixed order by one block (deterministic).
// Each thread keeps eight independent running sums, so that eight loads are
// in flight per thread instead of one (the partials come from other XCDs'
// L2 or from HBM).
__device__ __forceinline__ double thread_partials(const double* __restrict__ partials, int nparts) {
  const int bd = blockDim.x;
  double a[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  int k = threadIdx.x;
  for (; k + 7 * bd < nparts; k += 8 * bd) {
#pragma unroll
    for (int u = 0; u < 8; ++u) a[u] += partials[k + u * bd];
  }
#pragma unroll
  for (int u = 0; u < 8; ++u)
    if (k + u * bd < nparts) a[u] += partials[k + u * bd];
  return ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
}
__device__ __forceinline__ double sum_partials(const double* __restrict__ partials, int nparts, double* red) {
  return block_sum(thread_partials(partials, nparts), red);
}

// Partial sums of one item written by a pass whose tile may vary: `head`
// plain ones, then groups of r consecutive ones each, added as a binary tree
// (the tree continues the one in which the workgroup added its columns, so a
// group's sum does not depend on how many columns a workgroup took).
struct Parts {
  int groups, head, r;  // sums in all (plain ones and groups)
  __host__ __device__ Parts(int n = 0) : groups(n), head(n), r(1) {}
  __host__ __device__ Parts(int g, int h, int r_) : groups(g), head(h), r(r_) {}
  __host__ __device__ __forceinline__ int stride() const { return head + (groups - head) * r; }
};

// Share of thread t of T.
__device__ __forceinline__ double thread_parts(const double* __restrict__ partials, const Parts ps, int t, int T) {
  double acc = 0.0;
  for (int g = t; g < ps.groups; g += T) {
    if (g < ps.head) {
      acc += partials[g];
      continue;
    }
    const double* p = partials + ps.head + (long)(g - ps.head) * ps.r;
    if (ps.r == 1) {
      acc += p[0];
      continue;
    }
    double st[9], v = 0.0;  // binary counter of subtree sums (r <= 256)
    const int b = ps.r % 8 == 0 ? 8 : 1;  // leaves read at once
    for (int i = 0; i < ps.r / b; ++i) {
      if (b == 8) {
        double q[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) q[k] = p[8 * i + k];
        v = ((q[0] + q[1]) + (q[2] + q[3])) + ((q[4] + q[5]) + (q[6] + q[7]));
      } else {
        v = p[i];
      }
      bool go = true;
#pragma unroll
      for (int k = 0; k < 9; ++k)
        if (go) {
          if ((i >> k) & 1) {
            v = st[k] + v;
          } else {
            st[k] = v;
            go = false;
          }
        }
    }
    acc += v;
  }
  return acc;
}
__device__ __forceinline__ double sum_parts(const double* __restrict__ partials, const Parts ps, double* red) {
  // (plain sums with more loads in flight; groups in one order whatever r is)
  if (ps.groups == ps.head) return sum_partials(partials, ps.groups, red);
  return block_sum(thread_parts(partials, ps, threadIdx.x, blockDim.x), red);
}
// The same by a workgroup of any size, the same number for every size; buf:
// 256 doubles of LDS.
__device__ __forceinline__ double sum_parts_any(const double* __restrict__ partials, const Parts ps, double* buf) {
  __syncthreads();
  for (int t = threadIdx.x; t < 256; t += blockDim.x) buf[t] = thread_parts(partials, ps, t, 256);
  __syncthreads();
  for (int n = 128; n >= 1; n >>= 1) {
    for (int t = threadIdx.x; t < n; t += blockDim.x) buf[t] += buf[t + n];
    __syncthreads();
  }
  return buf[0];
}

// CG step length from s = p.Ap (or p.Aq): alpha = r.r / s (r.z / s
// preconditioned), or breakdown when s <= 0.  One thread.
__device__ __forceinline__ void krylov_alpha(KrylovScalars* ks, double s, int pcg) {
  ks->rr = ks->run_rr;
  ks->rz = ks->run_rz;
  ks->iter = ks->run_iter;
  ks->fresh = 0;
  ks->pAp = s;
  if (!(s > 0.0)) {
    ks->done = 1;
    ks->flag = 1;
    ks->publish();
  } else {
    ks->alpha1 = ks->alpha;
    ks->alpha = (pcg ? ks->rz : ks->rr) / s;
  }
}

// An iteration's r.r (and r.z): the direction's beta, and whether the solve
// ends here.
struct KrylovTest {
  double beta;
  int iter, done, flag;
};
__device__ __forceinline__ KrylovTest krylov_test(const KrylovScalars* ks, double rr, double rz, int pcg) {
  KrylovTest k;
  k.beta = pcg ? rz / ks->rz : rr / ks->rr;
  k.iter = ks->iter + 1;
  k.done = k.flag = 0;
  if (ks->tol2 > 0.0 && rr <= ks->tol2 * ks->rr0) {
    k.done = 1;
  } else if (k.iter >= ks->maxit) {
    k.done = 1;
    k.flag = (ks->tol2 > 0.0) ? 2 : 0;
  }
  return k;
}
// The same taken over by one thread.  beta is kept even when the solve stops
// here, so that a solve stopped at a fixed iteration count can be continued.
__device__ __forceinline__ void krylov_take(KrylovScalars* ks, double rr, double rz, int pcg) {
  const KrylovTest k = krylov_test(ks, rr, rz, pcg);
  ks->beta = k.beta;
  ks->iter = k.iter;
  ks->rr = rr;
  if (pcg) ks->rz = rz;
  ks->done = k.done;
  if (k.done) ks->flag = k.flag;
  ks->publish();
}

// End of an iteration from the partial sums of r.r (and r.z) that the N0 pass
// left, by one workgroup of any size, if that is still to be done.  `few`: the
// sums of k_plane, added as its direction pass adds them (XBLOCK threads).
__device__ __forceinline__ void krylov_close(KrylovScalars* ks, const double* __restrict__ prr,
                                             const double* __restrict__ prz, const Parts parts, bool few,
                                             double* buf /*256 doubles in LDS*/) {
  if (ks->done || ks->fresh) return;
  double rr, rz = 0.0;
  if (few) {
    rr = sum_partials(prr, parts.groups, buf);
    if (prz) rz = sum_partials(prz, parts.groups, buf + 16);
  } else {
    rr = sum_parts_any(prr, parts, buf);
    if (prz) rz = sum_parts_any(prz, parts, buf);
  }
  if (threadIdx.x == 0) krylov_take(ks, rr, rz, prz != nullptr);
}

// Tables of one 3-D plan (device pointers), in the working precision R.
template <typename R> struct SpecTables {
  const cplx<R>* tw0;   // W_{N0}^j, j < N0
  const cplx<R>* tw1;   // W_{N1}^j
  const cplx<R>* twM;   // W_M^j, M = N2/2
  const cplx<R>* post;  // W_{N2}^k, k < M (real <-> half-length complex)
  const R* cz;          // cos(pi kz / N0), exact 0 at kz = N0/2
  const R* sz;          // (2/h0) sin(pi kz / N0)
  const R* cy;          // cos(pi ky / N1)
  const R* sy;          // (2/h1) sin(pi ky / N1)
  const R* cx;          // cos(pi kx / N2), kx = 0..M, exact 0 at kx = M
  const R* sx;          // (2/h2) sin(pi kx / N2)
  const R* snz;         // sin(pi kz / N0)  (half-voxel phase factors e^{i q / 2})
  const R* sny;         // sin(pi ky / N1)
  const R* snx;         // sin(pi kx / N2), kx = 0..M
};

// ----------------------------------------------------------------------------
// Pass 1: real-to-complex along N2 for nlines lines (in place allowed).
// Workgroups of the two real passes have XBLOCK threads (LPB lines).
constexpr int XBLOCK = 128;

template <typename R, int M>
__global__ void __launch_bounds__(XBLOCK)
k_fft_x_r2c(const R* in, R* out, long nlines, SpecTables<R> tb, Skip skip) {
  using C = cplx<R>;
  using LS = Line<M>;
  constexpr int LPB = XBLOCK / LS::T;
  constexpr int PAD = (M >= 16) ? 1 : 0;
  __shared__ C lds[LPB * (M + PAD)];
  const int t = threadIdx.x % LS::T;
  const int ll = threadIdx.x / LS::T;
  const LineMap lm = map_line(skip, nlines, LPB, ll);
  if (skip.masked(lm.item)) return;
  const long line = lm.line;
  const bool active = lm.active;
  const C* src = reinterpret_cast<const C*>(in) + line * M;
  C* dst = reinterpret_cast<C*>(out) + line * M;
  C* my = lds + ll * (M + PAD);
  C v[LS::E];
#pragma unroll
  for (int e = 0; e < LS::E; ++e) v[e] = active ? src[LS::idxA(t, e)] : mk<C>(R(0), R(0));
  line_fft_AB<M, false>(v, my, 1, t, tb.twM);
#pragma unroll
  for (int e = 0; e < LS::E; ++e) my[LS::idxB(t, e)] = v[e];
  __syncthreads();
#pragma unroll
  for (int e = 0; e < LS::E; ++e) {
    const int k = LS::idxB(t, e);
    const C zk = my[k];
    C X;
    if (k == 0) {
      X = mk<C>(zk.x + zk.y, zk.x - zk.y);  // (Re X_0, Re X_M)
    } else {
      const C zm = my[M - k];
      const C ev = cscale(cadd(zk, cconj(zm)), R(0.5));
      const C od = cscale(mul_mi(csub(zk, cconj(zm))), R(0.5));
      X = cadd(ev, cmul(od, tb.post[k]));
    }
    if (active) dst[k] = X;
  }
}

// Inverse real pass: y = scale * x_out (type R, into out).
template <typename R, int M>
__global__ void __launch_bounds__(XBLOCK)
k_fft_x_c2r(const R* in, R* out, long nlines, SpecTables<R> tb, double scale, Skip skip) {
  using C = cplx<R>;
  using LS = Line<M>;
  constexpr int LPB = XBLOCK / LS::T;
  constexpr int PAD = (M >= 16) ? 1 : 0;
  __shared__ C lds[LPB * (M + PAD)];
  // the line's stage twiddles and the C2R pre-processing factors, read once
  // per workgroup (the barrier after the line load orders them); from the
  // caches they cost the pass 71 -> 65 us in single precision at 256^3
  __shared__ C stw[M], spost[M];
  for (int k = threadIdx.x; k < M; k += XBLOCK) {
    stw[k] = tb.twM[k];
    spost[k] = tb.post[k];
  }
  const int t = threadIdx.x % LS::T;
  const int ll = threadIdx.x / LS::T;
  const LineMap lm = map_line(skip, nlines, LPB, ll);
  if (skip.masked(lm.item)) return;
  const long line = lm.line;
  const bool active = lm.active;
  const C* src = reinterpret_cast<const C*>(in) + line * M;
  C* my = lds + ll * (M + PAD);
  // one global load per element; the mirror X[M - k] comes from LDS.  Double
  // precision streams both ways (measured at 256^3 on the 3-component
  // potential: 159 -> 143 us; single precision got slower, 71 -> 103 us)
  C v[LS::E];
#pragma unroll
  for (int e = 0; e < LS::E; ++e)
    v[e] = active ? (sizeof(R) == 8 ? ld_stream(src + LS::idxA(t, e)) : src[LS::idxA(t, e)]) : mk<C>(R(0), R(0));
#pragma unroll
  for (int e = 0; e < LS::E; ++e) my[LS::idxA(t, e)] = v[e];
  __syncthreads();
#pragma unroll
  for (int e = 0; e < LS::E; ++e) {
    const int k = LS::idxA(t, e);
    const C xk = v[e];
    if (k == 0) {
      v[e] = mk<C>(xk.x + xk.y, xk.x - xk.y);
    } else {
      const C xm = my[M - k];
      const C s = cadd(xk, cconj(xm));
      const C d = cmulc(csub(xk, cconj(xm)), spost[k]);  // * W^{-k}
      v[e] = cadd(s, mul_pi(d));
    }
  }
  __syncthreads();  // mirrors read before the exchange overwrites the buffer
  line_fft_AB<M, true>(v, my, 1, t, stw);
  // v[e] = N2 * (x[2n] + i x[2n+1]) with n = idxB(t, e)
  C* dst = reinterpret_cast<C*>(out) + line * M;
  const R sg = (R)scale;
#pragma unroll
  for (int e = 0; e < LS::E; ++e) {
    const int n = LS::idxB(t, e);
    const C y = cscale(v[e], sg);
    if (active) {
      if constexpr (sizeof(R) == 8)
        st_stream(dst + n, y);
      else
        dst[n] = y;
    }
  }
}

// ----------------------------------------------------------------------------
// Complex FFT of length L along one axis for tiles of B adjacent kx columns.
// Element e of the line of column col: base + e * estride, with
// base = data + blockIdx.y * ystride + blockIdx.z * zstride + blockIdx.x * B + col
// (complex units).  Used for the N1 pass (estride = M) and, in the diagnostic
// transforms, for the N0 pass (estride = N1 M).  CPT = 2 (single precision):
// each thread owns two adjacent columns, loaded and stored as one 16-byte
// vector, so a tile of B columns takes T B / 2 threads.
// With TWL the stage twiddles are copied into LDS after the exchange buffer
// (L B + L elements of dynamic LDS) and read from there.
template <typename R, int L, bool INV, int CPT, bool TWL = false>
__global__ void __launch_bounds__(256)
k_fft_axis(R* data, long estride, long ystride, long zstride, int B, const cplx<R>* __restrict__ twg,
           Skip skip) {
  using C = cplx<R>;
  using LS = Line<L>;
  extern __shared__ char smem_raw[];
  C* lds = reinterpret_cast<C*>(smem_raw);
  if (skip((long)blockIdx.y + (long)gridDim.y * blockIdx.z)) return;  // unit: plane (y) of line set (z)
  const C* tw = twg;
  if constexpr (TWL) {
    C* stw = lds + L * B;
    for (int k = threadIdx.x; k < L; k += blockDim.x) stw[k] = twg[k];
    __syncthreads();
    tw = stw;
  }
  const int BC = B / CPT;  // column groups per tile
  const int cg = threadIdx.x % BC;
  const int t = threadIdx.x / BC;
  C* base = reinterpret_cast<C*>(data) + (long)blockIdx.y * ystride + (long)blockIdx.z * zstride +
            (long)blockIdx.x * B + CPT * cg;
  if constexpr (CPT == 1) {
    C v[LS::E];
#pragma unroll
    for (int e = 0; e < LS::E; ++e) v[e] = base[(long)LS::idxA(t, e) * estride];
    line_fft_AB<L, INV>(v, lds + cg, B, t, tw);
#pragma unroll
    for (int e = 0; e < LS::E; ++e) base[(long)LS::idxB(t, e) * estride] = v[e];
  } else {
    static_assert(CPT == 2 && sizeof(R) == 4, "column pairs in single precision");
    C v0[LS::E], v1[LS::E];
#pragma unroll
    for (int e = 0; e < LS::E; ++e) {
      const float4 w = *reinterpret_cast<const float4*>(base + (long)LS::idxA(t, e) * estride);
      v0[e] = mk<C>(w.x, w.y);
      v1[e] = mk<C>(w.z, w.w);
    }
    line_fft_AB<L, INV>(v0, lds + 2 * cg, B, t, tw);
    line_fft_AB<L, INV>(v1, lds + 2 * cg + 1, B, t, tw);
#pragma unroll
    for (int e = 0; e < LS::E; ++e)
      *reinterpret_cast<float4*>(base + (long)LS::idxB(t, e) * estride) = make_float4(v0[e].x, v0[e].y, v1[e].x, v1[e].y);
  }
}

// ----------------------------------------------------------------------------
// Pass 3 with the projection (eq. (28), (30)): per row i of the 3x3 field,
// Z_ij = (sum_l A_il r_l) r_j / |r|^2 * scale, r the rotated-scheme vector.
// Grid (M/B, N1, 3 rows).  The kx = 0 column is left to k_fft_z_dc.
template <typename R> struct RVec {
  R x, y, z;
};

template <typename R>
__device__ __forceinline__ RVec<R> rot_vec(const SpecTables<R>& tb, int kz, int ky, int kx) {
  const R cz = tb.cz[kz], sz = tb.sz[kz];
  const R cy = tb.cy[ky], sy = tb.sy[ky];
  const R cx = tb.cx[kx], sx = tb.sx[kx];
  // components along axes 0 (z), 1 (y), 2 (x) of the grid = tensor index j
  RVec<R> r;
  r.x = sz * cy * cx;  // j = 0 (axis 0)
  r.y = cz * sy * cx;  // j = 1 (axis 1)
  r.z = cz * cy * sx;  // j = 2 (axis 2)
  return r;
}

template <typename R>
__device__ __forceinline__ R rget(const RVec<R>& r, int j) {
  return j == 0 ? r.x : (j == 1 ? r.y : r.z);
}

// LDS bytes of k_fft_z_proj beyond the L x B exchange buffer:
// the stage twiddles and the kz tables, staged once per workgroup (reading
// them from LDS inside each transform keeps the compiler from holding them in
// registers across the six transforms of a row).
template <typename R> constexpr size_t zpass_extra_lds(int L) {
  return (size_t)L * sizeof(cplx<R>) + 2 * (size_t)L * sizeof(R);
}

// kx = 0 column: the packed value is A + i B (A: plane kx = 0, B: plane
// kx = N2/2, both spectra of real fields).  A workgroup takes the column pair
// (ky, -ky), transforms along N0, separates
//   A(k) = (P(k) + conj P(-k)) / 2,   B(k) = (P(k) - conj P(-k)) / (2i),
// applies the operator at qx = 0 to A and at qx = pi to B, and recombines.
// One row per workgroup (grid.y = 3 rows per item), one wave per component: the
// components' loads and transforms run side by side, and wave j writes output j.
template <typename R, int L>
__global__ void __launch_bounds__(192)
k_fft_z_dc(R* data, int N1, int M, SpecTables<R> tb, R scale, Skip skip) {
  __shared__ cplx<R> lds[12 * L];  // an exchange buffer of the column pair per wave, and the three spectra
  if (skip(blockIdx.y)) return;
  const int ky0 = (int)blockIdx.x, row = (int)blockIdx.y;
  using C = cplx<R>;
  using LS = Line<L>;
  static_assert(2 * LS::T <= 64, "a column pair of lines per wave");
  const int grp = threadIdx.x / 64;
  const int col = threadIdx.x % 2;
  const int t = (threadIdx.x % 64) / 2;
  const bool lane_ok = t < LS::T;  // the other lanes take part in the barriers only
  C* xbuf = lds + grp * 2 * L;
  C* spec = lds + 6 * L;
  const int ky1 = (N1 - ky0) % N1;
  const int myky = col ? ky1 : ky0;
  const long plane = (long)N1 * M;
  const long comp = (long)L * plane;
  C* base = reinterpret_cast<C*>(data) + (long)myky * M;  // kx = 0
  const bool store = lane_ok && (col == 0 || ky1 != ky0);
  {
    const int c0 = 3 * row;
    {
      const int l = grp;
      C v[LS::E];
#pragma unroll
      for (int e = 0; e < LS::E; ++e) {
        v[e] = lane_ok ? base[(c0 + l) * comp + LS::idxA(t, e) * plane] : mk<C>(R(0), R(0));
      }
      if constexpr (LS::R2 == 1) {
        Dft<LS::R1, 1, false, C>::run(v);
      } else {
        // same two-stage transform, guarded for the idle lanes
#pragma unroll
        for (int u = 0; u < LS::U; ++u) {
          const int b = t + LS::T * u;
          Dft<LS::R1, 1, false, C>::run(v + u * LS::R1);
#pragma unroll
          for (int k1 = 1; k1 < LS::R1; ++k1)
            if (lane_ok) v[u * LS::R1 + k1] = twiddle_tab<false>(v[u * LS::R1 + k1], tb.tw0, (b * k1) % L);
          if (lane_ok)
#pragma unroll
            for (int k1 = 0; k1 < LS::R1; ++k1) xbuf[(k1 * LS::R2 + b) * 2 + col] = v[u * LS::R1 + k1];
        }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < LS::V; ++w) {
          const int k1 = t + LS::T * w;
          if (lane_ok)
#pragma unroll
            for (int n2 = 0; n2 < LS::R2; ++n2) v[w * LS::R2 + n2] = xbuf[(k1 * LS::R2 + n2) * 2 + col];
          Dft<LS::R2, 1, false, C>::run(v + w * LS::R2);
        }
        __syncthreads();
      }
      if (lane_ok)
#pragma unroll
        for (int e = 0; e < LS::E; ++e) spec[(l * 2 + col) * L + LS::idxB(t, e)] = v[e];
    }
    __syncthreads();
    // separate, apply, recombine: thread (t, col) owns kz = idxB(t, e) of its column
    C tA[LS::E], tB[LS::E];
#pragma unroll
    for (int e = 0; e < LS::E; ++e) tA[e] = tB[e] = mk<C>(R(0), R(0));
    if (lane_ok) {
#pragma unroll
      for (int e = 0; e < LS::E; ++e) {
        const int kz = LS::idxB(t, e);
        const int kzm = (L - kz) % L;
        C ta = mk<C>(R(0), R(0)), tbv = mk<C>(R(0), R(0));
        const RVec<R> rA = rot_vec(tb, kz, myky, 0);
        const RVec<R> rB = rot_vec(tb, kz, myky, M);
        for (int l = 0; l < 3; ++l) {
          const C P = spec[(l * 2 + col) * L + kz];
          const C Pm = spec[(l * 2 + (1 - col)) * L + kzm];
          const C A = cscale(cadd(P, cconj(Pm)), R(0.5));
          const C Bv = cscale(mul_mi(csub(P, cconj(Pm))), R(0.5));
          const R ra = rget(rA, l), rb = rget(rB, l);
          ta = mk<C>(ta.x + A.x * ra, ta.y + A.y * ra);
          tbv = mk<C>(tbv.x + Bv.x * rb, tbv.y + Bv.y * rb);
        }
        const R a2 = rA.x * rA.x + rA.y * rA.y + rA.z * rA.z;
        const R b2 = rB.x * rB.x + rB.y * rB.y + rB.z * rB.z;
        ta = cscale(ta, a2 > R(0) ? scale / a2 : R(0));
        tbv = cscale(tbv, b2 > R(0) ? scale / b2 : R(0));
        tA[e] = ta;
        tB[e] = tbv;
      }
    }
    {
      const int j = grp;
      C v[LS::E];
#pragma unroll
      for (int e = 0; e < LS::E; ++e) {
        const int kz = LS::idxB(t, e);
        const C a = cscale(tA[e], rget(rot_vec(tb, kz, myky, 0), j));
        const C b = cscale(tB[e], rget(rot_vec(tb, kz, myky, M), j));
        v[e] = cadd(a, mul_pi(b));  // A' + i B'
      }
      if constexpr (LS::R2 == 1) {
        Dft<LS::R1, 1, true, C>::run(v);
      } else {
#pragma unroll
        for (int w = 0; w < LS::V; ++w) {
          const int k1 = t + LS::T * w;
          Dft<LS::R2, 1, true, C>::run(v + w * LS::R2);
#pragma unroll
          for (int n2 = 1; n2 < LS::R2; ++n2)
            if (lane_ok) v[w * LS::R2 + n2] = twiddle_tab<true>(v[w * LS::R2 + n2], tb.tw0, (n2 * k1) % L);
          if (lane_ok)
#pragma unroll
            for (int n2 = 0; n2 < LS::R2; ++n2) xbuf[(n2 * LS::R1 + k1) * 2 + col] = v[w * LS::R2 + n2];
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < LS::U; ++u) {
          const int n2 = t + LS::T * u;
          if (lane_ok)
#pragma unroll
            for (int k1 = 0; k1 < LS::R1; ++k1) v[u * LS::R1 + k1] = xbuf[(n2 * LS::R1 + k1) * 2 + col];
          Dft<LS::R1, 1, true, C>::run(v + u * LS::R1);
        }
        __syncthreads();
      }
      if (store)
#pragma unroll
        for (int e = 0; e < LS::E; ++e) base[(c0 + j) * comp + LS::idxA(t, e) * plane] = v[e];
    }
  }
}

}  // namespace fg
