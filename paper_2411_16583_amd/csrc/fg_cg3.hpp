// Kernels of the CG on the operator of eq. (30) in divergence form.
//
// With D the corner-stencil gradient (fg_potential.hpp) every vector of the
// CG is a discrete gradient (r = D z, p = D pi, x = D xi), and the projection
// of a field Y is G*Y = D (D^T D)^+ D^T Y: its 3-component divergence
// s = D^T Y carries everything the projection needs.  The CG on G K is then
//   z_k = (D^T D)^+ s_k,  pi_k = z_k + beta pi_{k-1},  q = D^T K : (D pi_k),
//   alpha = r.r / p.Kp,   s_{k+1} = s_k - alpha q,     xi += alpha pi_k,
//   r.r = |D z|^2 = sum_q |s^(q)|^2 / (N |r(q)|^2)   (Parseval),
// the same scalars and iterates as the 9-component CG of Alg. 1, with three
// components through the transforms instead of nine, and with the residual
// kept where it is needed, in the spectrum (s^ is read and written by the N0
// pass; no real-space residual update).  Passes of one iteration (words per
// voxel, 62.7 in all; us at 256^3 in double / single precision):
//   k_c2r_dir    inverse N2 pass of z; xi += alpha pi, pi = z + beta pi     13.5  338 / 184
//   k_cg_op      q = D^T K : (D pi) by the stencils, p.Kp                   18.6  535 / 251
//   k_r2c_edges  N2 pass of q                                                6.6  152 /  91
//   k_n1         N1 pass into the block layout (+ alpha)                     6    146 /  76
//   k_n0         N0 pass: s^ -= alpha q^, r.r, z^ = s^ / |r|^2, and back    12    294 / 156
//   k_n1         inverse N1 pass (+ beta, the end of the solve)              6    175 /  79
// Bound by HBM: 5.4-5.8 TB/s in double precision (the operator 4.7, the inverse
// N1 pass 4.6) and 4.9-5.3 in single, where a plain copy reaches 4.4.  The
// iteration that carried nine components through the N2 and N1 passes and the
// residual in real space moved 81 words: 2180 / 1040 us against 1640 / 837 (sums
// of the passes; 1.66 / 0.86 ms an iteration with the gaps between them).
//
// On small grids the passes are bound by launches and memory latency: k_plane
// (fg_plane.hpp) takes the N1 and N0 passes in one, k_cg_lines
// (fg_cg_lines.hpp) the rest.
#pragma once
#include "fg_fft.hpp"
#include "fg_fft3.hpp"
#include "fg_potential.hpp"
#include "fg_tangent.hpp"

namespace fg {

template <typename R, typename PV> __device__ __forceinline__ R pk_get(const PV& v, int w) {
  return reinterpret_cast<const R*>(&v)[w];
}
template <typename R, typename PV> __device__ __forceinline__ void pk_set(PV& v, int w, R a) {
  reinterpret_cast<R*>(&v)[w] = a;
}
// nontemporal load of a W-vector (streams read once: the tangent state and
// the solution potential), so that they do not push the stencil's neighbour
// lines of rho and pi out of the caches
template <typename R, int W, typename PV> __device__ __forceinline__ PV pk_load_nt(const PV* p) {
  typedef R nvw __attribute__((ext_vector_type(W)));
  const nvw a = __builtin_nontemporal_load(reinterpret_cast<const nvw*>(p));
  PV v;
#pragma unroll
  for (int w = 0; w < W; ++w) pk_set<R>(v, w, a[w]);
  return v;
}

// W consecutive values in 16-byte stores (one of 8 where that is all).
template <int W, typename R> __device__ __forceinline__ void store_run(R* p, const R (&v)[W]) {
  constexpr int n = (W * (int)sizeof(R) > 16) ? 16 / (int)sizeof(R) : W;
  using PV = typename VecW<R, n>::type;
#pragma unroll
  for (int w = 0; w < W; w += n) {
    PV o;
#pragma unroll
    for (int k = 0; k < n; ++k) pk_set<R>(o, k, v[w + k]);
    reinterpret_cast<PV*>(p)[w / n] = o;
  }
}

// Per-item mask of a launch: items with a nonzero word are left alone.
struct Gate {
  const int* p = nullptr;
  int stride = 0;
  __device__ __forceinline__ bool operator()(long item) const { return p && p[item * stride] != 0; }
  static Gate done(const KrylovScalars* ks) { return Gate{&ks->stop, (int)(sizeof(KrylovScalars) / sizeof(int))}; }
  static Gate flags(const int* f) { return Gate{f, f ? 1 : 0}; }
};

// Layout of a spectral component after the N1 pass: blocks of B adjacent kx
// columns (128 bytes) of one ky, the N0 lines of a block together: element
// (i0, ky, kx) at ((kx / B) N1 + ky) bstr + i0 B + kx % B.  The N0 pass then
// reads and writes whole contiguous blocks, and the N1 passes still touch
// whole 128-byte lines.  The kx = 0 column (two real columns packed in one,
// see k_n0) lives in a compact array of its own, [component][ky][i0].
struct BlockLayout {
  int B;
  long bstr;  // complex values from one block to the next
  long cstr;  // complex values of a component
  __host__ __device__ __forceinline__ long at(int n1, int ky, int kx) const {
    const int b = kx / B;
    return ((long)b * n1 + ky) * bstr + (kx - b * B);
  }
};
template <typename R> constexpr int block_cols(int M) {
  int b = 1;
  while (M % (2 * b) == 0 && 2 * b * (int)sizeof(cplx<R>) <= 128) b *= 2;
  return b;
}
// Blocks of a power-of-two size are kept one line apart from each other.
template <typename R> inline BlockLayout block_layout(int n0, int n1, int M) {
  BlockLayout l;
  l.B = block_cols<R>(M);
  l.bstr = (long)n0 * l.B + (n0 >= 64 ? l.B : 0);
  l.cstr = (M / l.B) * (long)n1 * l.bstr;
  return l;
}

// ---------------------------------------------------------------------------
// Lines (i1) and lanes along N2 of a wave's patch: 8 x 8 lanes of W voxels,
// one 128-byte line of each plane per patch row.
constexpr int kPatch = 8;

// What the patches of k_cg_op cannot add up themselves, per component of q:
//   col  the step across the upper N2 edge of a patch: [line][patch] holds the
//        contribution of patch `patch` to the last node before it
//   row  the step across the upper line edge of a block of 8 lines:
//        [i0][block][x] holds the contribution of block `block` to the line
//        before it, and [i0][block][patch] in cor that of the corner.
// k_r2c_edges adds them while it loads q.
struct EdgeLayout {
  int W8;         // voxels of a patch along N2
  int np, nb;     // patches per line, blocks per plane
  long col, row, cor, comp;  // offsets of the arrays in a component, values per component
};
template <typename R> inline EdgeLayout edge_layout(int n0, int n1, int n2) {
  EdgeLayout e;
  e.W8 = kPatch * ((sizeof(R) == 4 && n2 % 4 == 0) ? 4 : 2);
  e.np = (n2 + e.W8 - 1) / e.W8;
  e.nb = (n1 + kPatch - 1) / kPatch;
  e.row = 0;
  e.col = (long)n0 * e.nb * n2;
  e.cor = e.col + (long)n0 * n1 * e.np;
  e.comp = (e.cor + (long)n0 * e.nb * e.np + 31) / 32 * 32;
  return e;
}

template <typename R, typename RQ> struct OpArgs {
  RQ* q;               // out: 3 N per item
  RQ* edge;            // out: 3 el.comp per item
  const R* pi;         // direction potential, 3 N per item:
  long pi2;            // the running iteration's of two buffers pi2 values apart
  const KrylovScalars* ks;
  const R* st;         // tangent state
  double* partials;    // p.Kp per workgroup
  Gate gate;
  EdgeLayout el;
  int n0, n1, n2;
  int K;       // node planes per wave
  int nseg;    // plane runs
  int groups;  // workgroups per item
  R q0, q1, q2;
};

constexpr int kOpThreads = 256;

// q = D^T Y with Y = K : (D pi).  A wave owns a patch of
// 8 lines x 8 W voxels of a run of K node planes and marches along i0: node
// plane m takes the voxel planes m and m + 1, so the previous plane's Y stays
// in registers.  Inside the patch a node's contributions come from the lanes
// of the next voxels and of the next line; what crosses the patch's edges is
// stored apart (EdgeLayout), so nothing is computed twice, no workgroup
// barrier is needed and the waves run freely.  RQ: precision of the divergence
// (the sums, q and its edges).
template <typename R, typename RQ, int W, int LAW>
__global__ void __launch_bounds__(kOpThreads) k_cg_op(OpArgs<R, RQ> a) {
  using PV = typename VecW<R, W>::type;
  __shared__ double red[16];
  const unsigned lb = xcd_contiguous(blockIdx.x, gridDim.x);
  const int item = (int)(lb / (unsigned)a.groups);
  if (a.gate(item)) return;
  const int grp = (int)(lb - (unsigned)item * (unsigned)a.groups);
  // patches fastest along N2, then lines, then plane runs
  const long wv = (long)grp * (kOpThreads / 64) + threadIdx.x / 64;
  const int lane = threadIdx.x & 63;
  const int l = lane >> 3, gx = lane & 7;
  const int patch = (int)(wv % a.el.np);
  const long rest = wv / a.el.np;
  const int blk = (int)(rest % a.el.nb);
  const int seg = (int)(rest / a.el.nb);
  const bool live = seg < a.nseg;
  const int i1 = blk * kPatch + l, x = patch * a.el.W8 + gx * W;
  const bool active = live && i1 < a.n1 && x < a.n2;
  const long N = (long)a.n0 * a.n1 * a.n2;
  const R* pi = a.pi + (long)item * 3 * N + (a.ks[item].run_iter & 1) * a.pi2;
  const R* st = a.st + (long)item * state_words(LAW) * N;
  RQ* q = a.q + (long)item * 3 * N;
  RQ* edge = a.edge + (long)item * 3 * a.el.comp;
  const RQ h0 = a.q0, h1 = a.q1, h2 = a.q2;
  // the next voxels (line) of the patch are in the lane one (eight) above
  const bool lastx = gx == kPatch - 1 || x + W >= a.n2;
  const bool lastl = l == kPatch - 1 || i1 + 1 >= a.n1;
  const int ps = seg * a.K, pe = live ? min(a.n0, ps + a.K) : ps - 1;
  double acc = 0.0;
  R Yp[9][W];
#pragma unroll
  for (int k = 0; k < 9; ++k)
#pragma unroll
    for (int w = 0; w < W; ++w) Yp[k][w] = R(0);
  const int xm = (x == 0) ? a.n2 - 1 : x - 1;
  const int i1m = (i1 == 0) ? a.n1 - 1 : i1 - 1;
  auto plane_sums = [&](int i0, R (&cs)[3][3][W]) {
    const R* r0 = pi + ((long)i0 * a.n1 + i1) * a.n2;
    const R* r1 = pi + ((long)i0 * a.n1 + i1m) * a.n2;
    // every load before the first use
    PV w0[3], w1[3];
    R h0[3], h1[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      w0[c] = *reinterpret_cast<const PV*>(r0 + c * N + x);
      w1[c] = *reinterpret_cast<const PV*>(r1 + c * N + x);
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      h0[c] = h1[c] = R(0);
      if (gx == 0) {
        h0[c] = r0[c * N + xm];
        h1[c] = r1[c * N + xm];
      }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      R u[2][W + 1];
      const PV v0 = w0[c], v1 = w1[c];
#pragma unroll
      for (int w = 0; w < W; ++w) {
        u[0][w + 1] = pk_get<R>(v0, w);
        u[1][w + 1] = pk_get<R>(v1, w);
      }
      // the corner x - 1 from the lane below where there is one
      u[0][0] = __shfl_up(u[0][W], 1);
      u[1][0] = __shfl_up(u[1][W], 1);
      if (gx == 0) {
        u[0][0] = h0[c];
        u[1][0] = h1[c];
      }
#pragma unroll
      for (int w = 0; w < W; ++w) {
        const R a0 = u[0][w + 1] + u[0][w], a1 = u[1][w + 1] + u[1][w];
        cs[c][0][w] = a0 + a1;
        cs[c][1][w] = a0 - a1;
        cs[c][2][w] = (u[0][w + 1] + u[1][w + 1]) - (u[0][w] + u[1][w]);
      }
    }
  };
  R pp[3][3][W];
  if (active) plane_sums(ps == 0 ? a.n0 - 1 : ps - 1, pp);
  constexpr int NS = (LAW == kLawSVK) ? 17 : 12;
  for (int v = ps; v <= pe; ++v) {
    const int i0 = (v == a.n0) ? 0 : v;
    const long line = (long)i0 * a.n1 + i1;
    R Yc[9][W];
#pragma unroll
    for (int k = 0; k < 9; ++k)
#pragma unroll
      for (int w = 0; w < W; ++w) Yc[k][w] = R(0);
    if (active) {
      const R* sp = st + line * a.n2 + x;
      PV A[NS];
#pragma unroll
      for (int k = 0; k < NS; ++k) A[k] = pk_load_nt<R, W>(reinterpret_cast<const PV*>(sp + k * N));
      R X[W][9];
      R cs[3][3][W];
      plane_sums(i0, cs);
#pragma unroll
      for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int w = 0; w < W; ++w) {
          X[w][3 * c] = a.q0 * (cs[c][0][w] - pp[c][0][w]);
          X[w][3 * c + 1] = a.q1 * (cs[c][1][w] + pp[c][1][w]);
          X[w][3 * c + 2] = a.q2 * (cs[c][2][w] + pp[c][2][w]);
          pp[c][0][w] = cs[c][0][w];
          pp[c][1][w] = cs[c][1][w];
          pp[c][2][w] = cs[c][2][w];
        }
#pragma unroll
      for (int w = 0; w < W; ++w) {
        R A0[9], Y0[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) A0[k] = pk_get<R>(A[k], w);
        if constexpr (LAW == kLawSVK) {
          R S0[6];
#pragma unroll
          for (int k = 0; k < 6; ++k) S0[k] = pk_get<R>(A[9 + k], w);
          svk_apply<R>(A0, S0, pk_get<R>(A[15], w), pk_get<R>(A[16], w), X[w], Y0);
        } else {
          tangent_apply<R>(A0, pk_get<R>(A[9], w), pk_get<R>(A[10], w), pk_get<R>(A[11], w), X[w], Y0);
        }
        double d = 0.0;
#pragma unroll
        for (int k = 0; k < 9; ++k) {
          d += (double)X[w][k] * (double)Y0[k];
          Yc[k][w] = Y0[k];
        }
        if (v < pe) acc += d;
      }
    }
    if (v > ps) {  // node plane v - 1 is complete
      const long nline = (long)(v - 1) * a.n1 + i1;
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        RQ f0[W], f1[W], c0[W], c1[W];  // to node i2 / node i2 - 1, of node line i1 (0) and i1 - 1 (1)
#pragma unroll
        for (int w = 0; w < W; ++w) {
          // no contraction: the contributions of equal neighbours cancel
          // exactly (a uniform field has zero divergence, not rounding)
#pragma clang fp contract(off)
          const RQ d0 = h0 * ((RQ)Yp[3 * i][w] - (RQ)Yc[3 * i][w]);
          const RQ s1 = h1 * ((RQ)Yp[3 * i + 1][w] + (RQ)Yc[3 * i + 1][w]);
          const RQ s2 = h2 * ((RQ)Yp[3 * i + 2][w] + (RQ)Yc[3 * i + 2][w]);
          const RQ u0 = d0 + s1, u1 = d0 - s1;
          f0[w] = u0 + s2;
          c0[w] = u0 - s2;
          f1[w] = u1 + s2;
          c1[w] = u1 - s2;
        }
        const RQ n0 = __shfl_down(c0[0], 1), n1 = __shfl_down(c1[0], 1);
        const RQ cl = __shfl_down(c1[0], kPatch);
        RQ Tp[W];
#pragma unroll
        for (int w = 0; w < W; ++w) {
          const RQ cp = (w + 1 < W) ? c0[w + 1 < W ? w + 1 : w] : (lastx ? RQ(0) : n0);
          const RQ cm = (w + 1 < W) ? c1[w + 1 < W ? w + 1 : w] : (lastx ? RQ(0) : n1);
          Tp[w] = f0[w] + cp;
          f1[w] += cm;  // the whole contribution to node line i1 - 1
        }
        RQ out[W];
#pragma unroll
        for (int w = 0; w < W; ++w) {
          const RQ t = __shfl_down(f1[w], kPatch);
          out[w] = Tp[w] + (lastl ? RQ(0) : t);
        }
        if (active) {
          store_run<W>(q + i * N + nline * a.n2 + x, out);
          RQ* ec = edge + i * a.el.comp;
          if (l == 0) {
            const long b = (long)(v - 1) * a.el.nb + blk;
            store_run<W>(ec + a.el.row + b * a.n2 + x, f1);
            if (gx == 0) ec[a.el.cor + b * a.el.np + patch] = c1[0];
          }
          if (gx == 0) ec[a.el.col + nline * a.el.np + patch] = c0[0] + (lastl ? RQ(0) : cl);
        }
      }
    }
#pragma unroll
    for (int k = 0; k < 9; ++k)
#pragma unroll
      for (int w = 0; w < W; ++w) Yp[k][w] = Yc[k][w];
  }
  const double s = block_sum(acc, red);
  if (threadIdx.x == 0) a.partials[(long)item * a.groups + grp] = s;
}

// Element k of a real line's half spectrum from its packed transform z (k = 0
// carries both ends); w = W_{N2}^k.
template <typename C> __device__ __forceinline__ C r2c_post(const C* z, int k, int M, C w) {
  using R = decltype(C::x);
  const C zk = z[k];
  if (k == 0) return mk<C>(zk.x + zk.y, zk.x - zk.y);
  const C zm = z[M - k];
  const C ev = cscale(cadd(zk, cconj(zm)), R(0.5));
  const C od = cscale(mul_mi(csub(zk, cconj(zm))), R(0.5));
  return cadd(ev, cmul(od, w));
}

// Tables of the N2 passes, read into registers with the workgroup's data and
// put in LDS behind it: one memory latency at the head of the pass, which is
// most of its time on a small grid.
template <typename C, int M> struct TwiddleRegs {
  static constexpr int n = (M + XBLOCK - 1) / XBLOCK;
  C a[n], b[n];
  template <typename TB> __device__ __forceinline__ explicit TwiddleRegs(const TB& tb) {
#pragma unroll
    for (int u = 0; u < n; ++u) {
      const int k = (int)threadIdx.x + u * XBLOCK;
      const int i = M % XBLOCK == 0 || k < M ? k : 0;
      a[u] = tb.twM[i];
      b[u] = tb.post[i];
    }
  }
  __device__ __forceinline__ void store(C* stw, C* spost) const {
#pragma unroll
    for (int u = 0; u < n; ++u) {
      const int k = (int)threadIdx.x + u * XBLOCK;
      if (M % XBLOCK == 0 || k < M) {
        stw[k] = a[u];
        spost[k] = b[u];
      }
    }
  }
};

// N2 transform of the 3-component fields q of k_cg_op with the patch edges
// added on load, into the line layout or (planes) the plane layout.  grid: line
// blocks of 3 N0 N1 lines per item, blockIdx.y = item.  Every load is issued
// before the first wait (256^3 FP64 167 -> 153 us, 64^3 8.4 -> 7.0).
template <typename R, int M>
__global__ void __launch_bounds__(XBLOCK)
k_r2c_edges(const R* __restrict__ q, const R* __restrict__ edge, EdgeLayout el, cplx<R>* __restrict__ out, int n0,
            int n1, SpecTables<R> tb, Gate gate, int planes) {
  using C = cplx<R>;
  using LS = Line<M>;
  constexpr int LPB = XBLOCK / LS::T, N2 = 2 * M;
  constexpr int PAD = (M >= 16) ? 1 : 0;
  constexpr int NP = (N2 + 15) / 16;  // most patches of a line
  __shared__ C lds[LPB * (M + PAD)];
  __shared__ C stw[M], spost[M];
  __shared__ R ecl[LPB][NP], ecr[LPB][NP];
  const int item = blockIdx.y;
  const int t = threadIdx.x % LS::T;
  const int ll = threadIdx.x / LS::T;
  const int nlines = n0 * n1;
  const int lin = (int)(blockIdx.x * LPB) + ll;
  const bool active = lin < 3 * nlines;
  const int comp = active ? lin / nlines : 0;
  const int line = active ? lin - comp * nlines : 0;
  const int i0 = line / n1, i1 = line - i0 * n1;
  const long base = ((long)item * 3 * nlines + (active ? lin : 0)) * M;
  const C* src = reinterpret_cast<const C*>(q) + base;
  const R* ec = edge + ((long)item * 3 + comp) * el.comp;
  // the last line of its block takes the row stored by the next block
  const bool lastl = i1 % kPatch == kPatch - 1 || i1 == n1 - 1;
  const long nb = (long)i0 * el.nb + ((i1 == n1 - 1) ? 0 : i1 / kPatch + 1);
  C* my = lds + ll * (M + PAD);
  C v[LS::E], r[LS::E];
#pragma unroll
  for (int e = 0; e < LS::E; ++e) v[e] = active ? ld_stream(src + LS::idxA(t, e)) : mk<C>(R(0), R(0));
  if (active && lastl) {
    const C* erow = reinterpret_cast<const C*>(ec + el.row + nb * N2);
#pragma unroll
    for (int e = 0; e < LS::E; ++e) r[e] = erow[LS::idxA(t, e)];
  } else {
#pragma unroll
    for (int e = 0; e < LS::E; ++e) r[e] = mk<C>(R(0), R(0));
  }
  // the line's edge values through LDS (one coalesced read each)
  constexpr int NPT = (NP + LS::T - 1) / LS::T;
  R cl[NPT], cr[NPT];
#pragma unroll
  for (int u = 0; u < NPT; ++u) {
    const int p = t + u * LS::T;
    cl[u] = cr[u] = R(0);
    if (active && p < el.np) {
      cl[u] = ec[el.col + (long)line * el.np + p];
      if (lastl) cr[u] = ec[el.cor + nb * el.np + p];
    }
  }
  TwiddleRegs<C, M> tw(tb);
  tw.store(stw, spost);
#pragma unroll
  for (int u = 0; u < NPT; ++u) {
    const int p = t + u * LS::T;
    if (p < NP) {
      ecl[ll][p] = cl[u];
      ecr[ll][p] = cr[u];
    }
  }
  if (gate(item)) return;  // (the mask is read with the data, not before it)
  __syncthreads();
  const int sh = 31 - __clz(el.W8);  // W8 is a power of two
#pragma unroll
  for (int e = 0; e < LS::E; ++e) {
    const int n = LS::idxA(t, e);
    const int xn = (2 * n + 2 == N2) ? 0 : 2 * n + 2;
    if ((xn & (el.W8 - 1)) == 0) {
      v[e].y += ecl[ll][xn >> sh];
      r[e].y += ecr[ll][xn >> sh];
    }
    v[e] = cadd(v[e], r[e]);
  }
  __syncthreads();
  line_fft_AB<M, false>(v, my, 1, t, stw);
#pragma unroll
  for (int e = 0; e < LS::E; ++e) my[LS::idxB(t, e)] = v[e];
  __syncthreads();
  auto post = [&](int k) { return r2c_post(my, k, M, spost[k]); };
  if (planes) {
    // plane layout: the workgroup's lines of one kx together
    C* o = out + (long)item * 3 * nlines * M;
    const int lin0 = (int)(blockIdx.x * LPB), c0 = lin0 / nlines;
    for (int i = threadIdx.x; i < LPB * M; i += XBLOCK) {
      const int k = i / LPB, j = i - k * LPB;
      if (lin0 + j >= 3 * nlines) continue;
      int c = c0, r = lin0 + j - c0 * nlines;
      while (r >= nlines) {
        r -= nlines;
        ++c;
      }
      o[((long)c * M + k) * nlines + r] = r2c_post(lds + j * (M + PAD), k, M, spost[k]);
    }
  } else if constexpr (sizeof(R) == 4 && M % (2 * LS::T) == 0) {
    // two adjacent elements per thread: whole 128-byte lines per store
#pragma unroll
    for (int j = 0; j < M / (2 * LS::T); ++j) {
      const int k = 2 * (j * LS::T + t);
      const C x0 = post(k), x1 = post(k + 1);
      if (active) st_stream_f4(out + base + k, make_float4(x0.x, x0.y, x1.x, x1.y));
    }
  } else {
#pragma unroll
    for (int e = 0; e < LS::E; ++e) {
      const int k = LS::idxB(t, e);
      const C X = post(k);
      if (active) st_stream(out + base + k, X);
    }
  }
}

// ---------------------------------------------------------------------------
// N1 pass between the line layout (component, i0, i1, kx) and the block
// layout: forward line -> block, inverse block -> line.  Grid (M / tile, N0,
// components).
template <typename R> struct N1Args {
  cplx<R>* lines;
  cplx<R>* blocks;
  cplx<R>* dc;  // kx = 0 column, [component][ky][i0]
  BlockLayout bl;
  int M, tile;
  const cplx<R>* tw;
  Gate gate;
  // forward pass of the CG: a workgroup per item forms alpha from the
  // partial sums of p.Kp (nothing before the N0 pass reads it)
  const double* pap;
  int npap;
  // inverse pass of the CG: a workgroup per item ends the iteration before
  // (krylov_close; nothing before the N2 pass reads it but the mask, and z is
  // not needed once that is set).  As a kernel of its own this took 4-6 us.
  const double *prr, *prz;
  Parts parts;
  KrylovScalars* ks;
  int pcg;  // alpha = r.z / p.Ap (preconditioned CG)
  int nc;   // components per item
};

template <typename R, int L, bool INV, bool TWL>
__global__ void __launch_bounds__(256) k_n1(N1Args<R> a) {
  using C = cplx<R>;
  using LS = Line<L>;
  extern __shared__ __align__(16) char smem_raw[];
  __shared__ double buf[256];
  C* lds = reinterpret_cast<C*>(smem_raw);
  // (with ks, a first row of workgroups for the scalars)
  const int row0 = a.ks ? 1 : 0, z = blockIdx.z, i0 = (int)blockIdx.y - row0, N0 = (int)gridDim.y - row0;
  if (a.gate(z / a.nc)) return;
  if (i0 < 0) {
    if (blockIdx.x != 0 || z % a.nc != 0) return;
    const int item = z / a.nc;
    if constexpr (INV) {
      const long o = (long)item * a.parts.stride();
      krylov_close(a.ks + item, a.prr + o, a.prz ? a.prz + o : nullptr, a.parts, false, buf);
    } else {
      const double s = sum_parts_any(a.pap + (long)item * a.npap, Parts(a.npap), buf);
      if (threadIdx.x == 0) krylov_alpha(a.ks + item, s, a.pcg);
    }
    return;
  }
  const int B = a.tile;
  const C* tw = a.tw;
  if constexpr (TWL) {
    C* stw = lds + L * B;
    for (int k = threadIdx.x; k < L; k += blockDim.x) stw[k] = a.tw[k];
    __syncthreads();
    tw = stw;
  }
  const int col = threadIdx.x % B;
  const int t = threadIdx.x / B;
  const int kx = blockIdx.x * B + col;
  C* ln = a.lines + (((long)z * N0 + i0) * L) * a.M + kx;            // + n M
  C* bk = a.blocks + (long)z * a.bl.cstr + a.bl.at(L, 0, kx) + (long)i0 * a.bl.B;  // + ky bstr
  C* dc = a.dc + (long)z * L * N0 + i0;                              // + ky N0
  const bool col0 = kx == 0;
  C v[LS::E];
#pragma unroll
  for (int e = 0; e < LS::E; ++e) {
    const int n = LS::idxA(t, e);
    if (INV && col0)
      v[e] = dc[(long)n * N0];
    else if constexpr (INV)
      v[e] = bk[n * a.bl.bstr];
    else  // the N2 pass streamed it out; double precision streams it in too (168 -> 147 us at 256^3)
      v[e] = sizeof(R) == 8 ? ld_stream(ln + (long)n * a.M) : ln[(long)n * a.M];
  }
  // a loop of one: inlined that late, the transform leaves every load of the line
  // in flight at once (170 registers; without it 104, and the inverse pass at
  // 256^3 in double precision takes 204 us instead of 173)
#pragma unroll
  for (int once = 0; once < 1; ++once) line_fft_AB<L, INV>(v, lds + col, B, t, tw);
#pragma unroll
  for (int e = 0; e < LS::E; ++e) {
    const int n = LS::idxB(t, e);
    if constexpr (INV)
      ln[(long)n * a.M] = v[e];
    else if (col0)
      dc[(long)n * N0] = v[e];
    else
      bk[n * a.bl.bstr] = v[e];
  }
}

// ---------------------------------------------------------------------------
// N0 pass on the block layout: forward N0 transform of q, the CG update of
// the spectral residual, the norm, the symbol, and the inverse N0 transform.
//   kN0Cg     s -= alpha q (stored), z = f s, partial sums of r.r
//   kN0Start  s = q (stored), z = f s, r.r
// SYM = kSymProj: f = 1 / (N |r|^2) with the rotated vector r of eq. (28) (0
// where r = 0), and r.r = sum over the full spectrum of f |s|^2 (the columns
// kx > 0 of the half spectrum count twice).  SYM = kSymLap (the scalar
// problems' preconditioner): f = 1 / (N (a0 + a1 lambda(q))), r.r = sum of
// |s|^2 / N and r.z = sum of f |s|^2, lambda = sum_j (2/h_j)^2 sin^2(q_j/2).
//
// The kx = 0 column packs the spectra A (kx = 0) and B (kx = N2/2) of real
// planes as A + i B: a leading slice of the launch takes its column pairs
// (ky, -ky), separates A(k) = (P(k) + conj P(-k)) / 2 and
// B(k) = (P(k) - conj P(-k)) / (2 i), scales each with its own symbol and
// recombines; the other workgroups leave that column alone.
constexpr int kSymProj = 0, kSymLap = 1;
constexpr int kN0Cg = 0, kN0Start = 1;

template <typename R, typename RO> struct N0Args {
  const cplx<R>* q;    // blocks
  const cplx<R>* dcq;  // kx = 0 column
  cplx<RO>* z;         // blocks (may be q)
  cplx<RO>* dcz;
  cplx<RO>* s;         // spectral residual, blocks
  cplx<RO>* dcs;
  BlockLayout bl, blo;  // of q, and of z and s
  int N1, M, tile, kymajor;
  SpecTables<R> tb;
  R scale;
  Gate gate;
  const KrylovScalars* ks;
  double* partials;  // per workgroup: column pairs, then [component][ky][tile]; items consecutive (Parts)
  double* partials2;  // the same of r.z (kSymLap)
  double a0, a1;      // kSymLap
  int nc;             // components per item
  int ndc, nmain;    // workgroups per component
};

template <typename R> constexpr size_t n0_extra_lds(int L) {
  return (size_t)L * sizeof(cplx<R>) + 2 * (size_t)L * sizeof(R);
}

// A tile's sum as a binary tree, over the threads of a column first and over
// the columns then: it continues over the tiles of a row in sum_parts, so the
// sum is the same number whatever the tile.  Thread t BC + g (t < T, in the
// first T BC threads) holds the CPT columns CPT g ...; cr: T BC CPT doubles of
// LDS.  Thread 0 has the result.
template <int T, int CPT>
__device__ __forceinline__ double tile_tree(double (&v)[CPT], int BC, double* cr) {
  const int nth = T * BC;
  const int wid = threadIdx.x / 64, lane = threadIdx.x & 63;
  const bool in = (int)threadIdx.x < nth;
#pragma unroll
  for (int c = 0; c < CPT; ++c)
    if (!in) v[c] = 0.0;
  for (int off = BC; off < min(64, nth); off <<= 1) {
#pragma unroll
    for (int c = 0; c < CPT; ++c) v[c] += __shfl_xor(v[c], off, 64);
  }
  __syncthreads();
  if (nth > 64) {
    const int cw = min(BC, 64), cpw = BC > 64 ? BC / 64 : 1, tw = nth / 64 / cpw;  // tw waves of one set of columns
    if (in && lane < cw) {
#pragma unroll
      for (int c = 0; c < CPT; ++c) cr[(wid * cw + lane) * CPT + c] = v[c];
    }
    __syncthreads();
    if ((int)threadIdx.x < BC) {
#pragma unroll
      for (int c = 0; c < CPT; ++c) {
        auto at = [&](int k) { return cr[((wid + k * cpw) * cw + lane) * CPT + c]; };
        if (tw == 1) v[c] = at(0);
        if (tw == 2) v[c] = at(0) + at(1);
        if (tw == 4) v[c] = (at(0) + at(1)) + (at(2) + at(3));
      }
    }
    __syncthreads();
  }
  double w = v[0];
  if constexpr (CPT == 2) w = v[0] + v[CPT - 1];
  for (int off = 1; off < min(BC, 64); off <<= 1) w += __shfl_xor(w, off, 64);
  if (BC > 64) {  // columns over several waves (short lines)
    if ((int)threadIdx.x < BC && lane == 0) cr[wid] = w;
    __syncthreads();
    if (threadIdx.x == 0) w = BC == 128 ? cr[0] + cr[1] : (cr[0] + cr[1]) + (cr[2] + cr[3]);
  }
  return w;
}

template <typename R, typename RO, int L, int CPT, int MODE, int SYM>
__global__ void __launch_bounds__(256) k_n0(N0Args<R, RO> a) {
  using C = cplx<R>;
  using CO = cplx<RO>;
  using LS = typename ZGradSel<R, L>::type;
  extern __shared__ __align__(16) char smem_raw[];
  __shared__ double red[16];
  const unsigned per_comp = (unsigned)(a.ndc + a.nmain), per_item = (unsigned)a.nc * per_comp;
  const int item = (int)(blockIdx.x / per_item);
  if (a.gate(item)) return;
  const unsigned rem = blockIdx.x - (unsigned)item * per_item;
  const bool isdc = rem < (unsigned)(a.nc * a.ndc);
  const int wdc = isdc ? a.ndc : a.nmain;
  const unsigned r2i = isdc ? rem : rem - (unsigned)(a.nc * a.ndc);
  const int comp = (int)(r2i / (unsigned)wdc);
  const int idx = (int)(r2i - (unsigned)comp * wdc);
  const long zc = (long)a.nc * item + comp;
  const int B = a.tile;
  C* stw = reinterpret_cast<C*>(smem_raw);
  R* scz = reinterpret_cast<R*>(stw + L);
  R* ssz = scz + L;
  C* lds = reinterpret_cast<C*>(ssz + L);
  for (int k = threadIdx.x; k < L; k += blockDim.x) {
    stw[k] = a.tb.tw0[k];
    scz[k] = a.tb.cz[k];
    ssz[k] = a.tb.sz[k];
  }
  __syncthreads();
  const R alpha = (MODE == kN0Cg) ? (R)a.ks[item].alpha : R(0);
  double acc[CPT], acc2[CPT];  // acc2: r.z (kSymLap)
#pragma unroll
  for (int c = 0; c < CPT; ++c) acc[c] = acc2[c] = 0.0;
  long part = blockIdx.x;
  if (isdc) {
    // threads beyond the pair's 2 T repeat the work of the first ones (equal
    // values to equal LDS places) and store nothing
    const int td = threadIdx.x % (2 * LS::T);
    const int col = td % 2, t = td / 2;
    const int ky0 = idx, ky1 = (ky0 == 0) ? 0 : a.N1 - ky0;
    const int ky = col ? ky1 : ky0;
    const bool store = (int)threadIdx.x < 2 * LS::T && (col == 0 || ky1 != ky0);
    const long off = (zc * a.N1 + ky) * L;
    C* sp = lds + 2 * L;
    C v[1][LS::E];
#pragma unroll
    for (int e = 0; e < LS::E; ++e) v[0][e] = a.dcq[off + LS::idxA(t, e)];
    LS::template fwd<false>(v[0], lds + col, 2, t, stw);
#pragma unroll
    for (int e = 0; e < LS::E; ++e) {
      const int kz = LS::idxB(t, e);
      if constexpr (MODE == kN0Cg) {
        const CO s = a.dcs[off + kz];
        v[0][e] = mk<C>((R)s.x - alpha * v[0][e].x, (R)s.y - alpha * v[0][e].y);
      }
      sp[col * L + kz] = v[0][e];
    }
    __syncthreads();
    const R cy = a.tb.cy[ky], sy = a.tb.sy[ky], sxM = a.tb.sx[a.M];
#pragma unroll
    for (int e = 0; e < LS::E; ++e) {
      const int kz = LS::idxB(t, e);
      const C P = v[0][e], Pm = sp[(1 - col) * L + (kz == 0 ? 0 : L - kz)];
      if (store) a.dcs[off + kz] = mk<CO>((RO)P.x, (RO)P.y);
      R fa, fb;
      if constexpr (SYM == kSymProj) {
        // rotated vector at qx = 0: (sz cy, cz sy, 0); at qx = pi: (0, 0, cz cy sx)
        const R ra = ssz[kz] * cy, rb = scz[kz] * sy, rc = scz[kz] * cy * sxM;
        const R a2 = ra * ra + rb * rb, b2 = rc * rc;
        fa = a2 > R(0) ? a.scale / a2 : R(0);
        fb = b2 > R(0) ? a.scale / b2 : R(0);
      } else {
        const double la = (double)(ssz[kz] * ssz[kz] + sy * sy);
        fa = (R)((double)a.scale / (a.a0 + a.a1 * la));
        fb = (R)((double)a.scale / (a.a0 + a.a1 * (la + (double)(sxM * sxM))));
      }
      const C A = cscale(cadd(P, cconj(Pm)), R(0.5));
      const C Bv = cscale(mul_mi(csub(P, cconj(Pm))), R(0.5));
      if (store) {
        const double na = (double)A.x * A.x + (double)A.y * A.y, nb = (double)Bv.x * Bv.x + (double)Bv.y * Bv.y;
        const double d = (double)fa * na + (double)fb * nb;
        if constexpr (SYM == kSymProj) {
          acc[0] += d;
        } else {
          acc[0] += (na + nb) * (double)a.scale;
          acc2[0] += d;
        }
      }
      v[0][e] = cadd(cscale(A, fa), mul_pi(cscale(Bv, fb)));
    }
    LS::inv(v[0], lds + col, 2, t, stw);
    if (store) {
#pragma unroll
      for (int e = 0; e < LS::E; ++e) a.dcz[off + LS::idxA(t, e)] = mk<CO>((RO)v[0][e].x, (RO)v[0][e].y);
    }
  } else {
    const int nkx = a.M / B;
    const int ktile = a.kymajor ? idx / a.N1 : idx % nkx;
    const int ky = a.kymajor ? idx - ktile * a.N1 : idx / nkx;
    const int BC = B / CPT;
    // (a workgroup wider than the tile, for the column pairs: repeats as above)
    const int tm = threadIdx.x % (LS::T * BC);
    const bool store = (int)threadIdx.x < LS::T * BC;
    const int col0 = CPT * (tm % BC);
    const int t = tm / BC;
    const int kx0 = ktile * B + col0;
    part = (long)item * per_item + (long)a.nc * a.ndc + ((long)comp * a.N1 + ky) * nkx + ktile;
    const C* src = a.q + zc * a.bl.cstr + a.bl.at(a.N1, ky, kx0);
    const long oo = zc * a.blo.cstr + a.blo.at(a.N1, ky, kx0);
    const int bi = a.bl.B, bo = a.blo.B;
    R f0[CPT], f1[CPT];
    const R cy = a.tb.cy[ky], sy = a.tb.sy[ky];
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      const R cx = a.tb.cx[kx0 + c], sx = a.tb.sx[kx0 + c];
      if constexpr (SYM == kSymProj) {
        const R x0 = cy * cx, x1 = sy * cx, x2 = cy * sx;
        f0[c] = x0 * x0;
        f1[c] = x1 * x1 + x2 * x2;
      } else {
        f0[c] = R(1);
        f1[c] = sy * sy + sx * sx;
      }
    }
    C v[CPT][LS::E];
    CO s[CPT][MODE == kN0Cg ? LS::E : 1];
    if constexpr (CPT == 2) {
      static_assert(sizeof(R) == 4 && sizeof(RO) == 4, "column pairs in single precision");
#pragma unroll
      for (int e = 0; e < LS::E; ++e) {
        const float4 w = ld_stream_f4(src + (long)LS::idxA(t, e) * bi);
        v[0][e] = mk<C>(w.x, w.y);
        v[CPT - 1][e] = mk<C>(w.z, w.w);
      }
      if constexpr (MODE == kN0Cg) {
#pragma unroll
        for (int e = 0; e < LS::E; ++e) {
          const float4 w = ld_stream_f4(a.s + oo + (long)LS::idxB(t, e) * bo);
          s[0][e] = mk<CO>(w.x, w.y);
          s[CPT - 1][e] = mk<CO>(w.z, w.w);
        }
      }
    } else {
#pragma unroll
      for (int e = 0; e < LS::E; ++e) v[0][e] = ld_stream(src + (long)LS::idxA(t, e) * bi);
      if constexpr (MODE == kN0Cg) {
#pragma unroll
        for (int e = 0; e < LS::E; ++e) s[0][e] = ld_stream(a.s + oo + (long)LS::idxB(t, e) * bo);
      }
    }
    LS::template fwd_cols<false, CPT>(v, lds + col0, B, t, stw);
#pragma unroll
    for (int e = 0; e < LS::E; ++e) {
      const int kz = LS::idxB(t, e);
#pragma unroll
      for (int c = 0; c < CPT; ++c) {
        if constexpr (MODE == kN0Cg)
          v[c][e] = mk<C>((R)s[c][e].x - alpha * v[c][e].x, (R)s[c][e].y - alpha * v[c][e].y);
      }
      CO* d = a.s + oo + (long)kz * bo;
      if constexpr (CPT == 2) {
        if (store && kx0 != 0)
          st_stream_f4(d, make_float4(v[0][e].x, v[0][e].y, v[CPT - 1][e].x, v[CPT - 1][e].y));
        else if (store)
          d[1] = v[CPT - 1][e];
      } else {
        if (store && kx0 != 0) st_stream(d, mk<CO>((RO)v[0][e].x, (RO)v[0][e].y));
      }
#pragma unroll
      for (int c = 0; c < CPT; ++c) {
        const R sz = ssz[kz], cz = scz[kz];
        R f;
        if constexpr (SYM == kSymProj) {
          const R r2 = sz * sz * f0[c] + cz * cz * f1[c];
          f = r2 > R(0) ? a.scale / r2 : R(0);
        } else {
          f = (R)((double)a.scale / (a.a0 + a.a1 * (double)(sz * sz + f1[c])));
        }
        if (store && kx0 + c != 0) {
          const double n = __fma_rn((double)v[c][e].x, (double)v[c][e].x, (double)v[c][e].y * (double)v[c][e].y);
          const double w = 2.0 * (double)(SYM == kSymProj ? f : a.scale);
          acc[c] = __fma_rn(w, n, acc[c]);
          if constexpr (SYM == kSymLap) acc2[c] = __fma_rn(2.0 * (double)f, n, acc2[c]);
        }
        v[c][e] = cscale(v[c][e], f);
      }
    }
    LS::template inv_cols<CPT>(v, lds + col0, B, t, stw);
#pragma unroll
    for (int e = 0; e < LS::E; ++e) {
      CO* d = a.z + oo + (long)LS::idxA(t, e) * bo;
      if constexpr (CPT == 2) {
        if (store && kx0 != 0)
          st_stream_f4(d, make_float4(v[0][e].x, v[0][e].y, v[CPT - 1][e].x, v[CPT - 1][e].y));
        else if (store)
          d[1] = v[CPT - 1][e];
      } else {
        if (store && kx0 != 0) st_stream(d, mk<CO>((RO)v[0][e].x, (RO)v[0][e].y));
      }
    }
  }
  double* cr = reinterpret_cast<double*>(smem_raw);
  auto emit = [&](double (&v)[CPT], double* out) {
    const double sum = isdc ? block_sum(v[0], red) : tile_tree<LS::T, CPT>(v, B / CPT, cr);
    if (threadIdx.x == 0) out[part] = sum;
  };
  emit(acc, a.partials);
  if constexpr (SYM == kSymLap) {
    __syncthreads();
    emit(acc2, a.partials2);
  }
}

// ---------------------------------------------------------------------------
// Inverse N2 pass of z fused with the CG vectors, per line of a component, in
// iteration k:
//   pi_k = z + beta pi_{k-1}  (pi_0 = z), into buffer k mod 2,
//   xi += alpha_{k-2} pi_{k-2} + alpha_{k-1} pi_{k-1}  for even k > 0 (xi
//   starts at 0): both steps in one pass over xi, 13.5 words per voxel on
//   average where a step in every iteration took 15.
// Without TWO (small grids, whose vectors stay in the last-level cache, and the
// scalar problems): one buffer, and
//   xi += alpha_{k-1} pi_{k-1}  (k > 0),  xi = 0  (k = 0).
// 256^3 iteration with / without TWO: 1653 / 1710 us FP64, 835 / 861 FP32; but
// 48 x 96 x 192 FP32 17.7 / 15.7 us of this pass, 96^3 FP64 20.2 / 19.2.
// grid: line blocks of the item's lines (nlines per component), blockIdx.y =
// item; in: line or (planes) plane layout.  Without ks: z alone, into pi.
//
// With prr (prz of the preconditioned CG), the partial sums of the iteration
// before that k_plane left (np per item): every workgroup adds them up itself, in
// the same order, for beta and the end of the solve, and one of them notes
// what it found for the passes behind.  A kernel of its own between the two
// took 2.6-4.6 us of an iteration of 30-60.
template <typename R> struct DirArgs {
  const cplx<R>* in;
  cplx<R>*pi, *xi;
  long pi2;  // distance of the second buffer of pi, or 0
  int nlines, nc, planes;
  SpecTables<R> tb;
  KrylovScalars* ks;
  const double *prr, *prz;
  int np;
};

template <typename R, int M, bool TWO>
__global__ void __launch_bounds__(XBLOCK) k_c2r_dir(DirArgs<R> a) {
  using C = cplx<R>;
  using LS = Line<M>;
  constexpr int LPB = XBLOCK / LS::T;
  constexpr int PAD = (M >= 16) ? 1 : 0;
  __shared__ C lds[LPB * (M + PAD)];
  __shared__ C stw[M], spost[M];
  __shared__ double red[16];
  const int item = blockIdx.y, nlines = a.nlines, planes = a.planes;
  const C* __restrict__ in = a.in;
  KrylovScalars* ks = a.ks ? a.ks + item : nullptr;
  const int k = ks ? ks->iter + (a.prr && !ks->fresh ? 1 : 0) : 0;  // this iteration
  const bool first = k == 0;
  const bool step = TWO ? (k & 1) == 0 && k > 0 : true;    // xi is taken on
  C* pi = a.pi + (TWO ? (k & 1) * a.pi2 : 0);              // pi_k (and pi_{k-2} before)
  const C* p1 = a.pi + (TWO ? ((k + 1) & 1) * a.pi2 : 0);  // pi_{k-1}
  C* xi = a.xi;
  const int t = threadIdx.x % LS::T;
  const int ll = threadIdx.x / LS::T;
  const int all = a.nc * nlines;  // lines of the item
  const int lin0 = (int)blockIdx.x * LPB, lin = lin0 + ll;
  const bool active = lin < all;
  const long ib = (long)item * all * M;
  const long base = ib + (long)(active ? lin : 0) * M;
  C* my = lds + ll * (M + PAD);
  C v[LS::E];
  if (planes) {
    static_assert(LPB * M == LS::E * XBLOCK, "elements per thread");
    const int c0 = lin0 / nlines;
#pragma unroll
    for (int e = 0; e < LS::E; ++e) {
      const int i = threadIdx.x + e * XBLOCK, k = i / LPB, j = i % LPB;
      int c = c0, r = lin0 + j - c0 * nlines;
      while (r >= nlines) {
        r -= nlines;
        ++c;
      }
      v[e] = lin0 + j < all ? in[ib + ((long)c * M + k) * nlines + r] : mk<C>(R(0), R(0));
    }
  } else {
#pragma unroll
    for (int e = 0; e < LS::E; ++e)
      v[e] = active ? (sizeof(R) == 8 ? ld_stream(in + base + LS::idxA(t, e)) : in[base + LS::idxA(t, e)])
                    : mk<C>(R(0), R(0));
  }
  // the vectors are read with the spectrum where the registers allow it (one
  // memory latency instead of two: what the pass costs on small grids)
  constexpr bool kAhead = LS::E * sizeof(C) <= 192;
  constexpr int NV = kAhead ? LS::E : (LS::E % 8 == 0 ? 8 : LS::E);  // elements read together
  C po[NV], qo[TWO ? NV : 1], xo[NV];
  auto vectors = [&](int e0) {
#pragma unroll
    for (int e = 0; e < NV; ++e) {
      const long n = base + LS::idxB(t, e0 + e);
      po[e] = p1[n];
      if constexpr (TWO) {
        qo[e] = xo[e] = mk<C>(R(0), R(0));
        if (step) {
          qo[e] = pi[n];
          if (k != 2) xo[e] = xi[n];  // (it starts there)
        }
      } else {
        xo[e] = xi[n];
      }
    }
  };
  if constexpr (kAhead) {
    if ((TWO ? !first : ks != nullptr) && active) vectors(0);  // (not used by the first iteration)
  }
  double rr = 0.0, rz = 0.0;
  if (a.prr) rr = thread_partials(a.prr + (long)item * a.np, a.np);
  if (a.prz) rz = thread_partials(a.prz + (long)item * a.np, a.np);
  TwiddleRegs<C, M> tw(a.tb);
  tw.store(stw, spost);
  if (ks && ks->done) return;  // (read with the data, not before it)
  const bool pending = ks && a.prr && !ks->fresh;
  R alpha = R(0), alpha1 = R(0), beta = R(0);
  if (!first) {
    alpha = (R)ks->alpha;
    if (TWO) alpha1 = (R)ks->alpha1;
    beta = (R)ks->beta;
  }
  if (pending) {
    rr = block_sum_all(rr, red);
    if (a.prz) rz = block_sum_all(rz, red + 8);
    const KrylovTest kt = krylov_test(ks, rr, rz, a.prz != nullptr);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      ks->run_rr = rr;
      ks->run_rz = rz;
      ks->run_iter = kt.iter;
      ks->stop = kt.done;
    }
    if (kt.done) return;
    beta = (R)kt.beta;
  }
  if (planes) {
#pragma unroll
    for (int e = 0; e < LS::E; ++e) {
      const int i = threadIdx.x + e * XBLOCK;
      lds[(i % LPB) * (M + PAD) + i / LPB] = v[e];
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < LS::E; ++e) v[e] = my[LS::idxA(t, e)];
  } else {
#pragma unroll
    for (int e = 0; e < LS::E; ++e) my[LS::idxA(t, e)] = v[e];
    __syncthreads();
  }
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
  if (!active) return;
  if (first) {
#pragma unroll
    for (int e = 0; e < LS::E; ++e) {
      const long n = base + LS::idxB(t, e);
      pi[n] = v[e];
      if (xi && !TWO) xi[n] = mk<C>(R(0), R(0));
    }
    return;
  }
#pragma unroll
  for (int e0 = 0; e0 < LS::E; e0 += NV) {
    if constexpr (!kAhead) vectors(e0);
#pragma unroll
    for (int e = 0; e < NV; ++e) {
      const long n = base + LS::idxB(t, e0 + e);
      const C p = po[e], z = v[e0 + e];
      if (step) {
        C x = xo[e];
        if constexpr (TWO) x = mk<C>(x.x + alpha1 * qo[e].x, x.y + alpha1 * qo[e].y);
        xi[n] = mk<C>(x.x + alpha * p.x, x.y + alpha * p.y);
      }
      pi[n] = mk<C>(z.x + beta * p.x, z.y + beta * p.y);
    }
  }
}

}  // namespace fg
