// The projection's first half on 9-component double-precision fields, with
// every product in the spectrum: s = D^T Y and (D^T D)^+ s of the CG's
// residual (the right-hand side and the Newton residual), and fg_project_grad.
//
// The CG iteration forms D^T Y in real space (k_cg_op): the rounding of those
// differences and of the transforms of s is white, about eps |Y| / h, and the
// division by |r|^2 in the spectrum amplifies it by 1 / |r|.  Within an
// iteration that is below what the iteration leaves; in the residual it is the
// error of the answer, so here the spectrum of Y is multiplied by the symbol
//   s^_i = -i e^{i Phi} sum_l r_l Y^_il,  r = (sz cy cx, cz sy cx, cz cy sx)
// (c* = cos(q/2), s* = (2/h) sin(q/2), Phi = (q0 + q1 + q2) / 2) and keeps
// eps |Y| whatever the voxel.
//
// Passes (words per voxel; us at 256^3): N2 transform of nine components (18;
// 436), k_rows_n1 (15: the two terms of a row that share the N0 factor cz are
// merged; 420), k_rows_n0 (6 in, 3 to 6 out; 324 into double, 260 into single),
// bound by HBM at 4.8-5.5 TB/s, once per Newton iteration.  fg_residual (two
// residuals and two stresses, us) with the differences in real space | here:
// 256^3 2470 | 2910, 128^3 361 | 374, 96^3 182 | 202, 64^3 100 | 116, 16^3 84 | 84
// (before the divergence form 3970, 552, 331, 169, 123).  |G*Y| of an equilibrated
// field, which is rounding: 0.9e-15 to 3e-15 |Y| on voxels of 8:1 to 32:1 | 2.0e-16
// to 2.5e-16 on every grid.
#pragma once
#include "fg_plane.hpp"

namespace fg {

// k_rows_n0: the start of a CG (s, z and r.r), r.r alone, z alone.
constexpr int kRowsStart = 0, kRowsNorm = 1, kRowsApply = 2;

// Forward N1 pass, in place: a row i of the 3 x 3 field per workgroup slice,
//   slot 3i     <- cy cx A_i0
//   slot 3i + 1 <- sy cx A_i1 + cy sx A_i2
// (slot 3i + 2 is left).  The kx = 0 column packs the real columns kx = 0 and
// kx = N2/2, whose factors differ: it goes transformed, unscaled and unmerged to
// the compact array dc, [9 components][ky][i0] per item.
// Grid (M / tile, N0, 3 rows per item).
struct RowsN1Args {
  double2* y;  // spectrum along N2 of 9 components per item
  double2* dc;
  int M, tile;
  SpecTables<double> tb;
  Gate gate;
};

template <int L> __global__ void __launch_bounds__(256) k_rows_n1(RowsN1Args a) {
  using C = double2;
  using LS = ZLine<L>;
  extern __shared__ __align__(16) char smem_raw[];
  const int row = blockIdx.z, i0 = blockIdx.y, N0 = gridDim.y, B = a.tile;
  if (a.gate(row / 3)) return;
  C* lds = reinterpret_cast<C*>(smem_raw);
  C* stw = lds + L * B;
  for (int k = threadIdx.x; k < L; k += blockDim.x) stw[k] = a.tb.tw1[k];
  __syncthreads();
  const int col = threadIdx.x % B, t = threadIdx.x / B;
  const int kx = blockIdx.x * B + col;
  const double cx = a.tb.cx[kx], sx = a.tb.sx[kx];
  const bool dc = kx == 0;
  const long comp = (long)N0 * L * a.M;
  C* b0 = a.y + 3L * row * comp + (long)i0 * L * a.M + kx;
  C *b1 = b0 + comp, *b2 = b1 + comp;
  C* d = a.dc + 3L * row * L * N0 + i0;  // + (slot L + ky) N0
  C v[LS::E], w[LS::E];
#pragma unroll
  for (int e = 0; e < LS::E; ++e) {
    v[e] = ld_stream(b0 + (long)LS::idxA(t, e) * a.M);
    w[e] = ld_stream(b1 + (long)LS::idxA(t, e) * a.M);
  }
  LS::template fwd<false>(v, lds + col, B, t, stw);
#pragma unroll
  for (int e = 0; e < LS::E; ++e) {
    const int ky = LS::idxB(t, e);
    st_stream(b0 + (long)ky * a.M, cscale(v[e], a.tb.cy[ky] * cx));
    if (dc) d[(long)ky * N0] = v[e];
  }
#pragma unroll
  for (int e = 0; e < LS::E; ++e) v[e] = ld_stream(b2 + (long)LS::idxA(t, e) * a.M);
  LS::template fwd<false>(w, lds + col, B, t, stw);
  LS::template fwd<false>(v, lds + col, B, t, stw);
#pragma unroll
  for (int e = 0; e < LS::E; ++e) {
    const int ky = LS::idxB(t, e);
    const double f1 = a.tb.sy[ky] * cx, f2 = a.tb.cy[ky] * sx;
    st_stream(b1 + (long)ky * a.M, mk<C>(w[e].x * f1 + v[e].x * f2, w[e].y * f1 + v[e].y * f2));
    if (dc) {
      d[(long)(L + ky) * N0] = w[e];
      d[(long)(2 * L + ky) * N0] = v[e];
    }
  }
}

// N0 pass on the output of k_rows_n1: s^, the partial sums of
// r.r = sum f |s^|^2 (f = 1 / (N |r|^2), the columns kx > 0 twice), and
// z^ = f s^ transformed back along N0.  s and z go to the block layout (z to be
// taken on by the inverse k_n1) or, with planes, to the plane layout: s as
// k_plane keeps it, (kz, ky), and z as (i0, ky) for k_rows_out.
// The kx = 0 column: pairs (ky, -ky) as in k_n0, with the three components of a
// row separated into those of kx = 0 and kx = N2/2 before they are merged.
template <typename RO, typename Z> struct RowsN0Args {
  const double2 *y, *dc;
  cplx<Z>*z, *dcz;
  cplx<RO>*s, *dcs;
  BlockLayout blo;
  int N1, M, tile, kymajor, planes;
  int ndc, nmain;  // workgroups per row
  SpecTables<double> tb;
  double scale, sign;
  Gate gate;
  double* partials;  // as k_n0
};

// LDS beside the exchange buffer of `tile` columns; the column pairs take
// eight columns of it.
inline size_t rows_n0_lds(int L, int tile) {
  return (size_t)L * ((tile > 8 ? tile : 8) + 1) * sizeof(double2) + 3 * (size_t)L * sizeof(double);
}

template <int L, typename RO, typename Z, int MODE>
__global__ void __launch_bounds__(256) k_rows_n0(RowsN0Args<RO, Z> a) {
  using C = double2;
  using LS = typename ZGradSel<double, L>::type;
  extern __shared__ __align__(16) char smem_raw[];
  __shared__ double red[16];
  const unsigned per_row = (unsigned)(a.ndc + a.nmain), per_item = 3 * per_row;
  const int item = (int)(blockIdx.x / per_item);
  if (a.gate(item)) return;
  const unsigned rem = blockIdx.x - (unsigned)item * per_item;
  const bool isdc = rem < 3u * (unsigned)a.ndc;
  const int wdc = isdc ? a.ndc : a.nmain;
  const unsigned r2i = isdc ? rem : rem - 3u * (unsigned)a.ndc;
  const int row = (int)(r2i / (unsigned)wdc);
  const int idx = (int)(r2i - (unsigned)row * wdc);
  const long zc = 3L * item + row;
  const int B = a.tile, N1 = a.N1, M = a.M;
  C* stw = reinterpret_cast<C*>(smem_raw);
  C* lds = stw + L;
  double* scz = reinterpret_cast<double*>(lds + L * (B > 8 ? B : 8));
  double* ssz = scz + L;
  double* snz = ssz + L;
  for (int k = threadIdx.x; k < L; k += blockDim.x) {
    stw[k] = a.tb.tw0[k];
    scz[k] = a.tb.cz[k];
    ssz[k] = a.tb.sz[k];
    snz[k] = a.tb.snz[k];
  }
  __syncthreads();
  double acc[1] = {0.0};
  long part = blockIdx.x;
  if (isdc) {
    // threads beyond the pair's 2 T repeat the work of the first ones (equal
    // values to equal LDS places) and store nothing
    const int td = threadIdx.x % (2 * LS::T);
    const int col = td % 2, t = td / 2;
    const int ky0 = idx, ky1 = (ky0 == 0) ? 0 : N1 - ky0;
    const int ky = col ? ky1 : ky0;
    const bool store = (int)threadIdx.x < 2 * LS::T && (col == 0 || ky1 != ky0);
    C* sp = lds + 2 * L;  // [component][column][kz]
    C v[LS::E];
#pragma unroll 1
    for (int l = 0; l < 3; ++l) {
      const C* src = a.dc + ((3 * zc + l) * N1 + ky) * L;
#pragma unroll
      for (int e = 0; e < LS::E; ++e) v[e] = src[LS::idxA(t, e)];
      LS::template fwd<false>(v, lds + col, 2, t, stw);
#pragma unroll
      for (int e = 0; e < LS::E; ++e) sp[(2 * l + col) * L + LS::idxB(t, e)] = v[e];
    }
    __syncthreads();
    const double cy = a.tb.cy[ky], sy = a.tb.sy[ky], sxM = a.tb.sx[M];
    const C ey = mk<C>(cy, a.tb.sny[ky]);
    const long o = a.planes ? zc * M * L * N1 + ky : (zc * N1 + ky) * L;
    const int st = a.planes ? N1 : 1;
    cplx<Z>* dz = a.planes ? a.z : a.dcz;
    cplx<RO>* ds = a.planes ? a.s : a.dcs;
#pragma unroll
    for (int e = 0; e < LS::E; ++e) {
      const int kz = LS::idxB(t, e), kzm = kz == 0 ? 0 : L - kz;
      // kx = 0: r = (sz cy, cz sy, 0); kx = N2/2: (0, 0, cz cy sx), where the
      // phase takes another factor i
      const double ra = ssz[kz] * cy, rb = scz[kz] * sy, rc = scz[kz] * cy * sxM;
      auto P = [&](int l) { return sp[(2 * l + col) * L + kz]; };
      auto Q = [&](int l) { return cconj(sp[(2 * l + 1 - col) * L + kzm]); };
      const C A0 = cscale(cadd(P(0), Q(0)), 0.5), A1 = cscale(cadd(P(1), Q(1)), 0.5);
      const C B2 = cscale(mul_mi(csub(P(2), Q(2))), 0.5);
      const C ph = cmul(mk<C>(scz[kz], snz[kz]), ey);
      const C sA = cscale(mul_mi(cmul(mk<C>(A0.x * ra + A1.x * rb, A0.y * ra + A1.y * rb), ph)), a.sign);
      const C sB = cscale(cmul(cscale(B2, rc), ph), a.sign);
      const double a2 = ra * ra + rb * rb, b2 = rc * rc;
      const double fa = a2 > 0.0 ? a.scale / a2 : 0.0, fb = b2 > 0.0 ? a.scale / b2 : 0.0;
      if constexpr (MODE == kRowsStart) {
        const C p = cadd(sA, mul_pi(sB));
        if (store) ds[o + (long)kz * st] = mk<cplx<RO>>((RO)p.x, (RO)p.y);
      }
      if (MODE != kRowsApply && store)
        acc[0] += fa * (sA.x * sA.x + sA.y * sA.y) + fb * (sB.x * sB.x + sB.y * sB.y);
      v[e] = cadd(cscale(sA, fa), mul_pi(cscale(sB, fb)));
    }
    if constexpr (MODE != kRowsNorm) {
      LS::inv(v, lds + col, 2, t, stw);
      if (store) {
#pragma unroll
        for (int e = 0; e < LS::E; ++e) dz[o + (long)LS::idxA(t, e) * st] = mk<cplx<Z>>((Z)v[e].x, (Z)v[e].y);
      }
    }
  } else {
    const int nkx = M / B;
    const int ktile = a.kymajor ? idx / N1 : idx % nkx;
    const int ky = a.kymajor ? idx - ktile * N1 : idx / nkx;
    // (a workgroup wider than the tile, for the column pairs: repeats as above)
    const int tm = threadIdx.x % (LS::T * B);
    const int col = tm % B, t = tm / B;
    const int kx = ktile * B + col;
    const bool store = (int)threadIdx.x < LS::T * B && kx != 0;
    part = (long)item * per_item + 3L * a.ndc + ((long)row * N1 + ky) * nkx + ktile;
    const long plane = (long)N1 * M;
    const C* src = a.y + 3 * zc * L * plane + (long)ky * M + kx;
    const double cy = a.tb.cy[ky], sy = a.tb.sy[ky], cx = a.tb.cx[kx], sx = a.tb.sx[kx];
    const double f0 = cy * cx, f1 = sy * cx, f2 = cy * sx;
    // -i e^{i (qy + qx) / 2}
    const C eyx = mul_mi(cmul(mk<C>(cy, a.tb.sny[ky]), mk<C>(cx, a.tb.snx[kx])));
    C v[LS::E], w[LS::E];
#pragma unroll
    for (int e = 0; e < LS::E; ++e) {
      v[e] = ld_stream(src + LS::idxA(t, e) * plane);
      w[e] = ld_stream(src + (L + LS::idxA(t, e)) * plane);
    }
    LS::template fwd<false>(v, lds + col, B, t, stw);
    LS::template fwd<false>(w, lds + col, B, t, stw);
    const long o = a.planes ? (zc * M + kx) * L * N1 + ky : zc * a.blo.cstr + a.blo.at(N1, ky, kx);
    const int st = a.planes ? N1 : a.blo.B;
#pragma unroll
    for (int e = 0; e < LS::E; ++e) {
      const int kz = LS::idxB(t, e);
      const double sz = ssz[kz], cz = scz[kz];
      const C ph = cmul(mk<C>(cz, snz[kz]), eyx);
      const C s = cscale(cmul(mk<C>(v[e].x * sz + w[e].x * cz, v[e].y * sz + w[e].y * cz), ph), a.sign);
      const double r2 = sz * sz * (f0 * f0) + cz * cz * (f1 * f1 + f2 * f2);
      const double f = r2 > 0.0 ? a.scale / r2 : 0.0;
      if constexpr (MODE == kRowsStart) {
        if (store) a.s[o + (long)kz * st] = mk<cplx<RO>>((RO)s.x, (RO)s.y);
      }
      if (MODE != kRowsApply && store) acc[0] += 2.0 * f * (s.x * s.x + s.y * s.y);
      v[e] = cscale(s, f);
    }
    if constexpr (MODE != kRowsNorm) {
      LS::inv(v, lds + col, B, t, stw);
      if (store) {
#pragma unroll
        for (int e = 0; e < LS::E; ++e) a.z[o + (long)LS::idxA(t, e) * st] = mk<cplx<Z>>((Z)v[e].x, (Z)v[e].y);
      }
    }
  }
  if constexpr (MODE != kRowsApply) {
    double* cr = reinterpret_cast<double*>(smem_raw);
    const double sum = isdc ? block_sum(acc[0], red) : tile_tree<LS::T, 1>(acc, B, cr);
    if (threadIdx.x == 0) a.partials[part] = sum;
  }
}

// Inverse N1 pass of the plane layout: rows (i0) of n1 contiguous values, into
// the working type (in place where it is double).  grid (row blocks, items).
constexpr int kRowsOutThreads = 256;
__host__ __device__ inline int rows_out_lines(int n1) { return n1 >= 2048 ? 1 : 2048 / n1; }

template <typename RO>
__global__ void __launch_bounds__(kRowsOutThreads)
k_rows_out(const double2* z, cplx<RO>* out, int n1, long nlines, const double2* __restrict__ tw, Gate gate) {
  extern __shared__ __align__(16) char smem_raw[];
  if (gate(blockIdx.y)) return;
  const int lpb = rows_out_lines(n1), LD = n1 | 1;
  const long first = (long)blockIdx.x * lpb;
  const int nl = (int)min((long)lpb, nlines - first);
  double2* x = reinterpret_cast<double2*>(smem_raw);
  double2* stw = x + lpb * LD;
  const long base = ((long)blockIdx.y * nlines + first) * n1;
  for (int k = threadIdx.x; k < n1; k += kRowsOutThreads) stw[k] = tw[k];
  for (int i = threadIdx.x; i < nl * n1; i += kRowsOutThreads) {
    const int l = i / n1;
    x[l * LD + i - l * n1] = z[base + i];
  }
  __syncthreads();
  switch (n1) {
#define FG_CASE(L_) \
  case L_: plane_rows_inv<L_>(x, out + base, nl, stw); break;
    FG_PLANE_LINES(FG_CASE)
#undef FG_CASE
  }
}

}  // namespace fg
