// Definitions of the FFT pass launchers (included by fg_fft_f64.hip and
// fg_fft_f32.hip, one working precision each).
#pragma once
#include <hip/hip_ext.h>
#include <algorithm>
#include <stdexcept>
#include <string>
#include <type_traits>

#include "fg_fft_sizes.hpp"
#include "fg_launch.hpp"

namespace fg {

template <typename R>
void launch_r2c(int M, const R* in, R* out, long nlines, const SpecTables<R>& tb, const Skip& skip,
                hipStream_t s) {
  switch (M) {
#define FG_CASE(L_)                                                                        \
  case L_: {                                                                               \
    constexpr int LPB = XBLOCK / Line<L_>::T;                                              \
    const long blocks = skip.line_blocks(nlines, LPB);                                     \
    hipLaunchKernelGGL((k_fft_x_r2c<R, L_>), dim3((unsigned)blocks), dim3(XBLOCK), 0, s, in, out, \
                       nlines, tb, skip);                                                  \
    return;                                                                                \
  }
    FG_FOR_M(FG_CASE)
#undef FG_CASE
  }
  throw std::invalid_argument("unsupported N2/2");
}

template <typename R>
void launch_c2r(int M, const R* in, R* out, long nlines, const SpecTables<R>& tb, double scale, const Skip& skip,
                hipStream_t s) {
  switch (M) {
#define FG_CASE(L_)                                                                                      \
  case L_: {                                                                                             \
    constexpr int LPB = XBLOCK / Line<L_>::T;                                                            \
    const long blocks = skip.line_blocks(nlines, LPB);                                                   \
    hipLaunchKernelGGL((k_fft_x_c2r<R, L_>), dim3((unsigned)blocks), dim3(XBLOCK), 0, s, in, out, nlines, \
                       tb, scale, skip);                                                                 \
    return;                                                                                              \
  }
    FG_FOR_M(FG_CASE)
#undef FG_CASE
  }
  throw std::invalid_argument("unsupported N2/2");
}

template <typename R>
void launch_axis(int L, bool inv, R* data, long estride, long ystride, long zstride, int M, int gy, int gz,
                 const cplx<R>* tw, const Skip& skip, hipStream_t s, int tile, hipEvent_t ev0, hipEvent_t ev1) {
  // single precision, on request: two columns per thread (16-byte accesses)
  int cpt = (sizeof(R) == 4 && (tile & kTileColumnPairs)) ? 2 : 1;
  tile &= ~kTileColumnPairs;
  const int T = line_threads(L);
  const int B = tile > 0 ? tile : column_tile_cpt(L, M, (int)sizeof(cplx<R>), cpt);
  if (B % cpt != 0) cpt = 1;
  // single precision reads the stage twiddles from LDS where they fit beside
  // the exchange buffer (the inverse N1 pass at 256^3: 94 -> 71 us); double
  // precision keeps them in the caches (its LDS is what bounds occupancy)
  const bool twl = sizeof(R) == 4 && (size_t)(L * B + L) * sizeof(cplx<R>) <= 65536;
  const size_t shm = (size_t)(L * B + (twl ? L : 0)) * sizeof(cplx<R>);
  dim3 grid((unsigned)(M / B), (unsigned)gy, (unsigned)gz);
  const dim3 block((unsigned)(T * B / cpt));
  constexpr int CP = (sizeof(R) == 4) ? 2 : 1;
  constexpr bool TW = sizeof(R) == 4;
  switch (L) {
#define FG_AXIS_GO(L_, INV_, CPT_)                                                                            \
  do {                                                                                                      \
    if (twl)                                                                                                \
      launch_ev((k_fft_axis<R, L_, INV_, CPT_, TW>), grid, block, shm, s, ev0, ev1, data, estride, ystride, \
                zstride, B, tw, skip);                                                                      \
    else                                                                                                    \
      launch_ev((k_fft_axis<R, L_, INV_, CPT_, false>), grid, block, shm, s, ev0, ev1, data, estride,       \
                ystride, zstride, B, tw, skip);                                                             \
  } while (0)
#define FG_CASE(L_)                 \
  case L_:                          \
    if (cpt == 2) {                 \
      if (inv)                      \
        FG_AXIS_GO(L_, true, CP);   \
      else                          \
        FG_AXIS_GO(L_, false, CP);  \
    } else {                        \
      if (inv)                      \
        FG_AXIS_GO(L_, true, 1);    \
      else                          \
        FG_AXIS_GO(L_, false, 1);   \
    }                               \
    return;
    FG_FOR_N1(FG_CASE)
#undef FG_CASE
#undef FG_AXIS_GO
  }
  throw std::invalid_argument("unsupported axis length");
}

template <typename R>
void launch_zproj(int N0, R* data, int N1, int M, const SpecTables<R>& tb, R scale, const Skip& skip,
                  hipStream_t s, int nitems, int tile) {
  const int T = zline_threads(N0);
  // built-in choice (tile 0): the largest tile, workgroups ky fastest
  const int kymajor = (tile == 0 || (tile & kTileKyMajor)) ? 1 : 0;
  tile &= ~kTileKyMajor;
  int B = tile > 0 ? tile : column_tile_t(T, N0, M, (int)sizeof(cplx<R>));
  while (B > 1 && T * B > 256) B /= 2;  // a tile chosen for the column-pair N0 pass
  const size_t shm = (size_t)N0 * B * sizeof(cplx<R>) + zpass_extra_lds<R>(N0);
  dim3 grid = kymajor ? dim3((unsigned)N1, (unsigned)(M / B), (unsigned)(3 * nitems))
                      : dim3((unsigned)(M / B), (unsigned)N1, (unsigned)(3 * nitems));
  dim3 gdc((unsigned)(N1 / 2 + 1), (unsigned)(3 * nitems), 1);
  switch (N0) {
#define FG_CASE(L_)                                                                                    \
  case L_:                                                                                             \
    hipLaunchKernelGGL((k_fft_z_proj<R, L_>), grid, dim3(T * B), shm, s, data, N1, M, B, tb, scale, skip, \
                       kymajor);                                                                       \
    hipLaunchKernelGGL((k_fft_z_dc<R, L_>), gdc, dim3(192), 0, s, data, N1, M, tb, scale, skip);       \
    return;
    FG_FOR_AXIS(FG_CASE)
#undef FG_CASE
  }
  throw std::invalid_argument("unsupported N0");
}

template <typename R, typename RQ>
int launch_cg_op(int law, RQ* q, RQ* edge, const R* pi, long pi2, const KrylovScalars* ks, const R* st,
                 double* partials, const Gate& gate, int n0, int n1, int n2, const double h[3], int nitems,
                 hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  OpArgs<R, RQ> a;
  a.el = edge_layout<R>(n0, n1, n2);
  const OpSplit sp = op_split(n0, n1, n2, a.el, nitems);
  a.q = q;
  a.edge = edge;
  a.pi = pi;
  a.pi2 = pi2;
  a.ks = ks;
  a.st = st;
  a.partials = partials;
  a.gate = gate;
  a.n0 = n0;
  a.n1 = n1;
  a.n2 = n2;
  a.K = sp.K;
  a.nseg = sp.nseg;
  a.groups = sp.groups;
  a.q0 = (R)(0.25 / h[0]);
  a.q1 = (R)(0.25 / h[1]);
  a.q2 = (R)(0.25 / h[2]);
  auto go = [&](auto width) {
    constexpr int W = decltype(width)::value;
    const dim3 grid((unsigned)((long)sp.groups * nitems)), block(kOpThreads);
    if (law == kLawSVK)
      launch_ev((k_cg_op<R, RQ, W, kLawSVK>), grid, block, 0, s, ev0, ev1, a);
    else
      launch_ev((k_cg_op<R, RQ, W, kLawNH>), grid, block, 0, s, ev0, ev1, a);
  };
  if constexpr (sizeof(R) == 4) {
    if (a.el.W8 == 4 * kPatch) {
      go(std::integral_constant<int, 4>());
      return sp.groups;
    }
  }
  go(std::integral_constant<int, 2>());
  return sp.groups;
}

template <typename R>
void launch_r2c_edges(int M, const R* q, const R* edge, const EdgeLayout& el, R* out, const Gate& gate, int n0, int n1,
                      const SpecTables<R>& tb, int nitems, int planes, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  switch (M) {
#define FG_CASE(L_)                                                                                              \
  case L_: {                                                                                                     \
    constexpr int LPB = XBLOCK / Line<L_>::T;                                                                    \
    const dim3 grid((unsigned)((3L * n0 * n1 + LPB - 1) / LPB), (unsigned)nitems);                               \
    launch_ev((k_r2c_edges<R, L_>), grid, dim3(XBLOCK), 0, s, ev0, ev1, q, edge, el, reinterpret_cast<cplx<R>*>(out), \
              n0, n1, tb, gate, planes);                                                                              \
    return;                                                                                                      \
  }
    FG_FOR_M(FG_CASE)
#undef FG_CASE
  }
  throw std::invalid_argument("unsupported N2/2");
}

template <typename R>
void launch_n1(int N1, bool inv, int N0, N1Args<R> a, int nitems, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  const int T = line_threads(N1);
  int B = a.tile & ~kTileColumnPairs;
  if (B == 0) B = column_tile(N1, a.M, (int)sizeof(cplx<R>));
  while (B > 1 && T * B > 256) B /= 2;  // a tile of column pairs: one column per thread here
  // single precision reads the stage twiddles from LDS where they fit beside
  // the exchange buffer (as launch_axis)
  const bool twl = sizeof(R) == 4 && (size_t)(N1 * B + N1) * sizeof(cplx<R>) <= 65536;
  const size_t shm = (size_t)(N1 * B + (twl ? N1 : 0)) * sizeof(cplx<R>);
  a.tile = B;
  const dim3 grid((unsigned)(a.M / B), (unsigned)(N0 + (a.ks ? 1 : 0)), (unsigned)(a.nc * nitems));
  const dim3 block((unsigned)(T * B));
  constexpr bool TW = sizeof(R) == 4;
  switch (N1) {
#define FG_N1_GO(L_, INV_)                                                                \
  do {                                                                                    \
    if (twl)                                                                              \
      launch_ev((k_n1<R, L_, INV_, TW>), grid, block, (unsigned)shm, s, ev0, ev1, a);     \
    else                                                                                  \
      launch_ev((k_n1<R, L_, INV_, false>), grid, block, (unsigned)shm, s, ev0, ev1, a);  \
  } while (0)
#define FG_CASE(L_)          \
  case L_:                   \
    if (inv)                 \
      FG_N1_GO(L_, true);    \
    else                     \
      FG_N1_GO(L_, false);   \
    return;
    FG_FOR_N1(FG_CASE)
#undef FG_CASE
#undef FG_N1_GO
  }
  throw std::invalid_argument("unsupported N1");
}

template <typename R> N0Tile n0_tile(int N0, int N1, int M, int tile, int nc) {
  const int eb = (int)sizeof(cplx<R>);
  const int T = zgrad_threads(N0, eb);
  N0Tile t;
  // built-in choice: the largest tile, workgroups ky fastest (consecutive
  // blocks in memory)
  t.kymajor = (tile == 0 || (tile & kTileKyMajor)) ? 1 : 0;
  int B = tile & ~kTileKyMajor;
  if (B == 0) B = zgrad_tile(N0, M, eb);
  // two columns per thread round differently from one (other contractions): no
  // single column where there are pairs
  if (B == 1 && zgrad_cpt(N0, eb) == 2 && M % 2 == 0) B = 2;
  auto cpt_of = [&](int b) { return (b % 2 == 0) ? zgrad_cpt(N0, eb) : 1; };
  while (B > 1 && T * B / cpt_of(B) > 256) B /= 2;  // a tile chosen for another line shape
  t.B = B;
  t.cpt = cpt_of(B);
  t.T = T;
  const int bm = M & -M;  // a row of ky in groups of the largest power of two of columns
  const int ndc = N1 / 2 + 1;
  t.parts = Parts(nc * (ndc + N1 * (M / bm)), nc * ndc, bm / B);
  return t;
}

template <typename R, typename RO>
Parts launch_n0(int N0, int mode, int sym, N0Args<R, RO> a, int nitems, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  const N0Tile t = n0_tile<R>(N0, a.N1, a.M, a.tile, a.nc);
  const int B = t.B, T = t.T, cpt = t.cpt;
  const Parts parts = t.parts;
  a.kymajor = t.kymajor;
  a.tile = B;
  a.ndc = a.N1 / 2 + 1;
  a.nmain = (a.M / B) * a.N1;
  const size_t shm = (size_t)N0 * std::max(B, 4) * sizeof(cplx<R>) + n0_extra_lds<R>(N0);
  const dim3 grid((unsigned)((long)parts.stride() * nitems));
  const dim3 block((unsigned)std::max(T * B / cpt, 2 * T));
  constexpr int CP = (sizeof(R) == 4) ? 2 : 1;
  constexpr bool kSame = sizeof(R) == sizeof(RO);
  switch (N0) {
#define FG_N0_GO(L_, MODE_, SYM_)                                                                \
  do {                                                                                           \
    if (cpt == 2)                                                                                \
      launch_ev((k_n0<R, RO, L_, CP, MODE_, SYM_>), grid, block, (unsigned)shm, s, ev0, ev1, a); \
    else                                                                                         \
      launch_ev((k_n0<R, RO, L_, 1, MODE_, SYM_>), grid, block, (unsigned)shm, s, ev0, ev1, a);  \
  } while (0)
#define FG_CASE(L_)                                              \
  case L_:                                                       \
    if (sym == kSymLap) {                                        \
      if constexpr (sizeof(R) == 8 && kSame) {                   \
        if (mode == kN0Cg)                                       \
          FG_N0_GO(L_, kN0Cg, kSymLap);                          \
        else                                                     \
          FG_N0_GO(L_, kN0Start, kSymLap);                       \
      }                                                          \
    } else if (mode == kN0Cg) {                                  \
      FG_N0_GO(L_, kN0Cg, kSymProj);                             \
    }                                                            \
    return parts;
    FG_FOR_AXIS(FG_CASE)
#undef FG_CASE
#undef FG_N0_GO
  }
  throw std::invalid_argument("unsupported N0");
}

template <typename R>
void launch_c2r_dir(int M, const DirArgs<R>& a, int nitems, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  switch (M) {
#define FG_CASE(L_)                                                                                              \
  case L_: {                                                                                                     \
    constexpr int LPB = XBLOCK / Line<L_>::T;                                                                    \
    const dim3 grid((unsigned)((a.nc * a.nlines + LPB - 1) / LPB), (unsigned)nitems);                            \
    if (a.pi2 != 0)                                                                                              \
      launch_ev((k_c2r_dir<R, L_, true>), grid, dim3(XBLOCK), 0, s, ev0, ev1, a);                                \
    else                                                                                                         \
      launch_ev((k_c2r_dir<R, L_, false>), grid, dim3(XBLOCK), 0, s, ev0, ev1, a);                               \
    return;                                                                                                      \
  }
    FG_FOR_M(FG_CASE)
#undef FG_CASE
  }
  throw std::invalid_argument("unsupported N2/2");
}

template <typename R>
int launch_cg_lines(int law, int M, LinesArgs<R> a, int nitems, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
  a.nb = (a.n1 + a.L - 1) / a.L;
  a.groups = a.n0 * a.nb;
  const dim3 grid((unsigned)(a.groups * nitems)), block(kLinesThreads);
  switch (M) {
#define FG_CASE(L_)                                                                                               \
  case L_: {                                                                                                      \
    const unsigned shm = (unsigned)lines_lds(sizeof(R), L_, a.L);                                                  \
    if (law == kLawSVK)                                                                                           \
      launch_ev((k_cg_lines<R, L_, kLawSVK>), grid, block, shm, s, ev0, ev1, a);                                  \
    else                                                                                                          \
      launch_ev((k_cg_lines<R, L_, kLawNH>), grid, block, shm, s, ev0, ev1, a);                                   \
    return a.groups;                                                                                              \
  }
    FG_FOR_LINES(FG_CASE)
#undef FG_CASE
  }
  throw std::invalid_argument("unsupported N2/2");
}

template <typename R, typename RO>
Parts launch_plane(int mode, int sym, PlaneArgs<R, RO> a, int nc, int nitems, hipStream_t s, hipEvent_t ev0,
                   hipEvent_t ev1) {
  a.P = planes_per_group(a.n0, a.n1, a.M, nc, nitems);
  a.groups = nc * a.M / a.P;
  a.dn1 = FastDiv(a.n1);
  const dim3 grid((unsigned)(a.groups * nitems));
  // a thread per line task where the bound allows
  const int tasks = a.P * std::max(a.n0 * zline_threads(a.n1), a.n1 * zline_threads(a.n0));
  // (see the kernel's launch bounds)
  const bool shared = sizeof(R) == 4 && a.groups * nitems > 256;
  const dim3 block((unsigned)std::min(sizeof(R) == 8 || shared ? 512 : 768, (tasks + 63) / 64 * 64));
  const unsigned shm = (unsigned)plane_lds<R>(a.n0, a.n1, a.P);
  auto go = [&](auto kernel) {
    if (shm > 65536) {
      // the limit belongs to the kernel and the device, not to this launch: every
      // launch sets the same one, so that plans of other planes in other
      // threads do not lower it between the two (setting it again is cheap)
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)kPlaneLds);
      if (e != hipSuccess) throw std::runtime_error(std::string("hipFuncSetAttribute: ") + hipGetErrorString(e));
    }
    launch_ev(kernel, grid, block, shm, s, ev0, ev1, a);
  };
  constexpr bool kSame = sizeof(R) == sizeof(RO);
  constexpr int TH = 512;
  if (sym == kSymLap) {
    if constexpr (sizeof(R) == 8 && kSame) {
      if (mode == kN0Cg)
        go(k_plane<R, RO, kN0Cg, kSymLap, TH>);
      else
        go(k_plane<R, RO, kN0Start, kSymLap, TH>);
    }
  } else if (mode == kN0Cg) {
    if constexpr (sizeof(R) == 4) {
      if (shared)
        go(k_plane<R, RO, kN0Cg, kSymProj, 1024>);
      else
        go(k_plane<R, RO, kN0Cg, kSymProj, 768>);
    } else {
      go(k_plane<R, RO, kN0Cg, kSymProj, TH>);
    }
  }
  return Parts(a.groups);
}

#define FG_INSTANTIATE_LAUNCHERS(R)                                                                     \
  template int launch_cg_op<R, R>(int, R*, R*, const R*, long, const KrylovScalars*, const R*, double*, const Gate&,  \
                                  int, int, int, const double*, int, hipStream_t, hipEvent_t, hipEvent_t); \
  template void launch_r2c_edges<R>(int, const R*, const R*, const EdgeLayout&, R*, const Gate&, int, int,            \
                                    const SpecTables<R>&, int, int, hipStream_t, hipEvent_t, hipEvent_t);  \
  template void launch_n1<R>(int, bool, int, N1Args<R>, int, hipStream_t, hipEvent_t, hipEvent_t);      \
  template N0Tile n0_tile<R>(int, int, int, int, int);                                                  \
  template Parts launch_n0<R, R>(int, int, int, N0Args<R, R>, int, hipStream_t, hipEvent_t, hipEvent_t);       \
  template Parts launch_plane<R, R>(int, int, PlaneArgs<R, R>, int, int, hipStream_t, hipEvent_t, hipEvent_t); \
  template int launch_cg_lines<R>(int, int, LinesArgs<R>, int, hipStream_t, hipEvent_t, hipEvent_t);     \
  template void launch_c2r_dir<R>(int, const DirArgs<R>&, int, hipStream_t, hipEvent_t, hipEvent_t);     \
  template void launch_r2c<R>(int, const R*, R*, long, const SpecTables<R>&, const Skip&, hipStream_t); \
  template void launch_c2r<R>(int, const R*, R*, long, const SpecTables<R>&, double, const Skip&, hipStream_t); \
  template void launch_axis<R>(int, bool, R*, long, long, long, int, int, int, const cplx<R>*, const Skip&, \
                               hipStream_t, int, hipEvent_t, hipEvent_t);                               \
  template void launch_zproj<R>(int, R*, int, int, const SpecTables<R>&, R, const Skip&, hipStream_t, int, int);

}  // namespace fg
