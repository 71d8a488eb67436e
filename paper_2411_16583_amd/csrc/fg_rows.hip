// Launchers of the projection's first half on 9-component fields.
#include <algorithm>
#include <stdexcept>

#include "fg_fft_sizes.hpp"
#include "fg_launch.hpp"
#include "fg_rows.hpp"

namespace fg {

void launch_rows_n1(int N1, int N0, double* y, double* dc, int M, int tile, const SpecTables<double>& tb,
                    const Gate& gate, int nitems, hipStream_t s) {
  tile &= ~kTileColumnPairs;
  const int T = zline_threads(N1);
  int B = tile > 0 ? tile : zgrad_tile(N1, M, (int)sizeof(double2));
  // (a tile chosen for the line shape of another N1 pass)
  while (B > 1 && (T * B > 256 || (size_t)N1 * (B + 1) * sizeof(double2) > 65536)) B /= 2;
  const unsigned shm = (unsigned)((size_t)N1 * (B + 1) * sizeof(double2));
  const dim3 grid((unsigned)(M / B), (unsigned)N0, (unsigned)(3 * nitems));
  const RowsN1Args a{reinterpret_cast<double2*>(y), reinterpret_cast<double2*>(dc), M, B, tb, gate};
  switch (N1) {
#define FG_CASE(L_) \
  case L_: hipLaunchKernelGGL((k_rows_n1<L_>), grid, dim3(T * B), shm, s, a); return;
    FG_FOR_N1(FG_CASE)
#undef FG_CASE
  }
  throw std::invalid_argument("unsupported N1");
}

template <typename RO, typename Z>
Parts launch_rows_n0(int N0, int mode, RowsN0Args<RO, Z> a, int nitems, hipStream_t s) {
  const N0Tile t = n0_tile<double>(N0, a.N1, a.M, a.tile, 3);
  a.kymajor = t.kymajor;
  a.tile = t.B;
  a.ndc = a.N1 / 2 + 1;
  a.nmain = (a.M / t.B) * a.N1;
  const unsigned shm = (unsigned)rows_n0_lds(N0, t.B);
  const dim3 grid((unsigned)((long)t.parts.stride() * nitems)), block((unsigned)(t.T * std::max(t.B, 2)));
  constexpr bool kF64 = sizeof(RO) == 8;
  switch (N0) {
#define FG_CASE(L_)                                                                              \
  case L_:                                                                                       \
    if (mode == kRowsStart)                                                                      \
      hipLaunchKernelGGL((k_rows_n0<L_, RO, Z, kRowsStart>), grid, block, shm, s, a);            \
    if constexpr (kF64) {                                                                        \
      if (mode == kRowsNorm)                                                                     \
        hipLaunchKernelGGL((k_rows_n0<L_, RO, Z, kRowsNorm>), grid, block, shm, s, a);           \
      if (mode == kRowsApply)                                                                    \
        hipLaunchKernelGGL((k_rows_n0<L_, RO, Z, kRowsApply>), grid, block, shm, s, a);          \
    }                                                                                            \
    return t.parts;
    FG_FOR_AXIS(FG_CASE)
#undef FG_CASE
  }
  throw std::invalid_argument("unsupported N0");
}

template <typename RO>
void launch_rows_out(int n1, long nlines, const double* z, RO* out, const SpecTables<double>& tb, const Gate& gate,
                     int nitems, hipStream_t s) {
  const int lpb = rows_out_lines(n1);
  const unsigned shm = (unsigned)(((size_t)lpb * (n1 | 1) + n1) * sizeof(double2));
  const dim3 grid((unsigned)((nlines + lpb - 1) / lpb), (unsigned)nitems);
  hipLaunchKernelGGL((k_rows_out<RO>), grid, dim3(kRowsOutThreads), shm, s, reinterpret_cast<const double2*>(z),
                     reinterpret_cast<cplx<RO>*>(out), n1, nlines, tb.tw1, gate);
}

template Parts launch_rows_n0<double, double>(int, int, RowsN0Args<double, double>, int, hipStream_t);
template Parts launch_rows_n0<float, float>(int, int, RowsN0Args<float, float>, int, hipStream_t);
template Parts launch_rows_n0<float, double>(int, int, RowsN0Args<float, double>, int, hipStream_t);
template void launch_rows_out<double>(int, long, const double*, double*, const SpecTables<double>&, const Gate&, int,
                                      hipStream_t);
template void launch_rows_out<float>(int, long, const double*, float*, const SpecTables<double>&, const Gate&, int,
                                     hipStream_t);

}  // namespace fg
