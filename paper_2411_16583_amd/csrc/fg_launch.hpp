// Host-side launchers of the FFT passes (size dispatch).  Defined once per
// working precision in fg_fft_f64.hip / fg_fft_f32.hip.
#pragma once
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include "fg_cg3.hpp"
#include "fg_plane.hpp"
#include "fg_cg_lines.hpp"
#include "fg_rows.hpp"

namespace fg {

struct Grid3 {
  int n0, n1, n2;
  double ih0, ih1, ih2;  // 1 / h_j
};

// Launch that takes a timing event pair itself when one is given (the
// kernel's own start and end, no marker packets on the stream): ev0 is
// recorded at the start of this kernel, ev1 at its end; either may be null.
template <typename F, typename... A>
inline void launch_ev(F kernel, dim3 grid, dim3 block, unsigned shm, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1,
                      A... args) {
  if (ev0 || ev1)
    hipExtLaunchKernelGGL(kernel, grid, block, shm, s, ev0, ev1, 0, args...);
  else
    hipLaunchKernelGGL(kernel, grid, block, shm, s, args...);
}

bool fft_length_supported(int L);       // complex line lengths
bool fft_axis_length_supported(int L);  // N1 (and N0 > 1)
bool fft_n0_length_supported(int L);    // N0: the axis lengths and 1 (a plane)
bool fft_n1_length_supported(int L);    // N1: the axis lengths and 512

// Largest power-of-two column tile dividing M with T * B <= 256 threads and
// an exchange buffer of L * B complex values within 64 KiB.
int column_tile(int L, int M, int elem_bytes);
int column_tile_t(int T, int L, int M, int elem_bytes);
// largest tile for cpt columns per thread: T tile / cpt <= 256 threads
int column_tile_cpt(int L, int M, int elem_bytes, int cpt);
int line_threads(int L);
int zline_threads(int L);  // threads per line of the fused N0 projection pass
// threads per line and columns per thread of the N0 pass of the CG
// (elem_bytes: bytes of one complex value of the working precision)
int zgrad_threads(int L, int elem_bytes);
int zgrad_cpt(int L, int elem_bytes);
int zgrad_tile(int L, int M, int elem_bytes);  // built-in tile of launch_n0

// Plane runs and workgroups of launch_cg_op for nitems fields.
struct OpSplit {
  int K, nseg, groups;  // planes per run, runs, workgroups (partial sums) per item
};
OpSplit op_split(int n0, int n1, int n2, const EdgeLayout& el, int nitems);

// q = D^T K : (D pi) for all items, as k_cg_op leaves it (q and its patch edges,
// in precision RQ);
// h: grid spacings.  Returns the number of partial sums of p.Kp per item.
template <typename R, typename RQ>
int launch_cg_op(int law, RQ* q, RQ* edge, const R* pi, long pi2, const KrylovScalars* ks, const R* st,
                 double* partials, const Gate& gate, int n0, int n1, int n2, const double h[3], int nitems,
                 hipStream_t s, hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);
// N2 transform of q with its patch edges added (el: the operator's).
template <typename R>
void launch_r2c_edges(int M, const R* q, const R* edge, const EdgeLayout& el, R* out, const Gate& gate, int n0, int n1,
                      const SpecTables<R>& tb, int nitems, int planes, hipStream_t s, hipEvent_t ev0 = nullptr,
                      hipEvent_t ev1 = nullptr);
// N1 pass between the line layout and the block layout (k_n1), 3 components
// per item; tile as for launch_axis.
template <typename R>
void launch_n1(int N1, bool inv, int N0, N1Args<R> a, int nitems, hipStream_t s, hipEvent_t ev0 = nullptr,
               hipEvent_t ev1 = nullptr);
// N0 pass in the block layout (k_n0) in one of its modes; returns the
// partial sums of r.r of an item.
template <typename R, typename RO>
Parts launch_n0(int N0, int mode, int sym, N0Args<R, RO> a, int nitems, hipStream_t s, hipEvent_t ev0 = nullptr,
              hipEvent_t ev1 = nullptr);
// How the N0 pass splits an item for a tile (0: its own choice): columns and
// threads per line of a workgroup, columns per thread, order, partial sums.
struct N0Tile {
  int B, T, cpt, kymajor;
  Parts parts;
};
template <typename R> N0Tile n0_tile(int N0, int N1, int M, int tile, int nc);
// most partial sums per item that launch_n0 writes, for any tile
inline long n0_max_parts(int N1, int M) { return 3L * ((long)M * N1 + N1 / 2 + 1); }
// Whether a grid's planes fit k_plane in double precision (which a mixed plan's
// scalar problems and wide iterations take too).
bool plane_fits(int n0, int n1);
// Planes of k_plane per workgroup: one, or several small ones where that
// leaves 512 workgroups.
int planes_per_group(int n0, int n1, int M, int nc, int nitems);
// N1 and N0 passes in one (k_plane), mode and symbol as launch_n0; a: q, z, s,
// tables, scalars and partial sums.  Returns the partial sums of an item.
template <typename R, typename RO>
Parts launch_plane(int mode, int sym, PlaneArgs<R, RO> a, int nc, int nitems, hipStream_t s, hipEvent_t ev0 = nullptr,
                   hipEvent_t ev1 = nullptr);
// Passes of the residual and of fg_project_grad on 9-component fields (fg_rows.hpp):
// the forward N1 pass with the rows merged (tile as for launch_axis), the N0
// pass in one of its modes (returns the partial sums of r.r of an item), and
// the inverse N1 pass of the plane layout.
void launch_rows_n1(int N1, int N0, double* y, double* dc, int M, int tile, const SpecTables<double>& tb,
                    const Gate& gate, int nitems, hipStream_t s);
template <typename RO, typename Z>
Parts launch_rows_n0(int N0, int mode, RowsN0Args<RO, Z> a, int nitems, hipStream_t s);
template <typename RO>
void launch_rows_out(int n1, long nlines, const double* z, RO* out, const SpecTables<double>& tb, const Gate& gate,
                     int nitems, hipStream_t s);
// Inverse N2 pass fused with the direction and solution updates (k_c2r_dir).
template <typename R>
void launch_c2r_dir(int M, const DirArgs<R>& a, int nitems, hipStream_t s, hipEvent_t ev0 = nullptr,
                    hipEvent_t ev1 = nullptr);

// Whether the open system of a mixed plan keeps the divergence of an iteration and
// its spectrum in double precision.
bool divergence_wide(const double h[3]);
// Lines per workgroup of k_cg_lines for a plan (0: the grid takes the passes).
int lines_per_group(int n0, int n1, int M, int nitems);
// The inverse N2 pass, the operator and the N2 pass of a CG iteration in one
// (k_cg_lines); returns the partial sums of p.Kp of an item.
template <typename R>
int launch_cg_lines(int law, int M, LinesArgs<R> a, int nitems, hipStream_t s, hipEvent_t ev0 = nullptr,
                    hipEvent_t ev1 = nullptr);

template <typename R>
void launch_r2c(int M, const R* in, R* out, long nlines, const SpecTables<R>& tb, const Skip& skip,
                hipStream_t s);
template <typename R>
void launch_c2r(int M, const R* in, R* out, long nlines, const SpecTables<R>& tb, double scale, const Skip& skip,
                hipStream_t s);
// tile: columns per workgroup (0: column_tile).
template <typename R>
void launch_axis(int L, bool inv, R* data, long estride, long ystride, long zstride, int M, int gy, int gz,
                 const cplx<R>* tw, const Skip& skip, hipStream_t s, int tile = 0, hipEvent_t ev0 = nullptr,
                 hipEvent_t ev1 = nullptr);
// N0 pass fused with the projection, for nitems 9-component fields (3 rows
// each).
template <typename R>
void launch_zproj(int N0, R* data, int N1, int M, const SpecTables<R>& tb, R scale, const Skip& skip,
                  hipStream_t s, int nitems = 1, int tile = 0);
// Flag on a projection-pass tile: workgroups ordered ky fastest.
constexpr int kTileKyMajor = 1 << 16;
// Flag on an N1-pass tile in single precision: two adjacent columns per
// thread (one 16-byte access; measured slower at 256^3, kept for the tuner).
constexpr int kTileColumnPairs = 1 << 17;
// Tile widths a pass accepts: powers of two dividing M with T tile <= 256
// threads and an L x tile exchange buffer (plus the pass's tables) within
// 64 KiB.  zproj: the fused N0 projection pass (L = N0), else the N1 pass.
bool tile_valid(bool zproj, int L, int M, int elem_bytes, int tile);
// q = A p of the phase-field (op = 0: coef = a) or Fick (op = 1: coef = w, A6)
// operator, or q = p (op = 2), with its N2 transform (k_scalar_op); returns the number of partial
// sums of p.q.
int launch_scalar_op(int op, int M, const double* p, const double* coef, const double* A6, double kdiff, const Grid3& g,
                     double* spec, double* partials, const Gate& gate, const SpecTables<double>& tb, int planes,
                     hipStream_t s);

}  // namespace fg
