// FFT pass launchers, double precision.
#include "fg_fft_impl.hpp"
namespace fg {
FG_INSTANTIATE_LAUNCHERS(double)
// CG start of the mixed form: double-precision pass, single-precision results
template Parts launch_n0<double, float>(int, int, int, N0Args<double, float>, int, hipStream_t, hipEvent_t, hipEvent_t);
template Parts launch_plane<double, float>(int, int, PlaneArgs<double, float>, int, int, hipStream_t, hipEvent_t,
                                           hipEvent_t);
}
