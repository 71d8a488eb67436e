// FFT pass launchers, double precision.
#include "fg_fft_impl.hpp"
namespace fg {
FG_INSTANTIATE_LAUNCHERS(double)
// mixed form with its divergence in double precision
template int launch_cg_op<float, double>(int, double*, double*, const float*, long, const KrylovScalars*, const float*,
                                         double*, const Gate&, int, int, int, const double*, int, hipStream_t,
                                         hipEvent_t, hipEvent_t);
template Parts launch_n0<double, float>(int, int, int, N0Args<double, float>, int, hipStream_t, hipEvent_t, hipEvent_t);
template Parts launch_plane<double, float>(int, int, PlaneArgs<double, float>, int, int, hipStream_t, hipEvent_t,
                                           hipEvent_t);
}
