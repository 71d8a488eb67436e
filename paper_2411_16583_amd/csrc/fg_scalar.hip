// Launcher of the scalar operators (phase field, Fick) fused with their N2
// transform.
#include <stdexcept>

#include "fg_fft_sizes.hpp"
#include "fg_scalar_op.hpp"

namespace fg {

int launch_scalar_op(int op, int M, const double* p, const double* coef, const double* A6, double kdiff, const Grid3& g,
                     double* spec, double* partials, const Gate& gate, const SpecTables<double>& tb, int planes,
                     hipStream_t s) {
  const long nlines = (long)g.n0 * g.n1;
  switch (M) {
#define FG_SCALAR_GO(L_, OP_)                                                                                  \
  hipLaunchKernelGGL((k_scalar_op<L_, OP_>), dim3(blocks), dim3(kScalarThreads), 0, s, p, coef, A6, kdiff, g,   \
                     reinterpret_cast<double2*>(spec), partials, tb, gate, planes)
#define FG_CASE(L_)                                                                       \
  case L_: {                                                                              \
    const int blocks = (int)((nlines + scalar_lines<L_>() - 1) / scalar_lines<L_>());     \
    if (op == 0)                                                                          \
      FG_SCALAR_GO(L_, 0);                                                                \
    else if (op == 1)                                                                     \
      FG_SCALAR_GO(L_, 1);                                                                \
    else                                                                                  \
      FG_SCALAR_GO(L_, 2);                                                                \
    return blocks;                                                                        \
  }
    FG_FOR_M(FG_CASE)
#undef FG_CASE
#undef FG_SCALAR_GO
  }
  throw std::invalid_argument("unsupported N2/2");
}

}  // namespace fg
