// Projector scatter of the nonlocal (KB) and Hubbard terms:
//
//   Y[s](x) += alpha * sum_j phi_j(x) Q[j][s]
//
// (Sec. II.A potential section: V_U psi = sum phi_m' U/2 (delta - 2D) <phi_m|psi>;
// Sec. II.B: implemented like the nonlocal projectors).  Each point owns its
// output (no atomics, deterministic).
//
// The grid is cut into bricks of 64 points; each stores the dense tile Phi_b
// over the functions touching it.  The update of a brick for 64 states is a
// small GEMM on the matrix cores (bricks.hip), so every table value is read
// once per 64 states.
#include "common.h"

namespace hcu {

template <typename T>
void launch_nl_scatter(const Ctx& c, int ik, T* Y, int64_t ld, int ncol, const T* Qt, double alpha,
                       hipStream_t st) {
  if (c.nproj == 0) return;
  launch_brick_pass<T>(c, (const T*)c.d_bval[ik], nullptr, Y, ld, ncol, Qt, alpha, true, false, st);
}

template void launch_nl_scatter<double>(const Ctx&, int, double*, int64_t, int, const double*, double, hipStream_t);
template void launch_nl_scatter<float>(const Ctx&, int, float*, int64_t, int, const float*, double, hipStream_t);
template void launch_nl_scatter<cplx<double>>(const Ctx&, int, cplx<double>*, int64_t, int, const cplx<double>*,
                                              double, hipStream_t);
template void launch_nl_scatter<cplx<float>>(const Ctx&, int, cplx<float>*, int64_t, int, const cplx<float>*,
                                             double, hipStream_t);

}  // namespace hcu
