// The Jacobi marching kernel under the limiter: n = 2..kJacMaxFuse forward
// steps in one launch, every new value clamped. One launch per step moved
// the state twice for each; at 4096^2 f64 a single step takes 48.6 us, a
// launch of 2, 3, 4 and 6 steps 60, 62, 67 and 77 us (the clamp about doubles a
// point's vector instructions). Call of 100 steps with ten snapshots, with the
// store-through runs: 18.16 -> 13.2 ms.

#include <hip/hip_runtime.h>

#include "adst.h"
#include "jacobi_march.h"
#include "kernels.h"

namespace adst {
namespace {

template <class R, int K>
hipError_t lim_launch(const StepShape& s, const R* x, R* y, hipStream_t st) {
  using G = Geom<R, K>;
  MarchGrid g;
  int64_t blocks;
  if (!make_grid_fit(s.nx, s.ny, G::OW, &g, &blocks, kRows, kJacShort<R>)) return hipErrorInvalidValue;
  const MarchExtra<R, K, true, false> ex{{R(s.lo), R(s.hi)}, {nullptr}};
  const dim3 grid((unsigned)blocks), block(kLanes);
  if (rows_aligned<R>(s.nx, x, y))
    jacobi_march<R, K, false, true, true><<<grid, block, 0, st>>>(x, y, s.nx, s.ny, g, R(s.p0), ex);
  else
    jacobi_march<R, K, false, false, true><<<grid, block, 0, st>>>(x, y, s.nx, s.ny, g, R(s.p0),
                                                                   ex);
  return hipGetLastError();
}

template <class R>
hipError_t lim_n(const StepShape& s, const void* xv, void* yv, int n, hipStream_t st) {
  const R* x = static_cast<const R*>(xv);
  R* y = static_cast<R*>(yv);
  switch (n) {
    case 2: return lim_launch<R, 2>(s, x, y, st);
    case 3: return lim_launch<R, 3>(s, x, y, st);
    case 4: return lim_launch<R, 4>(s, x, y, st);
    case 5: return lim_launch<R, 5>(s, x, y, st);
    case 6: return lim_launch<R, 6>(s, x, y, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_jacobi_march_lim(const StepShape& s, const void* x, void* y, int32_t n,
                                   hipStream_t stream) {
  if (s.kind != ADST_JACOBI2D5 || !s.limit) return hipErrorInvalidValue;
  return s.dtype == ADST_F64 ? lim_n<double>(s, x, y, n, stream)
                             : lim_n<float>(s, x, y, n, stream);
}

}  // namespace adst
