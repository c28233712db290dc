// The Jacobi marching kernel as a store-through run: n = 2..kJacMaxStore
// forward steps whose every state is kept, in one launch that reads the
// first state once and writes each of the n (8 + 8n bytes a point in f64
// instead of 16n), with or without the limiter.

#include <hip/hip_runtime.h>

#include "adst.h"
#include "jacobi_march.h"
#include "kernels.h"

namespace adst {
namespace {

template <class R, int K, bool LIM>
hipError_t store_launch(const StepShape& s, const R* x, void* const* ys, hipStream_t st) {
  using G = Geom<R, K>;
  MarchGrid g;
  int64_t blocks;
  if (!make_grid_fit(s.nx, s.ny, G::OW, &g, &blocks, kRows, kJacShort<R>)) return hipErrorInvalidValue;
  MarchExtra<R, K, LIM, true> ex{};
  ex.lim = {R(s.lo), R(s.hi)};
  R* y = static_cast<R*>(ys[K - 1]);
  bool vec = rows_aligned<R>(s.nx, x, y);
  for (int k = 0; k < K - 1; ++k) {
    ex.mid[k] = static_cast<R*>(ys[k]);
    vec = vec && rows_aligned<R>(s.nx, ex.mid[k], nullptr);
  }
  const dim3 grid((unsigned)blocks), block(kLanes);
  const R w = R(s.p0);
  if (vec)
    jacobi_march<R, K, false, true, LIM, true, kStoreNT><<<grid, block, 0, st>>>(x, y, s.nx, s.ny,
                                                                                g, w, ex);
  else
    jacobi_march<R, K, false, false, LIM, true, kStoreNT><<<grid, block, 0, st>>>(x, y, s.nx,
                                                                                 s.ny, g, w, ex);
  return hipGetLastError();
}

template <class R, bool LIM>
hipError_t store_n(const StepShape& s, const void* xv, void* const* ys, int n, hipStream_t st) {
  const R* x = static_cast<const R*>(xv);
  switch (n) {
    case 2: return store_launch<R, 2, LIM>(s, x, ys, st);
    case 3: return store_launch<R, 3, LIM>(s, x, ys, st);
    case 4: return store_launch<R, 4, LIM>(s, x, ys, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_jacobi_store(const StepShape& s, const void* x, void* const* ys, int32_t n,
                               hipStream_t stream) {
  if (s.kind != ADST_JACOBI2D5) return hipErrorInvalidValue;
  if (s.dtype == ADST_F64)
    return s.limit ? store_n<double, true>(s, x, ys, n, stream)
                   : store_n<double, false>(s, x, ys, n, stream);
  return s.limit ? store_n<float, true>(s, x, ys, n, stream)
                 : store_n<float, false>(s, x, ys, n, stream);
}

}  // namespace adst
