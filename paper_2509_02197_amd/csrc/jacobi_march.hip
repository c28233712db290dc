// Temporal blocking of the Jacobi kind on gfx950: n = 3..kJacMaxFuse steps,
// forward or gather adjoint, in one launch with the intermediate time levels
// in registers.
//
// The step (adst.h, ADST_JACOBI2D5): interior points take
//     x'[c] = w * ((((x[c] + x[W]) + x[E]) + x[S]) + x[N]),
// the ring is copied; the adjoint is its transpose in gather form,
//     interior m: g'[m] = w * (g[m] + (((gi[W] + gi[E]) + gi[S]) + gi[N]))
//     ring m:     g'[m] = g[m] + w * (((gi[W] + gi[E]) + gi[S]) + gi[N])
// with gi = g on interior points and 0 on the ring (and outside the grid).
// A point two or more cells from the edge sees only interior neighbours, so
// there both take their unmasked form. The step is linear in the carried
// state, so its adjoint reads no forward state (Sec. IV) and n steps of
// either compose without any stored value in between.
//
// Layout. A workgroup is one wave of 64 lanes owning a strip of 64 * V
// columns (V elements, 16 bytes, per lane) and a chunk of rows. It marches
// along the rows carrying the last three rows of each of the n time levels:
// when input row q arrives, level k evaluates row q - k from level k - 1's
// rows q - k - 1, q - k, q - k + 1. East/west neighbours of a lane's first
// and last element come from the adjacent lanes by DPP whole-wave shifts.
// Each level is valid on one column fewer at each side of the strip and one
// row fewer at each end of the chunk, so strips overlap by H >= n columns
// (whole vectors) and a chunk reads n rows beyond each of its ends. Every
// point evaluates the single-step expressions above, so any split of the
// steps into launches gives the same bits.
//
// Memory. Each input row is loaded kAhead rows before it enters the
// pipeline, into registers that nothing touches until then (its validity
// mask is applied on entry), so the loads stay in flight behind the
// arithmetic. Rows beyond the ones a chunk needs are never fetched from new
// addresses. Odd chunks march downward, so the rows two neighbouring chunks
// share are read by both at about the same time and the second read can hit
// the L2 cache they share (their blocks go to the same XCD); measured, this
// cut the fetched bytes from 1.46x to 1.24x the state's size.
//
// Boundary. Blocks of kUnroll consecutive input rows whose evaluated rows all
// lie two or more cells from the top and bottom edge, in a strip two or more
// cells from the side edges, take the unmasked forms; the others evaluate the
// ring logic. A strip's first and last chunk are short, so the slower blocks
// near the top and bottom edge do not make their waves the launch's tail;
// the first and last strip (the side edges) take short chunks throughout,
// and every XCD gets an equal share of them.
//
// The same layout carries the limiter's one-step adjoint (jacobi_lim_adjoint
// below), which masks g by the branch outcome and transposes it in one pass.

#include <hip/hip_runtime.h>

#include <type_traits>

#include "adst.h"
#include "jacobi_march.h"
#include "kernels.h"

namespace adst {
namespace {

template <class R, int K, bool ADJ>
hipError_t march_launch(const StepShape& s, const R* x, R* y, hipStream_t st) {
  using G = Geom<R, K>;
  if (ADJ && s.nx <= G::V) return hipErrorInvalidValue;  // a lane would hold both ring columns
  MarchGrid g;
  int64_t blocks;
  if (!make_grid_fit(s.nx, s.ny, G::OW, &g, &blocks, kRows, kJacShort<R>)) return hipErrorInvalidValue;
  if (rows_aligned<R>(s.nx, x, y))
    jacobi_march<R, K, ADJ, true><<<dim3((unsigned)blocks), dim3(kLanes), 0, st>>>(
        x, y, s.nx, s.ny, g, R(s.p0), {});
  else
    jacobi_march<R, K, ADJ, false><<<dim3((unsigned)blocks), dim3(kLanes), 0, st>>>(
        x, y, s.nx, s.ny, g, R(s.p0), {});
  return hipGetLastError();
}

// ------------------------------------------- the limiter's adjoint, fused
// One Jacobi adjoint step under the limiter: g_t is masked by the branch
// each point took at step t (its unlimited value re-evaluated from x_{t-1}
// with the forward's expression; 0 where it left [lo, hi]) and the masked g
// is transposed with the single-step adjoint's expressions, in one pass
// that reads x and g once and writes g' once. A wave marches down a strip
// carrying three rows of x, the g rows waiting for their mask and three
// masked g rows: when input row p arrives, row p-1 is masked (its x
// neighbourhood is complete) and row p-2 transposed. The mask reads x one
// column beyond the masked g, so strips overlap by V >= 2 columns.
// DP (instead of the mask): g passes unmasked and the pass adds this step's
// share of dL/dw, sum over interior points of g[c] * ((((x[c]+x[W])+x[E])
// +x[S])+x[N]) (the forward's sum, in double), over the work item's output
// points; a wave butterfly then adds it into the item's slot
// (dp_part[item], or overwrites it on the step t = T).
template <class R, bool VEC, bool DP, bool NT>
__global__ __launch_bounds__(kLanes) void jacobi_lim_adjoint(const R* __restrict__ x,
                                                             const R* __restrict__ g,
                                                             R* __restrict__ gp, int nx, int ny,
                                                             MarchGrid grid, R w, R lo, R hi,
                                                             double* dp_part, int dp_first) {
  // six rows of each array in flight: the pass is lighter than the n-step
  // march and registers allow it
  constexpr int V = 16 / sizeof(R), H = V, OW = kLanes * V - 2 * H, P = 6, U = kUnroll;
  static_assert(H >= 2, "the mask reaches two columns beyond an output");
  static_assert(U % P == 0, "register slots must stay static");
  int strip, chunk, r0, r1, item;
  if (!march_item(grid, ny, &strip, &chunk, &r0, &r1, &item)) return;
  const int lane = threadIdx.x;
  const int s0 = strip * OW;
  const int c0 = s0 - H + lane * V;
  const int nit = (r1 - r0) + 4;  // input rows r0-2 .. r1+1
  double a0 = 0.0;
  const int lo_need = max(r0 - 2, 0), hi_need = min(r1 + 1, ny - 1);
  auto cin = [&](int c) { return c >= 1 && c <= nx - 2; };
  bool cok[V], cI[V], cW[V], cE[V];
#pragma unroll
  for (int e = 0; e < V; ++e) {
    const int c = c0 + e;
    cok[e] = c >= 0 && c < nx;
    cI[e] = cin(c);
    cW[e] = cin(c - 1);
    cE[e] = cin(c + 1);
  }
  const bool strip_in = s0 - H >= 2 && s0 - H + kLanes * V <= nx - 2;
  const bool st_lane = lane * V >= H && lane * V < H + OW;
  // x and g are read once per step, with the non-temporal hint (NT: 4096^2
  // f64: 90.5 -> 83.5 us per step; the hint on x alone did nothing)
  auto load = [&](const R* a, int row, R* out, auto inner_t) {
    const int rr = min(max(row, lo_need), hi_need);
    load_block<R, VEC, decltype(inner_t)::value, NT>(a + (int64_t)rr * nx, c0, nx, out);
  };
  enum { kFast = 0, kGeneral = 2 };
  auto march = [&](auto dir_t, auto mid_t) {
    constexpr int DIR = decltype(dir_t)::value;
    const int ifirst = DIR > 0 ? r0 - 2 : r1 + 1;  // row of input index 0
    // slot p mod 3 holds pipeline index p (row ifirst + DIR*p)
    R xw[3][V], gr[3][V], mg[3][V];
    R px[P][V], pg[P][V];
    constexpr auto inner = std::bool_constant<decltype(mid_t)::value == kFast>{};
#pragma unroll
    for (int s3 = 0; s3 < 3; ++s3)
#pragma unroll
      for (int e = 0; e < V; ++e) xw[s3][e] = gr[s3][e] = mg[s3][e] = R(0);
#pragma unroll
    for (int u = 0; u < P; ++u) {
      load(x, ifirst + DIR * u, px[u], inner);
      load(g, ifirst + DIR * u, pg[u], inner);
    }
    auto block = [&](int base, auto mode_t) {
      constexpr int MODE = decltype(mode_t)::value;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int rr = base + u;
        {  // input row rr enters; the rows P ahead are requested
          const int row = ifirst + DIR * rr;
          const bool rok = row >= 0 && row < ny;
#pragma unroll
          for (int e = 0; e < V; ++e) {
            const bool ok = MODE == kFast || (rok && cok[e]);
            xw[u % 3][e] = ok ? px[u % P][e] : R(0);
            gr[u % 3][e] = ok ? pg[u % P][e] : R(0);
          }
          load(x, row + DIR * P, px[u % P], inner);
          load(g, row + DIR * P, pg[u % P], inner);
        }
        {  // mask row index rr-1 from x rows rr-2 .. rr
          const int m = ifirst + DIR * (rr - 1);
          constexpr int off = 6;
          const int sOld = (u - 2 + off) % 3, sc = (u - 1 + off) % 3, sNew = u % 3;
          const R* a = xw[sc];
          const R* S = xw[DIR > 0 ? sOld : sNew];
          const R* N = xw[DIR > 0 ? sNew : sOld];
          const R wl = from_prev(a[V - 1]), er = from_next(a[0]);
          const bool rm = m >= 1 && m <= ny - 2;
          const bool own = m >= r0 && m < r1 && st_lane;  // this item's output row
#pragma unroll
          for (int e = 0; e < V; ++e) {
            const R Wn = e > 0 ? a[e > 0 ? e - 1 : 0] : wl;
            const R En = e < V - 1 ? a[e < V - 1 ? e + 1 : 0] : er;
            const R sum = (((a[e] + Wn) + En) + S[e]) + N[e];
            if constexpr (DP) {
              mg[sc][e] = gr[sc][e];
              if ((MODE == kFast || (cI[e] && rm)) && own)
                a0 += (double)gr[sc][e] * (double)sum;
            } else {
              const R yv = (MODE == kFast || (cI[e] && rm)) ? w * sum : a[e];
              mg[sc][e] = (yv < lo || yv > hi) ? R(0) : gr[sc][e];
            }
          }
        }
        {  // transpose row index rr-2 from masked rows rr-3 .. rr-1
          const int j = ifirst + DIR * (rr - 2);
          constexpr int off = 6;
          const int sOld = (u - 3 + off) % 3, sc = (u - 2 + off) % 3, sNew = (u - 1 + off) % 3;
          const R* a = mg[sc];
          const R* S = mg[DIR > 0 ? sOld : sNew];
          const R* N = mg[DIR > 0 ? sNew : sOld];
          const R wl = from_prev(a[V - 1]), er = from_next(a[0]);
          const bool rj = j >= 1 && j <= ny - 2, rS = j >= 2 && j <= ny - 1,
                     rN = j >= 0 && j <= ny - 3;
          R o[V];
#pragma unroll
          for (int e = 0; e < V; ++e) {
            const R Wn = e > 0 ? a[e > 0 ? e - 1 : 0] : wl;
            const R En = e < V - 1 ? a[e < V - 1 ? e + 1 : 0] : er;
            if constexpr (MODE == kFast) {
              o[e] = w * (a[e] + (((Wn + En) + S[e]) + N[e]));
            } else {
              R sum = (cW[e] && rj) ? Wn : R(0);
              sum += (cE[e] && rj) ? En : R(0);
              sum += (cI[e] && rS) ? S[e] : R(0);
              sum += (cI[e] && rN) ? N[e] : R(0);
              o[e] = (cI[e] && rj) ? w * (a[e] + sum) : a[e] + w * sum;
            }
          }
          if (j >= r0 && j < r1 && st_lane) {
            store_block<R, VEC>(gp + (int64_t)j * nx, c0, nx, o);
          }
        }
      }
    };
    // A block of U input rows touches rows ifirst + DIR*[base - 4, base + U - 1];
    // blocks [fa, fb) have all of them in [2, ny - 3].
    constexpr int R4 = 4;
    int fa, fb;
    if (DIR > 0) {
      fa = 2 + R4 - ifirst;
      fb = ny - 1 - ifirst - U;
    } else {
      fa = ifirst + R4 - (ny - 3);
      fb = ifirst - U;
    }
    fa = ((max(fa, 0) + U - 1) / U) * U;
    using General = std::integral_constant<int, kGeneral>;
    int base = 0;
    for (; base < nit && base < fa; base += U) block(base, General{});
    for (; base < nit && base < fb; base += U) block(base, mid_t);
    for (; base < nit; base += U) block(base, General{});
  };
  using Up = std::integral_constant<int, 1>;
  using Down = std::integral_constant<int, -1>;
  using Fast = std::integral_constant<int, kFast>;
  using General = std::integral_constant<int, kGeneral>;
  if (strip_in) {
    if (chunk & 1)
      march(Down{}, Fast{});
    else
      march(Up{}, Fast{});
  } else {
    if (chunk & 1)
      march(Down{}, General{});
    else
      march(Up{}, General{});
  }
  if constexpr (DP) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) a0 += __shfl_xor(a0, off, kLanes);
    if (lane == 0) dp_part[item] = dp_first ? a0 : dp_part[item] + a0;
  }
}

// One pass reading x and g: the limiter's masked adjoint (dp_part null) or
// the adjoint with dL/dw's share (dp_part: jacobi_x_adjoint_slots doubles).
template <class R>
hipError_t lim_adjoint_launch(const StepShape& s, const R* x, const R* g, R* gp,
                              double* dp_part, bool dp_first, hipStream_t st) {
  constexpr int V = 16 / sizeof(R), OW = kLanes * V - 2 * V;
  MarchGrid grid;
  int64_t blocks;
  // the slots of dL/dw belong to chunks of kLimRows
  if (!(dp_part ? make_grid(s.nx, s.ny, OW, &grid, &blocks, kLimRows)
                : make_grid_fit(s.nx, s.ny, OW, &grid, &blocks, kLimRows, kJacShort<R>)))
    return hipErrorInvalidValue;
  const bool vec = rows_aligned<R>(s.nx, x, g) && rows_aligned<R>(s.nx, gp, nullptr);
  const dim3 gr((unsigned)blocks), bl(kLanes);
  const R w = R(s.p0), lo = R(s.lo), hi = R(s.hi);
  const int first = dp_first ? 1 : 0;
  // Rows off the 16-byte grid share their lines between waves and rows: where
  // two states fit the Infinity Cache, a line read without the hint is still
  // there for the other reader (steps with dL/dw, calls of 24 steps, us, with and
  // without: f64 1501 x 2003 1115 and 985, 3001 x 3003 1981 and 1950, 5001 x 5003
  // 4903 and 5477; under the limiter too f32 3001 x 3003 1981 and 1836).
  const bool nt = vec || int64_t(s.nx) * s.ny * int64_t(sizeof(R)) >= kStreamBytes / 2;
#define ADST_LIM_ADJ(VECV, DPV, NTV)                                                     \
  jacobi_lim_adjoint<R, VECV, DPV, NTV><<<gr, bl, 0, st>>>(x, g, gp, s.nx, s.ny, grid, w, \
                                                           lo, hi, dp_part, first)
  if (dp_part && vec)
    ADST_LIM_ADJ(true, true, true);
  else if (dp_part && nt)
    ADST_LIM_ADJ(false, true, true);
  else if (dp_part)
    ADST_LIM_ADJ(false, true, false);
  else if (vec)
    ADST_LIM_ADJ(true, false, true);
  else if (nt)
    ADST_LIM_ADJ(false, false, true);
  else
    ADST_LIM_ADJ(false, false, false);
#undef ADST_LIM_ADJ
  return hipGetLastError();
}

template <class R, bool ADJ>
hipError_t march_n(const StepShape& s, const void* xv, void* yv, int n, hipStream_t st) {
  const R* x = static_cast<const R*>(xv);
  R* y = static_cast<R*>(yv);
  switch (n) {
    case 3: return march_launch<R, 3, ADJ>(s, x, y, st);
    case 4: return march_launch<R, 4, ADJ>(s, x, y, st);
    case 5: return march_launch<R, 5, ADJ>(s, x, y, st);
    case 6: return march_launch<R, 6, ADJ>(s, x, y, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_jacobi_lim_adjoint(const StepShape& s, const void* x, const void* g, void* gp,
                                     hipStream_t stream) {
  if (s.kind != ADST_JACOBI2D5 || !s.limit || !x) return hipErrorInvalidValue;
  if (s.dtype == ADST_F64)
    return lim_adjoint_launch<double>(s, static_cast<const double*>(x),
                                      static_cast<const double*>(g), static_cast<double*>(gp),
                                      nullptr, false, stream);
  return lim_adjoint_launch<float>(s, static_cast<const float*>(x), static_cast<const float*>(g),
                                   static_cast<float*>(gp), nullptr, false, stream);
}

hipError_t launch_jacobi_dp_adjoint(const StepShape& s, const void* x, const void* g, void* gp,
                                    double* dp_part, bool dp_first, hipStream_t stream) {
  if (s.kind != ADST_JACOBI2D5 || !x || !dp_part) return hipErrorInvalidValue;
  if (s.dtype == ADST_F64)
    return lim_adjoint_launch<double>(s, static_cast<const double*>(x),
                                      static_cast<const double*>(g), static_cast<double*>(gp),
                                      dp_part, dp_first, stream);
  return lim_adjoint_launch<float>(s, static_cast<const float*>(x), static_cast<const float*>(g),
                                   static_cast<float*>(gp), dp_part, dp_first, stream);
}

int64_t jacobi_x_adjoint_slots(const StepShape& s) {
  const int V = s.dtype == ADST_F64 ? 2 : 4, OW = kLanes * V - 2 * V;  // as lim_adjoint_launch
  MarchGrid g;
  int64_t blocks;
  if (!make_grid(s.nx, s.ny, OW, &g, &blocks, kLimRows)) return 0;
  return int64_t(g.nedge) * g.ce + int64_t(g.ns - g.nedge) * g.ci;
}

hipError_t launch_jacobi_march(const StepShape& s, const void* x, void* y, int32_t n, bool adjoint,
                               hipStream_t stream) {
  if (s.kind != ADST_JACOBI2D5 || n < 3 || n > kJacMaxFuse) return hipErrorInvalidValue;
  if (s.dtype == ADST_F64)
    return adjoint ? march_n<double, true>(s, x, y, n, stream)
                   : march_n<double, false>(s, x, y, n, stream);
  return adjoint ? march_n<float, true>(s, x, y, n, stream)
                 : march_n<float, false>(s, x, y, n, stream);
}

}  // namespace adst
