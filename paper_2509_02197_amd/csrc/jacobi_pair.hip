// Two Jacobi adjoint steps that read state, t and t-1, in one launch: under
// the limiter (each step's gradient masked by the branch its points took) or
// with dL/dw's shares. It reads g_t, x_{t-1} and x_{t-2} once and writes
// g_{t-2}: 4 values a point instead of the 6 of two launches of
// jacobi_lim_adjoint (jacobi_march.hip), whose layout, expressions and order
// it keeps, so any split into launches gives the same bits. At 4096^2 f64 a
// launch takes 115 us (4.7 TB/s) against 80 for one step, and the limited call
// of 100 steps with ten snapshots 13.25 -> 11.4 ms.
//
// When input row p arrives (x_{t-2}'s a row later), row p-1 is masked by
// x_{t-1}, row p-2 transposed into g_{t-1} and masked by x_{t-2}, row p-3
// transposed into g_{t-2}. Strips overlap by four columns a side (three are
// lost). In f32 that is the single step's overlap, so its work items and
// their partial sums of dL/dw are the single step's too; in f64 they are not,
// and dL/dw keeps one launch per step there.

#include <hip/hip_runtime.h>

#include <type_traits>

#include "adst.h"
#include "jacobi_march.h"
#include "kernels.h"

namespace adst {
namespace {

constexpr int kPairH = 4;
constexpr int kPairAhead = 3;  // six rows ahead: no faster in f64, 13% slower in f32
constexpr int kPairRows = 192;  // 128: 119.5 against 114.6 us at 4096^2 f64, 64: 121.7

template <class R, bool VEC, bool DP, bool NT>
__global__ __launch_bounds__(kLanes) void jacobi_pair_adjoint(
    const R* __restrict__ x1, const R* __restrict__ x2, const R* __restrict__ g,
    R* __restrict__ gp, int nx, int ny, MarchGrid grid, R w, R lo, R hi, double* dp_part,
    int dp_first) {
  constexpr int V = 16 / (int)sizeof(R), H = kPairH, OW = kLanes * V - 2 * H, P = kPairAhead,
                U = kUnroll;
  static_assert(H % V == 0 && U % P == 0, "whole blocks; register slots stay static");
  int strip, chunk, r0, r1, item;
  // with dL/dw the chunks are make_grid's: as a value read from grid their edge
  // rows cost the 2501 x 3003 f32 call 5% (2.92 -> 3.07 ms)
  if (!march_item<!DP>(grid, ny, &strip, &chunk, &r0, &r1, &item)) return;
  const int lane = threadIdx.x;
  const int s0 = strip * OW;
  const int c0 = s0 - H + lane * V;
  const int nit = (r1 - r0) + 6;  // input rows r0-3 .. r1+2
  double a0 = 0.0, a1 = 0.0;
  const int lo_need = max(r0 - 3, 0), hi_need = min(r1 + 2, ny - 1);
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
  enum { kFast = 0, kGeneral = 2 };
  auto march = [&](auto dir_t, auto mid_t) {
    constexpr int DIR = decltype(dir_t)::value;
    constexpr bool INNER = decltype(mid_t)::value == kFast;
    const int ifirst = DIR > 0 ? r0 - 3 : r1 + 2;  // row of input index 0
    auto load = [&](const R* a, int row, R* out) {
      const int rr = min(max(row, lo_need), hi_need);
      load_block<R, VEC, INNER, NT>(a + (int64_t)rr * nx, c0, nx, out);
    };
    // slot p mod 3 holds pipeline index p (row ifirst + DIR*p); xw2's is of
    // the index its row enters at, one later
    R xw[3][V], xw2[3][V], gr[3][V], mg[3][V], mg2[3][V];
    R px[P][V], px2[P][V], pg[P][V];
#pragma unroll
    for (int s3 = 0; s3 < 3; ++s3)
#pragma unroll
      for (int e = 0; e < V; ++e)
        xw[s3][e] = xw2[s3][e] = gr[s3][e] = mg[s3][e] = mg2[s3][e] = R(0);
#pragma unroll
    for (int u = 0; u < P; ++u) {
      load(x1, ifirst + DIR * u, px[u]);
      load(g, ifirst + DIR * u, pg[u]);
      load(x2, ifirst + DIR * (u - 1), px2[u]);
    }
    auto block = [&](int base, auto mode_t) {
      constexpr int MODE = decltype(mode_t)::value;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int rr = base + u;
        constexpr int off = 12;
        {  // input row rr enters; the rows P ahead are requested
          const int row = ifirst + DIR * rr, row2 = row - DIR;
          const bool rok = row >= 0 && row < ny, rok2 = row2 >= 0 && row2 < ny;
#pragma unroll
          for (int e = 0; e < V; ++e) {
            const bool ok = MODE == kFast || (rok && cok[e]);
            const bool ok2 = MODE == kFast || (rok2 && cok[e]);
            xw[u % 3][e] = ok ? px[u % P][e] : R(0);
            gr[u % 3][e] = ok ? pg[u % P][e] : R(0);
            xw2[u % 3][e] = ok2 ? px2[u % P][e] : R(0);
          }
          load(x1, row + DIR * P, px[u % P]);
          load(g, row + DIR * P, pg[u % P]);
          load(x2, row2 + DIR * P, px2[u % P]);
        }
        // The gradient `in` of the step that reads x's rows (slots sO, sC, sN)
        // at row m: masked by the branch taken, or unmasked with its share of
        // dL/dw added to acc.
        auto mask = [&](const R(&xr)[3][V], int sOld, int sc, int sNew, int m, const R* in, R* out,
                        double& acc) {
          const R* a = xr[sc];
          const R* S = xr[DIR > 0 ? sOld : sNew];
          const R* N = xr[DIR > 0 ? sNew : sOld];
          const R wl = from_prev(a[V - 1]), er = from_next(a[0]);
          const bool rm = m >= 1 && m <= ny - 2;
          const bool own = m >= r0 && m < r1 && st_lane;  // this item's output row
#pragma unroll
          for (int e = 0; e < V; ++e) {
            const R Wn = e > 0 ? a[e > 0 ? e - 1 : 0] : wl;
            const R En = e < V - 1 ? a[e < V - 1 ? e + 1 : 0] : er;
            const R sum = (((a[e] + Wn) + En) + S[e]) + N[e];
            if constexpr (DP) {
              out[e] = in[e];
              if ((MODE == kFast || (cI[e] && rm)) && own) acc += (double)in[e] * (double)sum;
            } else {
              const R yv = (MODE == kFast || (cI[e] && rm)) ? w * sum : a[e];
              out[e] = (yv < lo || yv > hi) ? R(0) : in[e];
            }
          }
        };
        // row j of the transposed step from the masked rows in m's slots
        auto transpose = [&](const R(&m)[3][V], int sOld, int sc, int sNew, int j, R* o) {
          const R* a = m[sc];
          const R* S = m[DIR > 0 ? sOld : sNew];
          const R* N = m[DIR > 0 ? sNew : sOld];
          const R wl = from_prev(a[V - 1]), er = from_next(a[0]);
          const bool rj = j >= 1 && j <= ny - 2, rS = j >= 2 && j <= ny - 1,
                     rN = j >= 0 && j <= ny - 3;
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
        };
        // slots of the indices rr-4 .. rr
        const int p4 = (u - 4 + off) % 3, p3 = (u - 3 + off) % 3, p2 = (u - 2 + off) % 3,
                  p1 = (u - 1 + off) % 3, p0 = u % 3;
        mask(xw, p2, p1, p0, ifirst + DIR * (rr - 1), gr[p1], mg[p1], a0);
        R g1[V];  // g_{t-1} of row index rr-2
        transpose(mg, p3, p2, p1, ifirst + DIR * (rr - 2), g1);
        // x_{t-2}'s rows rr-3, rr-2, rr-1 entered at rr-2, rr-1, rr
        mask(xw2, p2, p1, p0, ifirst + DIR * (rr - 2), g1, mg2[p2], a1);
        const int j = ifirst + DIR * (rr - 3);
        R o[V];
        transpose(mg2, p4, p3, p2, j, o);
        if (j >= r0 && j < r1 && st_lane) store_block<R, VEC>(gp + (int64_t)j * nx, c0, nx, o);
      }
    };
    // A block of U input rows touches rows ifirst + DIR*[base - 6, base + U - 1];
    // blocks [fa, fb) have all of them in [2, ny - 3].
    constexpr int R6 = 6;
    int fa, fb;
    if (DIR > 0) {
      fa = 2 + R6 - ifirst;
      fb = ny - 1 - ifirst - U;
    } else {
      fa = ifirst + R6 - (ny - 3);
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
    for (int o = 32; o > 0; o >>= 1) {
      a0 += __shfl_xor(a0, o, kLanes);
      a1 += __shfl_xor(a1, o, kLanes);
    }
    if (lane == 0) dp_part[item] = (dp_first ? a0 : dp_part[item] + a0) + a1;
  }
}

template <class R>
hipError_t pair_launch(const StepShape& s, const R* x1, const R* x2, const R* g, R* gp,
                       double* dp_part, bool dp_first, hipStream_t st) {
  constexpr int V = 16 / (int)sizeof(R), OW = kLanes * V - 2 * kPairH;
  MarchGrid grid;
  int64_t blocks;
  // the slots of dL/dw belong to chunks of kLimRows
  if (!(dp_part ? make_grid(s.nx, s.ny, OW, &grid, &blocks, kLimRows)
                : make_grid_fit(s.nx, s.ny, OW, &grid, &blocks, kPairRows, kJacShort<R>)))
    return hipErrorInvalidValue;
  const bool vec = rows_aligned<R>(s.nx, x1, x2) && rows_aligned<R>(s.nx, g, gp);
  const dim3 gr((unsigned)blocks), bl(kLanes);
  const R w = R(s.p0), lo = R(s.lo), hi = R(s.hi);
  const int first = dp_first ? 1 : 0;
  // the hint as for the single step (lim_adjoint_launch), with four states
  // (limited calls of 24 steps, us, with and without: f64 2049 x 2049 764 and 722,
  // 3001 x 3003 1472 and 1521; f32 3001 x 3003 869 and 836, 5001 x 5003 2101 and
  // 2253)
  const bool nt = vec || int64_t(s.nx) * s.ny * int64_t(sizeof(R)) >= kStreamBytes / 4;
#define ADST_PAIR(VECV, DPV, NTV)                                                              \
  jacobi_pair_adjoint<R, VECV, DPV, NTV><<<gr, bl, 0, st>>>(x1, x2, g, gp, s.nx, s.ny, grid, w, \
                                                            lo, hi, dp_part, first)
  if (dp_part) {
    if constexpr (V == kPairH) {  // the single step's work items
      if (vec)
        ADST_PAIR(true, true, true);
      else if (nt)
        ADST_PAIR(false, true, true);
      else
        ADST_PAIR(false, true, false);
    } else {
      return hipErrorInvalidValue;
    }
  } else if (vec) {
    ADST_PAIR(true, false, true);
  } else if (nt) {
    ADST_PAIR(false, false, true);
  } else {
    ADST_PAIR(false, false, false);
  }
#undef ADST_PAIR
  return hipGetLastError();
}

}  // namespace

// Times of 20 adjoint steps as pairs against single launches: f64 under the
// limiter 0.74 to 0.98 from 8 x 8 to 2500 x 3003, thin grids among them. In
// f32 the pair's general form, which masks columns and rows, takes longer than
// two single steps': under the limiter 1.04 to 1.34 on grids of up to 8 rows
// (all of them near an edge), 0.82 to 0.98 from 16 x 16 on; with dL/dw, whose
// chunks are long, 1.13 to 1.27 where an interior strip reaches the last
// columns or there is none (16 x 16 to 400 x 400, 5000 x 48, 128 x 500), 1.3 on
// grids of one or two rows, 0.85 to 0.89 elsewhere (700 x 700, 48 x 5000, 2500 x
// 3003).
bool jacobi_pairs_adjoint(const StepShape& s, bool dparams) {
  if (s.kind != ADST_JACOBI2D5) return false;
  if (!(dparams ? !s.limit && s.dtype == ADST_F32 : s.limit != 0)) return false;
  if (s.dtype == ADST_F64) return true;
  if (s.ny <= 2 * kEndRows) return false;
  if (!dparams) return true;
  constexpr int V = 16 / (int)sizeof(float), OW = kLanes * V - 2 * kPairH;
  const int last = (s.nx + OW - 1) / OW - 2;  // the last interior strip
  return last >= 1 && int64_t(last) * OW - kPairH + kLanes * V <= s.nx - 2;
}

hipError_t launch_jacobi_pair_adjoint(const StepShape& s, const void* x1, const void* x2,
                                      const void* g, void* gp, double* dp_part, bool dp_first,
                                      hipStream_t stream) {
  if (!jacobi_pairs_adjoint(s, dp_part != nullptr) || !x1 || !x2) return hipErrorInvalidValue;
  if (dp_part && dp_first) {  // the slots of the unused second constant
    const int64_t n = dparam_slots(s);
    const hipError_t e = launch_fill_zero(dp_part + n, n * (int64_t)sizeof(double), stream);
    if (e != hipSuccess) return e;
  }
  if (s.dtype == ADST_F64)
    return pair_launch<double>(s, static_cast<const double*>(x1), static_cast<const double*>(x2),
                               static_cast<const double*>(g), static_cast<double*>(gp), dp_part,
                               dp_first, stream);
  return pair_launch<float>(s, static_cast<const float*>(x1), static_cast<const float*>(x2),
                            static_cast<const float*>(g), static_cast<float*>(gp), dp_part,
                            dp_first, stream);
}

}  // namespace adst
