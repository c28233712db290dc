// Variable-coefficient diffusion on gfx950 as a register march: two forward
// steps in one launch.
//
// The step (adst.h, ADST_VARDIFF2D9): x'[c] = x[c] + dt * acc, acc the sum
// over the in-grid neighbours n, in the order W, E, S, N, SW, SE, NW, NE, of
// (c_n * (K[c] + K[n])) * (x[n] - x[c]). The weight is the same from both ends
// of an edge and the difference changes only its sign, so an edge's term at
// one end is exactly the negative of that at the other: each edge is
// evaluated once, four a point instead of eight, and the fused second step
// uses the first one's weights again. A dropped edge enters as +0, which
// leaves the sum's bits (it starts from +0 and so is never -0).
//
// Layout. As in the Jacobi march (jacobi_march.h): a workgroup is one wave
// owning 64 blocks of V columns and a chunk of rows, marching along the rows.
// When row q arrives, the edges between rows q-1 and q are evaluated; with the
// ones kept from rows q-2 and q-1 they complete the first step's row q-1, and
// the second step does the same one row behind. Values and edge terms that
// cross a lane's side come from the adjacent lanes by whole-wave shifts. Every
// point's terms and their order are those of the single step, so the bits are
// too.
//
// The LDS tiles that this replaces evaluated eight edges a point, 1.1 times
// the points, and waited at two barriers a tile. Two steps in one launch,
// before and after: 8192^2 f32 245 -> 200 us (4.0 TB/s on its 12 bytes a
// point), storing both states 283 -> 266; 4096^2 f64 162 -> 94, 185 -> 126;
// 2048^2 f32 30 -> 16, 200 x 300 f64 17 -> 10. Three waves a SIMD (a register
// cap of 168) were no faster. It is bound by memory latency: two waves a SIMD
// with four rows of two arrays in flight.

#include <hip/hip_runtime.h>

#include <type_traits>

#include "adst.h"
#include "jacobi_march.h"
#include "kernels.h"

namespace adst {
namespace {

// Rows per chunk of an interior strip: the chunk's four extra rows weigh
// little at these (f32, 8192^2, one launch: 64 / 96 / 128 rows 205 / 200 / 214
// us, storing both states 300 / 288 / 268), and grids that give a launch
// fewer waves than the chip holds take shorter ones (1023 x 1537 f64: 42 us
// with 96 rows, 21 with 24).
constexpr int kVdRows = 96, kVdStoreRows = 128;
constexpr int kVdAhead = 4; // rows requested ahead

// Terms of the edges of one row: to the row after it (n, ne, nw) and along it
// (e).
template <class R, int V>
struct Edges {
  R e[V], n[V], ne[V], nw[V];
};

// One step's state between rows: the current row, its first and last values'
// neighbours in the adjacent lanes, and the terms its points have from the
// row before.
template <class R, int V>
struct Step {
  R x[V], xr;               // row q-1; the right lane's first value of it
  R s[V], sw[V], se[V];
};

template <class R, bool VEC, bool ST, bool NT>
__global__ __launch_bounds__(kLanes) void vd_march(const R* __restrict__ x, const R* __restrict__ K,
                                                   R* __restrict__ y, R* __restrict__ mid, int nx,
                                                   int ny, MarchGrid g, R dt, R ca, R cd) {
  constexpr int V = 16 / (int)sizeof(R), H = V, OW = kLanes * V - 2 * H, P = kVdAhead;
  static_assert(H >= 2, "two steps lose two columns a side");
  int strip, chunk, r0, r1;
  if (!march_item(g, ny, &strip, &chunk, &r0, &r1)) return;
  const int lane = (int)threadIdx.x;
  const int s0 = strip * OW, c0 = s0 - H + lane * V;
  const int nit = (r1 - r0) + 4, q0 = r0 - 2;  // rows r0-2 .. r1+1 arrive
  const int lo_need = max(r0 - 2, 0), hi_need = min(r1 + 1, ny - 1);
  const bool strip_in = s0 - H >= 1 && s0 - H + kLanes * V <= nx - 1;
  const bool st_lane = lane * V >= H && lane * V < H + OW;
  bool cE[V], cC[V], cW[V];  // the column has an E neighbour, is in the grid, has a W neighbour
#pragma unroll
  for (int e = 0; e < V; ++e) {
    const int c = c0 + e;
    cE[e] = c >= 0 && c + 1 < nx;
    cC[e] = c >= 0 && c < nx;
    cW[e] = c >= 1 && c < nx;
  }
  auto march = [&](auto inner_t) {
    constexpr bool INNER = decltype(inner_t)::value;
    auto load = [&](const R* a, int row, R* out) {
      const int rr = min(max(row, lo_need), hi_need);
      load_block<R, VEC, INNER, false>(a + (int64_t)rr * nx, c0, nx, out);
    };
    R px[P][V], pk[P][V];
#pragma unroll
    for (int u = 0; u < P; ++u) {
      load(x, q0 + u, px[u]);
      load(K, q0 + u, pk[u]);
    }
    Step<R, V> a{}, b{};      // first and second step
    Edges<R, V> wb{};         // weights of row q-2's edges
    R kc[V], kr = R(0);       // K's row q-1
#pragma unroll
    for (int e = 0; e < V; ++e) kc[e] = R(0);

    // One step's row r from the row after it (nxt), with the edges' weights;
    // out receives the new values. rows: both rows are in the grid (uniform).
    auto step = [&](Step<R, V>& s, const Edges<R, V>& wt, const R* nxt, bool rows, R* out) {
      const R nl = from_prev(nxt[V - 1]), nr = from_next(nxt[0]);
      Edges<R, V> f;
#pragma unroll
      for (int e = 0; e < V; ++e) {
        const R xc = s.x[e];
        const R xe = e + 1 < V ? s.x[e + 1 < V ? e + 1 : 0] : s.xr;
        const R xne = e + 1 < V ? nxt[e + 1 < V ? e + 1 : 0] : nr;
        const R xnw = e > 0 ? nxt[e > 0 ? e - 1 : 0] : nl;
        f.e[e] = wt.e[e] * (xe - xc);
        f.n[e] = wt.n[e] * (nxt[e] - xc);
        f.ne[e] = wt.ne[e] * (xne - xc);
        f.nw[e] = wt.nw[e] * (xnw - xc);
        if constexpr (!INNER) {
          f.e[e] = cE[e] ? f.e[e] : R(0);
          f.n[e] = cC[e] ? f.n[e] : R(0);
          f.ne[e] = cE[e] ? f.ne[e] : R(0);
          f.nw[e] = cW[e] ? f.nw[e] : R(0);
        }
        f.n[e] = rows ? f.n[e] : R(0);
        f.ne[e] = rows ? f.ne[e] : R(0);
        f.nw[e] = rows ? f.nw[e] : R(0);
      }
      const R wl = from_prev(f.e[V - 1]);
#pragma unroll
      for (int e = 0; e < V; ++e) {
        R acc = R(0);
        acc -= e > 0 ? f.e[e > 0 ? e - 1 : 0] : wl;
        acc += f.e[e];
        acc += s.s[e];
        acc += f.n[e];
        acc += s.sw[e];
        acc += s.se[e];
        acc += f.nw[e];
        acc += f.ne[e];
        out[e] = s.x[e] + dt * acc;
      }
      const R sw = from_prev(f.ne[V - 1]), se = from_next(f.nw[0]);
#pragma unroll
      for (int e = 0; e < V; ++e) {
        s.s[e] = -f.n[e];
        s.sw[e] = -(e > 0 ? f.ne[e > 0 ? e - 1 : 0] : sw);
        s.se[e] = -(e + 1 < V ? f.nw[e + 1 < V ? e + 1 : 0] : se);
        s.x[e] = nxt[e];
      }
      s.xr = nr;
    };

    auto arrive = [&](int q, auto slot_t) {
      constexpr int U = decltype(slot_t)::value;
      R xn[V], kn[V];
#pragma unroll
      for (int e = 0; e < V; ++e) {
        xn[e] = px[U][e];
        kn[e] = pk[U][e];
      }
      load(x, q + P, px[U]);
      load(K, q + P, pk[U]);
      // weights of row q-1's edges
      const R kl = from_prev(kn[V - 1]), krn = from_next(kn[0]);
      Edges<R, V> w;
#pragma unroll
      for (int e = 0; e < V; ++e) {
        w.e[e] = ca * (kc[e] + (e + 1 < V ? kc[e + 1 < V ? e + 1 : 0] : kr));
        w.n[e] = ca * (kc[e] + kn[e]);
        w.ne[e] = cd * (kc[e] + (e + 1 < V ? kn[e + 1 < V ? e + 1 : 0] : krn));
        w.nw[e] = cd * (kc[e] + (e > 0 ? kn[e > 0 ? e - 1 : 0] : kl));
      }
      R x1[V], x2[V];
      step(a, w, xn, q >= 1 && q < ny, x1);            // row q-1
      if constexpr (ST) {
        if (q - 1 >= r0 && q - 1 < r1 && st_lane)
          store_block<R, VEC, NT>(mid + (int64_t)(q - 1) * nx, c0, nx, x1);
      }
      step(b, wb, x1, q >= 2 && q - 1 < ny, x2);       // row q-2
      if (q - 2 >= r0 && q - 2 < r1 && st_lane)
        store_block<R, VEC, NT>(y + (int64_t)(q - 2) * nx, c0, nx, x2);
      wb = w;
#pragma unroll
      for (int e = 0; e < V; ++e) kc[e] = kn[e];
      kr = krn;
    };
    int i = 0;
    for (; i + P <= nit; i += P) {
      arrive(q0 + i, std::integral_constant<int, 0>{});
      arrive(q0 + i + 1, std::integral_constant<int, 1>{});
      arrive(q0 + i + 2, std::integral_constant<int, 2>{});
      arrive(q0 + i + 3, std::integral_constant<int, 3>{});
    }
    if (i < nit) arrive(q0 + i, std::integral_constant<int, 0>{});
    if (i + 1 < nit) arrive(q0 + i + 1, std::integral_constant<int, 1>{});
    if (i + 2 < nit) arrive(q0 + i + 2, std::integral_constant<int, 2>{});
  };
  static_assert(P == 4, "the row loop is unrolled by it");
  if (strip_in)
    march(std::true_type{});
  else
    march(std::false_type{});
}

template <class R>
hipError_t vd_run(const StepShape& s, const R* x, const R* K, R* y, R* mid, hipStream_t st) {
  constexpr int V = 16 / (int)sizeof(R), OW = kLanes * V - 2 * V;
  MarchGrid g;
  int64_t blocks;
  if (!make_grid_fit(s.nx, s.ny, OW, &g, &blocks, mid ? kVdStoreRows : kVdRows, INT32_MAX))
    return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks), block(kLanes);
  const R dt = R(s.p0), ca = R(1) / R(3), cd = R(1) / R(12);
  const bool vec = rows_aligned<R>(s.nx, x, K) && rows_aligned<R>(s.nx, y, mid);
  const bool nt = int64_t(s.nx) * s.ny * int64_t(sizeof(R)) >= kStreamBytes;
#define ADST_VD(VECV, STV, NTV) \
  vd_march<R, VECV, STV, NTV><<<grid, block, 0, st>>>(x, K, y, mid, s.nx, s.ny, g, dt, ca, cd)
  if (vec && mid && nt) ADST_VD(true, true, true);
  else if (vec && mid) ADST_VD(true, true, false);
  else if (vec && nt) ADST_VD(true, false, true);
  else if (vec) ADST_VD(true, false, false);
  else if (mid && nt) ADST_VD(false, true, true);
  else if (mid) ADST_VD(false, true, false);
  else if (nt) ADST_VD(false, false, true);
  else ADST_VD(false, false, false);
#undef ADST_VD
  return hipGetLastError();
}

}  // namespace

hipError_t launch_vardiff_march(const StepShape& s, const void* x, const void* K, void* y,
                                void* mid, hipStream_t st) {
  if (s.kind != ADST_VARDIFF2D9 || s.limit) return hipErrorInvalidValue;
  if (s.dtype == ADST_F64)
    return vd_run<double>(s, static_cast<const double*>(x), static_cast<const double*>(K),
                          static_cast<double*>(y), static_cast<double*>(mid), st);
  return vd_run<float>(s, static_cast<const float*>(x), static_cast<const float*>(K),
                       static_cast<float*>(y), static_cast<float*>(mid), st);
}

}  // namespace adst
