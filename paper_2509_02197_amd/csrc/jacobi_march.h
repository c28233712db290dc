// Device code of the Jacobi marching kernel (see jacobi_march.hip for the
// layout and its reasons).
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "adst.h"
#include "device_common.h"
#include "kernels.h"

namespace adst {
namespace {

constexpr int kLanes = 64;
constexpr int kRows = 48;      // rows per chunk of an interior strip (42 for the
                               // adjoint measured the same: 56.3 against 56.1 us
                               // per 6-step launch at 4096^2, one rocprofv3 job)
constexpr int kLimRows = 128;  // rows per chunk of the limiter's one-step adjoint:
                               // with x and g read non-temporally, 64 / 96 /
                               // 128 / 160 / 192 / 256 / 384 rows took 82.0 /
                               // 82.3 / 81.5 / 86.5 / 83.4 / 97.2 / 115.0 us
                               // per launch at 4096^2 f64 (before the hint,
                               // 192 was best: 90.4 against 92.7 us at 128)
constexpr int kEdgeRows = 12;  // rows per chunk of the first and last strip (fewer on
                               // small grids, see make_grid_fit)
constexpr int kEndRows = 6;    // rows of a strip's first and last chunk, whose
                               // blocks near the grid's top and bottom edge
                               // take the slower general path
constexpr int kAhead = 3;      // input rows loaded ahead of the pipeline
constexpr int kUnroll = 6;     // input rows per straight-line block
constexpr bool kStoreNT = true;  // kept states are read again only after many launches:
                                 // 4096^2 f64 limited call 13.65 -> 13.21 ms
constexpr int kXcds = 8;       // workgroup i runs on XCD i mod 8
static_assert(kUnroll % kAhead == 0 && kUnroll % 3 == 0, "register slots must stay static");
static_assert(2 * kEndRows <= kRows && kEdgeRows <= kRows && kRows <= 64, "chunk sizes");

// Whole-wave lane shifts: lane i receives lane i-1's value (lane 0: 0) or
// lane i+1's (lane 63: 0).
__device__ inline uint32_t shr1(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x138, 0xf, 0xf, true);
}
__device__ inline uint32_t shl1(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x130, 0xf, 0xf, true);
}
__device__ inline float from_prev(float v) { return __uint_as_float(shr1(__float_as_uint(v))); }
__device__ inline float from_next(float v) { return __uint_as_float(shl1(__float_as_uint(v))); }
__device__ inline double from_prev(double v) {
  const uint64_t a = __double_as_longlong(v);
  return __longlong_as_double(
      (long long)(((uint64_t)shr1((uint32_t)(a >> 32)) << 32) | shr1((uint32_t)a)));
}
__device__ inline double from_next(double v) {
  const uint64_t a = __double_as_longlong(v);
  return __longlong_as_double(
      (long long)(((uint64_t)shl1((uint32_t)(a >> 32)) << 32) | shl1((uint32_t)a)));
}

template <class R, int K>
struct Geom {
  static constexpr int V = 16 / sizeof(R);
  static constexpr int H = ((K + V - 1) / V) * V;  // column overlap, whole vectors
  static constexpr int OW = kLanes * V - 2 * H;    // output columns per strip
};

// Work list: the chunks of the first and last strip (E of them) and of the
// interior strips (I). XCD x takes edge chunks [x*pe, (x+1)*pe) and interior
// chunks [x*pi, (x+1)*pi), edge chunks first.
struct MarchGrid {
  int ns, nedge, ce, ci, pe, pi;
  int rows;  // rows per chunk of an interior strip
  int erows; // and of the first and last strip
};

// This workgroup's strip and chunk of rows [r0, r1); false when the
// workgroup has no work (the grid is rounded up to whole XCD shares).
// FIT false: a work list of make_grid, whose edge chunks are kEdgeRows rows.
// item (optional): the work item's index, edge items first, unique in
// [0, nedge*ce + (ns-nedge)*ci).
template <bool FIT = true>
__device__ inline bool march_item(const MarchGrid& g, int ny, int* strip, int* chunk, int* r0,
                                  int* r1, int* item = nullptr) {
  const int xcd = (int)blockIdx.x % kXcds, slot = (int)blockIdx.x / kXcds;
  int nch, mid;
  if (slot < g.pe) {
    const int t = xcd * g.pe + slot;
    if (t >= g.nedge * g.ce) return false;
    *strip = (t / g.ce == 0) ? 0 : g.ns - 1;
    *chunk = t % g.ce;
    nch = g.ce;
    mid = FIT ? g.erows : kEdgeRows;
    if (item) *item = t;
  } else {
    const int t = xcd * g.pi + (slot - g.pe);
    if (t >= (g.ns - g.nedge) * g.ci) return false;
    *strip = 1 + t / g.ci;
    *chunk = t % g.ci;
    nch = g.ci;
    mid = g.rows;
    if (item) *item = g.nedge * g.ce + t;
  }
  // kEndRows at each end of the strip, mid rows between
  const int c = *chunk;
  if (nch == 1) {
    *r0 = 0;
    *r1 = ny;
  } else if (c == 0) {
    *r0 = 0;
    *r1 = kEndRows;
  } else if (c == nch - 1) {
    *r0 = ny - kEndRows;
    *r1 = ny;
  } else {
    *r0 = kEndRows + (c - 1) * mid;
    *r1 = min(*r0 + mid, ny - kEndRows);
  }
  return true;
}

// The work list for strips of ow output columns; false if it is too long.
inline bool make_grid(int nx, int ny, int ow, MarchGrid* g, int64_t* blocks, int rows = kRows,
                      int erows = kEdgeRows) {
  g->rows = rows;
  g->erows = erows;
  g->ns = (nx + ow - 1) / ow;
  g->nedge = g->ns >= 2 ? 2 : 1;
  auto chunks = [&](int mid) {
    return ny > 2 * kEndRows ? 2 + (ny - 2 * kEndRows + mid - 1) / mid : 1;
  };
  g->ce = chunks(erows);
  g->ci = chunks(rows);
  const int64_t E = int64_t(g->nedge) * g->ce, I = int64_t(g->ns - g->nedge) * g->ci;
  g->pe = (int)((E + kXcds - 1) / kXcds);
  g->pi = (int)((I + kXcds - 1) / kXcds);
  *blocks = int64_t(kXcds) * (g->pe + g->pi);
  return *blocks > 0 && *blocks <= INT32_MAX;
}

// As make_grid, with the rows per chunk halved while the launch has fewer
// workgroups (waves) than fill the chip: a launch of few waves takes the time
// of one, the chunk's rows and those beyond its ends (1000 x 1000 f64 under the
// limiter, T = 60: 1.92 -> 0.84 ms). Half and twice the count were within 4%
// for the variable coefficients.
constexpr int kFillWaves = 2048;
// With at most half a wave a SIMD even at kEdgeRows rows, every chunk is as
// short as the end ones: twice the waves still have a SIMD each (64 x 64 f64
// Jacobi call, T = 10: 46.9 -> 42.7 us; 120 x 118 f32 variable coefficients
// with dK, T = 20: 442 -> 361).
constexpr int kFewWaves = 512;
// Jacobi launches of several steps evaluate up to twelve rows beyond a chunk, as
// many as the shortest chunk has, so they take chunks of less than 2 *
// kEdgeRows only where the interior strips have fewer chunks than this (calls of
// 36 steps, us, 24 and 12 rows: f64 1400^2 188 and 210, 2048^2 284 and 301 with
// 285 at 48, 1000^2 178 and 172, 500^2 164 and 149, 4096 x 500 222 and 211, under
// the limiter 2048^2 1113 and 1206, 1000^2 527 and 473; f32 2500^2 257 and 281,
// 14 limited forward steps at 2048^2 61 and 53).
template <class R>
constexpr int kJacShort = sizeof(R) == 8 ? 550 : 700;
inline bool make_grid_fit(int nx, int ny, int ow, MarchGrid* g, int64_t* blocks, int rows,
                          int short_below) {
  if (!make_grid(nx, ny, ow, g, blocks, rows)) return false;
  while (rows > kEdgeRows && *blocks < kFillWaves) {
    if (rows / 2 < 2 * kEdgeRows && int64_t(g->ns - g->nedge) * g->ci >= short_below) break;
    rows = rows / 2 < kEdgeRows ? kEdgeRows : rows / 2;
    if (!make_grid(nx, ny, ow, g, blocks, rows)) return false;
  }
  if (rows <= kEdgeRows && *blocks < kFewWaves)
    return make_grid(nx, ny, ow, g, blocks, kEndRows, kEndRows);
  return true;
}

// The V elements from column c0 (a multiple of V) of the row at src, those
// outside the row with any value. VEC: nx is a multiple of V and rows are
// 16-byte aligned, so a block is in the grid or outside it and one 16-byte load,
// clamped into the row, brings it. INNER: c0 .. c0 + V - 1 lie in the grid; one
// 16-byte load at element alignment where rows are not aligned (with one load
// per element, the waves waited on four times as many: a 2501 x 3003 f32 call of
// 60 steps with dL/dw, 4.21 -> 3.51 ms). Elsewhere one load per element,
// clamped: nothing may touch a value before it enters the pipeline, and with
// one load and its elements moved to their places here, every row of the first
// and last strip waited for its own load (calls of 24 steps with dL/dw, so
// against as it is: 500 x 127 f64 606 and 278 us, 400 x 401 f32 668 and 343;
// moved on entry instead, plain f32 calls took 1.07 times as long as now). NT:
// the non-temporal hint.
template <class R, bool VEC, bool INNER, bool NT>
__device__ inline void load_block(const R* src, int c0, int nx, R* out) {
  constexpr int V = 16 / sizeof(R);
  typedef R vec_t __attribute__((ext_vector_type(V), aligned(VEC ? 16 : sizeof(R))));
  if constexpr (!VEC && !INNER) {
#pragma unroll
    for (int e = 0; e < V; ++e) out[e] = src[min(max(c0 + e, 0), nx - 1)];
  } else {
    const int cc = VEC ? min(max(c0, 0), nx - V) : c0;
    const vec_t* p = reinterpret_cast<const vec_t*>(src + cc);
    vec_t t;
    if constexpr (NT)
      t = __builtin_nontemporal_load(p);
    else
      t = *p;
#pragma unroll
    for (int e = 0; e < V; ++e) out[e] = t[e];
  }
}

// Stores the block's elements that lie in the row at dst.
template <class R, bool VEC, bool NT = false>
__device__ inline void store_block(R* dst, int c0, int nx, const R* o) {
  constexpr int V = 16 / sizeof(R);
  typedef R vec_t __attribute__((ext_vector_type(V), aligned(VEC ? 16 : sizeof(R))));
  if (c0 + V <= nx) {
    vec_t t;
#pragma unroll
    for (int e = 0; e < V; ++e) t[e] = o[e];
    if constexpr (NT)
      __builtin_nontemporal_store(t, reinterpret_cast<vec_t*>(dst + c0));
    else
      *reinterpret_cast<vec_t*>(dst + c0) = t;
  } else if constexpr (!VEC) {
#pragma unroll
    for (int e = 0; e < V; ++e)
      if (c0 + e < nx) dst[c0 + e] = o[e];
  }
}

// 16-byte rows: a block never holds a row's end and is 16-byte aligned.
template <class R>
inline bool rows_aligned(int nx, const void* a, const void* b) {
  return nx % (16 / (int)sizeof(R)) == 0 &&
         ((reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b)) & 15u) == 0;
}

// What the forward variants add: LIM: the limiter's bounds (every new value,
// ring included, is clamped); ST: the buffers of levels 1 .. K-1, whose rows
// of the chunk are stored too (a run of steps whose every state is kept reads
// once and writes n states). NTM: those stores take the non-temporal hint.
template <class R, int K, bool LIM, bool ST>
struct MarchExtra {
  Limit<R> lim;
  R* mid[ST ? K - 1 : 1];
};
template <class R, int K>
struct MarchExtra<R, K, false, false> {};

template <class R, int K, bool ADJ, bool VEC, bool LIM = false, bool ST = false, bool NTM = false>
__global__ __launch_bounds__(kLanes) void jacobi_march(const R* __restrict__ x, R* __restrict__ y,
                                                       int nx, int ny, MarchGrid g, R w,
                                                       MarchExtra<R, K, LIM, ST> ex) {
  static_assert(!ADJ || (!LIM && !ST), "forward variants");
  using G = Geom<R, K>;
  constexpr int V = G::V, H = G::H, OW = G::OW, P = kAhead, U = kUnroll;
  int strip, chunk, r0, r1;
  if (!march_item(g, ny, &strip, &chunk, &r0, &r1)) return;
  const int lane = threadIdx.x;
  const int s0 = strip * OW;
  const int c0 = s0 - H + lane * V;  // first column of this lane
  const int nit = (r1 - r0) + 2 * K;  // input rows through the pipeline
  const int lo_need = max(r0 - K, 0), hi_need = min(r1 + K - 1, ny - 1);

  // Per-lane column facts of the V columns.
  auto cin = [&](int c) { return c >= 1 && c <= nx - 2; };
  bool cok[V], cI[V];
  int side[V];  // 0: column 0, 1: column nx-1, -1: neither
#pragma unroll
  for (int e = 0; e < V; ++e) {
    const int c = c0 + e;
    cok[e] = c >= 0 && c < nx;
    cI[e] = cin(c);
    side[e] = c == 0 ? 0 : (c == nx - 1 ? 1 : -1);
  }
  const bool strip_in = s0 - H >= 2 && s0 - H + kLanes * V <= nx - 2;
  const bool st_lane = lane * V >= H && lane * V < H + OW;
  // This lane's ring column, if any (a lane holds at most one: nx > V), and
  // its element; with 16-byte rows, column 0 is a lane's first element and
  // column nx-1 its last.
  int rside = -1, relem = 0;
#pragma unroll
  for (int e = 0; e < V; ++e)
    if (side[e] >= 0) {
      rside = side[e];
      relem = e;
    }

  // Raw load of input row `row` (clamped to the rows the chunk needs, and
  // to the grid, so every address is in bounds); masked on entry. INNER: all
  // the strip's columns lie in the grid.
  auto load = [&](int row, R* out, auto inner_t) {
    const int rr = min(max(row, lo_need), hi_need);
    load_block<R, VEC, decltype(inner_t)::value, false>(x + (int64_t)rr * nx, c0, nx, out);
  };

  // The adjoint's pipeline holds gi: every ring cell and every cell outside
  // the grid holds +0 there, so each interior point's masked neighbour sum
  // is the plain sum of the pipeline's values (the terms a mask would drop
  // are +0 already). The ring's own values, g + w*sum, read no other ring
  // value and are kept beside the pipeline: ring_lo and ring_hi hold the
  // bottom and top ring rows at the highest level that has evaluated them
  // (one level reaches a given row per input row), and the one interior
  // neighbour a ring-column cell has is recorded at every level in LDS, from
  // which the ring columns of the chunk's rows are summed after the march.
  // Rows of the record: every row a level may evaluate, [r0 - K - U, r1 + K + U).
  constexpr int NR = kRows + 2 * (K + U);
  __shared__ R nbr[ADJ ? 2 * K * NR + kLanes : 1];
  // LDS index of row j's record at level k: nbr_lane + (k-1)*NR + j, or the
  // lane's scratch cell when it has no ring column
  const bool has_ring = rside >= 0;
  const int nbr_lane = rside * K * NR + (K + U) - r0;
  enum { kFast = 0, kCols = 1, kGeneral = 2 };
  // mid_t: the mode of the blocks away from the top and bottom edge.
  auto march = [&](auto dir_t, auto mid_t) {
    constexpr int DIR = decltype(dir_t)::value;  // +1 upward, -1 downward
    const int ifirst = DIR > 0 ? r0 - K : r1 - 1 + K;  // row of input index 0
    // Level k's row of pipeline index p (row ifirst + DIR*p) sits in slot p mod 3.
    R lv[K][3][V];
    R pf[P][V];
    R ring_lo[V], ring_hi[V];
    constexpr auto inner = std::bool_constant<decltype(mid_t)::value == kFast>{};
#pragma unroll
    for (int e = 0; e < V; ++e) ring_lo[e] = ring_hi[e] = R(0);
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int s3 = 0; s3 < 3; ++s3)
#pragma unroll
        for (int e = 0; e < V; ++e) lv[k][s3][e] = R(0);
#pragma unroll
    for (int u = 0; u < P; ++u) load(ifirst + DIR * u, pf[u], inner);

    // kFast: rows in [2, ny-3], strip in columns [2, nx-3]: unmasked forms.
    // kCols: rows in [2, ny-3], strip touching the side edges.
    // kGeneral: anything (rows near or beyond the top and bottom edge).
    auto block = [&](int base, auto mode_t) {
      constexpr int MODE = decltype(mode_t)::value;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int rr = base + u;
        {  // input row rr enters level 0; the row P ahead is requested
          const int row = ifirst + DIR * rr;
          if constexpr (MODE == kFast) {
#pragma unroll
            for (int e = 0; e < V; ++e) lv[0][u % 3][e] = pf[u % P][e];
          } else if constexpr (!ADJ) {
            const bool rok = row >= 0 && row < ny;
#pragma unroll
            for (int e = 0; e < V; ++e)
              lv[0][u % 3][e] = (rok && cok[e]) ? pf[u % P][e] : R(0);
          } else {
            if constexpr (MODE == kGeneral) {
#pragma unroll
              for (int e = 0; e < V; ++e) {
                const R v = cok[e] ? pf[u % P][e] : R(0);
                ring_lo[e] = row == 0 ? v : ring_lo[e];
                ring_hi[e] = row == ny - 1 ? v : ring_hi[e];
              }
            }
            const bool rin = MODE == kCols || (row >= 1 && row <= ny - 2);
#pragma unroll
            for (int e = 0; e < V; ++e) lv[0][u % 3][e] = (rin && cI[e]) ? pf[u % P][e] : R(0);
          }
          load(row + DIR * P, pf[u % P], inner);
        }
#pragma unroll
        for (int k = 1; k <= K; ++k) {
          const int j = ifirst + DIR * (rr - k);  // row level k evaluates now
          constexpr int off = 3 * (K + 2);
          const int sOld = (u - k - 1 + off) % 3, sc = (u - k + off) % 3,
                    sNew = (u - k + 1 + off) % 3;
          const R* a = lv[k - 1][sc];
          const R* S = lv[k - 1][DIR > 0 ? sOld : sNew];
          const R* N = lv[k - 1][DIR > 0 ? sNew : sOld];
          const R wl = from_prev(a[V - 1]), er = from_next(a[0]);
          const bool rj = MODE != kGeneral || (j >= 1 && j <= ny - 2);  // uniform
          R o[V];
          if constexpr (!ADJ) {
#pragma unroll
            for (int e = 0; e < V; ++e) {
              const R Wn = e > 0 ? a[e > 0 ? e - 1 : 0] : wl;
              const R En = e < V - 1 ? a[e < V - 1 ? e + 1 : 0] : er;
              const R f = w * ((((a[e] + Wn) + En) + S[e]) + N[e]);
              if constexpr (MODE == kFast)
                o[e] = f;
              else
                o[e] = (cI[e] && rj) ? f : a[e];
              if constexpr (LIM) o[e] = limited(o[e], ex.lim);
            }
          } else {
            R sum[V], Ws[V], Es[V];
#pragma unroll
            for (int e = 0; e < V; ++e) {
              Ws[e] = e > 0 ? a[e > 0 ? e - 1 : 0] : wl;
              Es[e] = e < V - 1 ? a[e < V - 1 ? e + 1 : 0] : er;
              sum[e] = ((Ws[e] + Es[e]) + S[e]) + N[e];
            }
#pragma unroll
            for (int e = 0; e < V; ++e) {
              if constexpr (MODE == kFast)
                o[e] = w * (a[e] + sum[e]);
              else
                o[e] = (cI[e] && rj) ? w * (a[e] + sum[e]) : R(0);
            }
            if constexpr (MODE != kFast) {
              // record the ring cell's interior neighbour (E of column 0, W
              // of column nx-1) for rows of this chunk; other lanes write
              // their own scratch cell
              R nb;
              if constexpr (VEC) {
                nb = rside == 0 ? Es[0] : Ws[V - 1];
              } else {
                nb = R(0);
#pragma unroll
                for (int e = 0; e < V; ++e) nb = relem == e ? (rside == 0 ? Es[e] : Ws[e]) : nb;
              }
              nbr[has_ring ? nbr_lane + (k - 1) * NR + j : 2 * K * NR + lane] = nb;
            }
            if constexpr (MODE == kGeneral) {
#pragma unroll
              for (int e = 0; e < V; ++e) {
                ring_lo[e] = j == 0 ? (cok[e] ? ring_lo[e] + w * sum[e] : R(0)) : ring_lo[e];
                ring_hi[e] = j == ny - 1 ? (cok[e] ? ring_hi[e] + w * sum[e] : R(0)) : ring_hi[e];
              }
            }
          }
          if (k < K) {
#pragma unroll
            for (int e = 0; e < V; ++e) lv[k][sc][e] = o[e];
            if constexpr (ST) {
              if (j >= r0 && j < r1 && st_lane)
                store_block<R, VEC, NTM>(ex.mid[k - 1] + (int64_t)j * nx, c0, nx, o);
            }
          } else if (j >= r0 && j < r1 && st_lane) {
            if constexpr (ADJ && MODE == kGeneral) {  // ring rows
#pragma unroll
              for (int e = 0; e < V; ++e)
                o[e] = j == 0 ? ring_lo[e] : (j == ny - 1 ? ring_hi[e] : o[e]);
            }
            store_block<R, VEC>(y + (int64_t)j * nx, c0, nx, o);
          }
        }
      }
    };

    // A block of U input rows evaluates rows ifirst + DIR*[base - K, base + U - 1];
    // blocks [fa, fb) have all of them in [2, ny - 3].
    int fa, fb;
    if (DIR > 0) {
      fa = 2 + K - ifirst;
      fb = ny - 1 - ifirst - U;
    } else {
      fa = ifirst + K - (ny - 3);
      fb = ifirst - U;
    }
    fa = ((max(fa, 0) + U - 1) / U) * U;
    using General = std::integral_constant<int, kGeneral>;
    int base = 0;
    for (; base < nit && base < fa; base += U) block(base, General{});
    for (; base < nit && base < fb; base += U) block(base, mid_t);
    for (; base < nit; base += U) block(base, General{});
  };
  // Each combination gets its own straight code path, chosen before any
  // state is live.
  using Up = std::integral_constant<int, 1>;
  using Down = std::integral_constant<int, -1>;
  using Fast = std::integral_constant<int, kFast>;
  using Cols = std::integral_constant<int, ADJ ? kCols : kGeneral>;
  if (strip_in) {
    if (chunk & 1)
      march(Down{}, Fast{});
    else
      march(Up{}, Fast{});
    return;
  }
  if (chunk & 1)
    march(Down{}, Cols{});
  else
    march(Up{}, Cols{});
  if constexpr (ADJ) {
    // The ring columns of this chunk's interior rows, one row per lane:
    // g_n = g_0 + w*(((0 + E) + 0) + 0) level by level on the left,
    // g_0 + w*(((W + 0) + 0) + 0) on the right, E and W the recorded
    // neighbours. All earlier stores and LDS writes complete first.
    __builtin_amdgcn_s_waitcnt(0);
    asm volatile("" ::: "memory");
    const int jr = r0 + lane;
    if (lane < kRows && jr < r1 && jr >= 1 && jr <= ny - 2) {
#pragma unroll
      for (int sd = 0; sd < 2; ++sd) {
        const int col = sd == 0 ? 0 : nx - 1;
        if (col < s0 || col >= s0 + OW) continue;  // not this strip's output column
        const int64_t q = (int64_t)jr * nx + col;
        R g = x[q];
#pragma unroll
        for (int k = 0; k < K; ++k) {
          const R v = nbr[(sd * K + k) * NR + (K + U) + lane];
          const R sum = sd == 0 ? ((R(0) + v) + R(0)) + R(0) : ((v + R(0)) + R(0)) + R(0);
          g = g + w * sum;
        }
        y[q] = g;
      }
    }
  }
}

}  // namespace
}  // namespace adst
