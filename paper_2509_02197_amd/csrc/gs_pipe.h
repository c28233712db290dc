// Device code of the persistent Gauss-Seidel pipeline (host side and the
// reasons for the layout: gs_pipe.hip).
#pragma once

#include <cstdint>

namespace adst {
namespace {

constexpr int kGpLanes = 64;  // one wave per strip and run of kGpQ phases
constexpr int kGpQ = 2;       // phases a wave carries in registers
constexpr int kGpB = 8;       // clocks between two barriers (a macro step)
constexpr int kGpFlagInts = 32;  // a progress counter has a 128-byte line of its own

struct GpArgs {
  void* buf;         // the state, updated in place
  const void* src;   // where the launch's first group reads (the first sweep's input, or buf)
  int* flags;        // ticket, then one progress counter per (group, column)
  void* halo;        // [min(2, ngroups)][nj][phases of a group][ny] values
  int nx, ny;
  int nph;           // phases of this launch
  int ph0, ph_all;   // the first one's index, and how many the whole run has
  int ngroups, ncol, nj;  // groups, columns of workgroups (the most any group has), strips
};

template <class R>
struct alignas(16) GpVec {
  static constexpr int V = 16 / (int)sizeof(R);
  R v[V];  // processing order
};

template <class R, int NW>
struct GpShared {
  // Entry l+1 of a slot: lane l's block; entry 0: only its last value, the
  // left neighbour's. Inputs of wave a; the last one: output.
  GpVec<R> ring[NW + 1][2][kGpB][kGpLanes + 1];
  R edge[NW][2][kGpB][kGpQ];  // the left strip's last value, by clock and phase
  int ticket;
};

template <class T>
__device__ inline T agent_load(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ inline void agent_store(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline uint32_t gp_shr1(uint32_t v, uint32_t edge) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)edge, (int)v, 0x138, 0xf, 0xf, false);
}
// Lane i receives lane i+1's value, lane 63 its own `edge`.
__device__ inline uint32_t gp_shl1(uint32_t v, uint32_t edge) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)edge, (int)v, 0x130, 0xf, 0xf, false);
}
// Every lane of a group of four receives the value of the group's lane K.
template <int K>
__device__ inline uint32_t gp_quad(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, K * 0x55, 0xf, 0xf, true);
}
template <class F>
__device__ inline float gp_each(float v, float edge, F f) {
  return __uint_as_float(f(__float_as_uint(v), __float_as_uint(edge)));
}
template <class F>
__device__ inline double gp_each(double v, double edge, F f) {
  const uint64_t a = (uint64_t)__double_as_longlong(v), e = (uint64_t)__double_as_longlong(edge);
  const uint32_t lo = f((uint32_t)a, (uint32_t)e);
  const uint32_t hi = f((uint32_t)(a >> 32), (uint32_t)(e >> 32));
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
// Lane i receives lane i-1's value, lane 0 its own `edge`; and the opposite.
template <class R>
__device__ inline R gp_prev(R v, R edge) {
  return gp_each(v, edge, [](uint32_t a, uint32_t e) { return gp_shr1(a, e); });
}
template <class R>
__device__ inline R gp_next(R v, R edge) {
  return gp_each(v, edge, [](uint32_t a, uint32_t e) { return gp_shl1(a, e); });
}
template <int K, class R>
__device__ inline R gp_quad_lane(R v) {
  return gp_each(v, v, [](uint32_t a, uint32_t) { return gp_quad<K>(a); });
}

// m is all ones or zero: a where it is ones, else b (one bit select an
// element half: from C++ selects the compiler makes branches around the
// arithmetic, and masks kept in scalar registers spill), and a or +0.
__device__ inline uint32_t gp_sel32(uint32_t m, uint32_t a, uint32_t b) {
  uint32_t r;
  asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(r) : "v"(m), "v"(a), "v"(b));
  return r;
}
__device__ inline float gp_sel(uint32_t m, float a, float b) {
  return __uint_as_float(gp_sel32(m, __float_as_uint(a), __float_as_uint(b)));
}
__device__ inline double gp_sel(uint32_t m, double a, double b) {
  const uint64_t ua = (uint64_t)__double_as_longlong(a), ub = (uint64_t)__double_as_longlong(b);
  const uint32_t lo = gp_sel32(m, (uint32_t)ua, (uint32_t)ub);
  const uint32_t hi = gp_sel32(m, (uint32_t)(ua >> 32), (uint32_t)(ub >> 32));
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
__device__ inline float gp_keep(uint32_t m, float a) {
  return __uint_as_float(m & __float_as_uint(a));
}
__device__ inline double gp_keep(uint32_t m, double a) {
  const uint64_t ua = (uint64_t)__double_as_longlong(a);
  return __longlong_as_double(
      (long long)(((uint64_t)(m & (uint32_t)(ua >> 32)) << 32) | (m & (uint32_t)ua)));
}
// A mask in a vector register: hidden from the compiler, which otherwise
// turns it back into a lane mask in scalar registers.
__device__ inline uint32_t gp_mask(bool b) {
  uint32_t m = b ? ~0u : 0u;
  asm("" : "+v"(m));
  return m;
}

__device__ inline void gp_wait_memory() {
  __builtin_amdgcn_s_waitcnt(0);
  asm volatile("" ::: "memory");
}

// NW: waves of a workgroup, each kGpQ phases after the one before.
template <class R, bool ADJ, int NW>
__global__ __launch_bounds__(kGpLanes * NW) void gs_pipe(GpArgs p, R w) {
  constexpr int V = GpVec<R>::V, Q = kGpQ, B = kGpB, NL = kGpLanes;
  constexpr int S = Q * NW;                    // phases of a group
  constexpr int NC = NL * V;                   // columns of a strip
  constexpr int kGpThreads = NL * NW;
  constexpr int kItems = B * NL / kGpThreads;  // state blocks a thread moves per macro step
  static_assert(B * NL % kGpThreads == 0 && (Q + 1) * B <= NL && NL % B == 0, "item mapping");
  static_assert(Q <= 4, "the phases' edges come from the lanes of one quad");
  typedef GpVec<R> Vec;
  __shared__ GpShared<R, NW> sm;
  const int tid = (int)threadIdx.x, lane = tid % NL;
  const int a = __builtin_amdgcn_readfirstlane(tid / NL);
  if (tid == 0) sm.ticket = atomicAdd(p.flags, 1);
  __syncthreads();
  int t = __builtin_amdgcn_readfirstlane(sm.ticket);
  if (t >= p.ngroups * p.ncol) return;
  // the ticket's group and column: by their sum, the smaller group first
  int d = 0, G = 0;
  const int ramp = p.ngroups * (p.ngroups - 1) / 2;
  if (p.ncol > p.ngroups && t >= ramp) {  // sums of ngroups tickets each
    const int k = min((t - ramp) / p.ngroups, p.ncol - p.ngroups);
    d = p.ngroups - 1 + k;
    t -= ramp + k * p.ngroups;
  }
  for (;; ++d) {
    G = max(0, d - p.ncol + 1);
    const int n = min(d, p.ngroups - 1) - G + 1;
    if (t < n) break;
    t -= n;
  }
  G += t;
  // strips whose columns some phase of group g touches
  auto j_lo = [&](int g) { return g * S / NC; };
  auto waves_of = [&](int g) { return (min(S, p.nph - g * S) + Q - 1) / Q; };
  auto j_hi = [&](int g) { return (p.nx - 1 + g * S + waves_of(g) * Q - 1) / NC; };
  const int J = j_lo(G) + d - G;
  if (J > j_hi(G)) return;
  const int nwa = waves_of(G);
  const int nx = p.nx, ny = p.ny;
  const int C0 = NC * J - G * S;  // lane 0's first column in the group's first phase
  const int KL = nwa * Q - 1;     // the group's last phase
  auto macros = [&](int nw) { return (ny + NL + 2 + 2 * (nw * Q - 1) + B - 1) / B; };
  const int nmac = macros(nwa), NT = nmac + nwa, NTfull = macros(NW) + NW;
  auto exists = [&](int g, int j) { return g >= 0 && j >= j_lo(g) && j <= j_hi(g); };
  auto flag_of = [&](int g, int j) {
    return p.flags + (int64_t)(1 + g * p.ncol + (j - j_lo(g))) * kGpFlagInts;
  };
  const bool hasL = J - 1 >= j_lo(G), hasR = J + 1 <= j_hi(G);
  // 0: the strip's own columns, 1: the column left of them, both one group
  // earlier; 2: the left strip; 3: the reader of the halo slots this group
  // writes over
  int* const self = flag_of(G, J);
  const bool dep[4] = {exists(G - 1, J), exists(G - 1, J - 1), hasL, hasR && exists(G - 2, J + 1)};
  const int* fl[4];
  fl[0] = dep[0] ? flag_of(G - 1, J) : self;
  fl[1] = dep[1] ? flag_of(G - 1, J - 1) : self;
  fl[2] = dep[2] ? flag_of(G, J - 1) : self;
  fl[3] = dep[3] ? flag_of(G - 2, J + 1) : self;
  const int* const myfl = (lane & 3) == 0   ? fl[0]
                          : (lane & 3) == 1 ? fl[1]
                          : (lane & 3) == 2 ? fl[2]
                                            : fl[3];
  int seen[4] = {0, 0, 0, 0};
  auto wait_for = [&](int q, int need) {
    if (!dep[q] || seen[q] >= need) return;
    int v;
    while ((v = __builtin_amdgcn_readfirstlane(agent_load(fl[q]))) < need)
      __builtin_amdgcn_s_sleep(1);
    seen[q] = v;
  };

  R* const buf = static_cast<R*>(p.buf);
  const R* const in = G == 0 ? static_cast<const R*>(p.src) : buf;
  const int64_t hrow = (int64_t)S * ny;  // halo values of one strip
  R* const halo_out = static_cast<R*>(p.halo) + ((int64_t)(G & 1) * p.nj + J) * hrow;
  const R* const halo_in = halo_out - hrow;
  auto row_ok = [&](int rho) { return rho >= 0 && rho < ny; };
  // offset of the processing cell (rho, cp) from the first processing cell
  auto cell = [&](int rho, int cp) {
    const int64_t o = (int64_t)rho * nx + cp;
    return ADJ ? (int64_t)ny * nx - 1 - o : o;
  };
  const int64_t mstep = ADJ ? -(int64_t)B * nx : (int64_t)B * nx;  // one macro step on
  constexpr int cs = ADJ ? -1 : 1;                                 // one column on

  // State blocks this thread loads and stores: lane l, clock i of a macro
  // step, so that neighbouring threads move neighbouring blocks of a row.
  // Row and address are of the next macro step to be moved.
  int irow[kItems], orow[kItems], icol[kItems], ocol[kItems];
  int64_t ioff[kItems], ooff[kItems];
#pragma unroll
  for (int q = 0; q < kItems; ++q) {
    const int id = tid + q * kGpThreads, i = id % B, l = (id / B + i) % NL;
    irow[q] = i - 1 - l;
    orow[q] = i - 3 - l - 2 * KL;
    icol[q] = C0 + 1 + l * V;
    ocol[q] = C0 - KL + l * V;
    ioff[q] = cell(irow[q], icol[q]);
    ooff[q] = cell(orow[q], ocol[q]);
  }
  int erow = tid;  // the column left of the strip: threads 0 .. B-1
  int64_t eoff = cell(erow, C0);

  // Phase kinds of this wave: recur, finish, and phases past the last, which
  // only carry values along. Masks of each phase's elements in this lane:
  // interior column (cin); ring column that collects in this phase (ract);
  // the first column (first); the next, the previous element is no ring cell
  // (nok, pok).
  bool starts = false, ends = false;
  uint32_t recur[Q], finish[Q], idle[Q];
  uint32_t cin[Q][V], ract[Q][V], first[Q][V], nok[Q][V], pok[Q][V];
#pragma unroll
  for (int k = 0; k < Q; ++k) {
    const int K = Q * a + k, ph = G * S + K;
    const bool live = nx >= 3 && ny >= 3 && ph < p.nph;
    const bool rec = ADJ && p.ph0 + ph == 0, fin = ADJ && p.ph0 + ph == p.ph_all - 1;
    starts = starts || rec;
    ends = ends || !live || fin;
    recur[k] = gp_mask(rec);
    finish[k] = gp_mask(fin);
    idle[k] = gp_mask(!live);
#pragma unroll
    for (int e = 0; e < V; ++e) {
      const int cp = C0 - K + lane * V + e;
      cin[k][e] = gp_mask(live && cp >= 1 && cp <= nx - 2);
      ract[k][e] = gp_mask(live && ((cp == 0 && !rec) || (cp == nx - 1 && !fin)));
      first[k][e] = gp_mask(cp == 0);
      nok[k][e] = gp_mask(cp != nx - 2);
      pok[k][e] = gp_mask(cp != 1);
    }
  }
  // every column of the wave lies two or more columns from the side edges
  const bool cols_in = C0 - (Q * a + Q - 1) >= 2 && C0 - Q * a + NC - 1 <= nx - 3;

  // Of each phase: its result of the last clock (O); its row's old values
  // with the one after them (X); the left lane's last result of the clock
  // before the last (shp; innb for the input); the last lane's last results
  // of the macro step's clocks, clock i in lane NL - B + i (hist).
  Vec O[Q];
  R X[Q][V + 1], shp[Q], hist[Q], innb = R(0);
#pragma unroll
  for (int k = 0; k < Q; ++k) {
#pragma unroll
    for (int e = 0; e < V; ++e) O[k].v[e] = X[k][e] = R(0);
    X[k][V] = shp[k] = hist[k] = R(0);
  }

  // COLS: some column of the wave may be within two of a side edge; ROWS:
  // some row of the macro step within two of the first or last. SPEC: 1: the
  // wave's first phase may be the run's; 2: any phase may be the run's last
  // or past it.
  auto clocks = [&](auto cols_t, auto rows_t, auto spec_t, int mu, int pr, int pw) {
    constexpr bool COLS = decltype(cols_t)::value, ROWS = decltype(rows_t)::value;
    constexpr int SPEC = decltype(spec_t)::value;
    // An LDS access holds the CU's LDS for about 14 cycles however few lanes
    // it is for, so lane 0's values of all phases come in one (in lanes 0 to
    // Q-1) and lane 63's go out once a macro step (hist): with one access a
    // phase and clock each way, LDS was what bounded the loop.
    const int edge_lane = min(lane, Q - 1);
    Vec inN;
    R nbN, edN;
    auto fetch = [&](int i) {
      inN = sm.ring[a][pr][i][lane + 1];
      nbN = sm.ring[a][pr][i][lane].v[V - 1];
      edN = sm.edge[a][pr][i][edge_lane];
    };
    fetch(0);
    // row masks of phase k's row: interior, the first two and the last two
    struct Rows {
      uint32_t rin, row0, row1, rowN2, rowN1;
    };
    Rows rm[3][Q];  // this clock's, the last one's, the one's before
    auto row_masks = [&](Rows& r, int row) {
      r.rin = gp_mask(row >= 1 && row <= ny - 2);
      r.row0 = gp_mask(row == 0);
      r.row1 = gp_mask(row == 1);
      r.rowN2 = gp_mask(row == ny - 2);
      r.rowN1 = gp_mask(row == ny - 1);
    };
    const int t0 = B * mu - 2 - 2 * Q * a - lane;  // phase 0's row at the first clock
    if constexpr (ROWS) {
#pragma unroll
      for (int k = 0; k < Q; ++k) {
        row_masks(rm[0][k], t0 - 1 - 2 * k);
        row_masks(rm[1][k], t0 - 2 - 2 * k);
      }
    }
#pragma unroll
    for (int i = 0; i < B; ++i) {
      const Vec x0 = inN;
      const R x0n = nbN;
      R sh[Q];
      sh[0] = gp_prev(O[0].v[V - 1], edN);
      if constexpr (Q > 1) sh[1 % Q] = gp_prev(O[1 % Q].v[V - 1], gp_quad_lane<1>(edN));
      if constexpr (Q > 2) sh[2 % Q] = gp_prev(O[2 % Q].v[V - 1], gp_quad_lane<2>(edN));
      if constexpr (Q > 3) sh[3 % Q] = gp_prev(O[3 % Q].v[V - 1], gp_quad_lane<3>(edN));
      sm.ring[a + 1][pw][i][lane + 1] = O[Q - 1];
      if (i + 1 < B) fetch(i + 1);
      if constexpr (ROWS) {  // phase k is where phase k-1 was two clocks ago
#pragma unroll
        for (int k = 0; k < Q; ++k) {
          rm[2][k] = rm[1][k];
          rm[1][k] = rm[0][k];
        }
#pragma unroll
        for (int k = Q - 1; k > 0; --k) rm[0][k] = rm[2][k - 1];
        row_masks(rm[0][0], t0 + i);
      }
#pragma unroll
      for (int k = Q - 1; k >= 0; --k) {
        R N[V + 1];  // the next row's old values, as X
        N[0] = k == 0 ? innb : shp[k > 0 ? k - 1 : 0];
#pragma unroll
        for (int e = 0; e < V; ++e) N[e + 1] = k == 0 ? x0.v[e] : O[k > 0 ? k - 1 : 0].v[e];
        const Vec PR = O[k];
        const Rows& rk = rm[0][k];
        R px = sh[k];
        Vec y;
#pragma unroll
        for (int e = 0; e < V; ++e) {
          const R cv = X[k][e], nxv = X[k][e + 1], nr = N[e], pv = PR.v[e];
          uint32_t inner = cin[k][e];
          if constexpr (ROWS) inner &= rk.rin;
          R r;
          if constexpr (!ADJ) {
            r = w * ((((cv + nxv) + nr) + pv) + px);
            if constexpr (COLS) r = gp_sel(inner, r, cv);
            else if constexpr (SPEC == 2) r = gp_sel(idle[k], cv, r);
          } else {
            // a ring cell enters its interior neighbour's sums as 0
            R hW = nxv, hS = nr, hN = pv, hE = px;
            if constexpr (COLS) {
              hW = gp_keep(nok[k][e], hW);
              hE = gp_keep(pok[k][e], hE);
            }
            if constexpr (ROWS) {
              hS = gp_keep(~rk.rowN2, hS);
              hN = gp_keep(~rk.row1, hN);
            }
            R gin = w * ((cv + hW) + hS);
            if constexpr (SPEC != 0) {
              if (k == 0) gin = gp_sel(recur[k], cv, gin);
            }
            R yi = (gin + w * hN) + w * hE;
            if constexpr (SPEC == 2) yi = gp_sel(finish[k], gin, yi);
            r = yi;
            if constexpr (COLS) {
              // Ring cells collect w * h of their interior neighbour, phase
              // by phase: the first column and row from its old value (the
              // result of the phase before), the last ones from its new one.
              R nb = gp_sel(first[k][e], nxv, px);
              uint32_t act = ract[k][e];
              if constexpr (ROWS) {
                nb = gp_sel(rk.row0, nr, gp_sel(rk.rowN1, pv, nb));
                act = (act & rk.rin) |
                      (cin[k][e] & ((rk.row0 & ~recur[k]) | (rk.rowN1 & ~finish[k])));
              }
              R yr = cv + w * nb;
              if constexpr (ROWS || SPEC != 0) {
                if (ROWS || SPEC == 2 || k == 0) yr = gp_sel(act, yr, cv);
              }
              r = gp_sel(inner, yi, yr);
            } else if constexpr (SPEC == 2) {
              r = gp_sel(idle[k], cv, r);
            }
          }
          px = r;
          y.v[e] = r;
        }
        hist[k] = gp_next(hist[k], PR.v[V - 1]);
#pragma unroll
        for (int e = 0; e <= V; ++e) X[k][e] = N[e];
        O[k] = y;
      }
#pragma unroll
      for (int k = 0; k < Q; ++k) shp[k] = sh[k];
      innb = x0n;
    }
  };

  for (int M = -1; M < NT; ++M) {
    const int rd = (M + 1) & 1, wr = M & 1;  // LDS halves read and written (M = -1: writes half 1)
    // ---- waits: what the stores and loads below touch (see gs_pipe.hip)
    wait_for(3, min(M - NL / B, NTfull));
    if (M + 1 < nmac) {
      wait_for(0, min((B * (M + 2) - 1 + 2 * S) / B + NW + 1, NTfull));
      wait_for(1, min((B * (M + 2) - 1 + NL + 2 * S) / B + NW + 1, NTfull));
    }
    wait_for(2, min((B * (M + 2) - 1 + NL) / B + 2, NT));
    asm volatile("" ::: "memory");
    // ---- results of the time before
    {
      const int mu = M - nwa;
      if (mu >= 0 && mu < nmac) {
#pragma unroll
        for (int q = 0; q < kItems; ++q) {
          const int id = tid + q * kGpThreads, i = id % B, l = (id / B + i) % NL;
          if (row_ok(orow[q])) {
            const Vec r = sm.ring[nwa][rd][i][l + 1];
#pragma unroll
            for (int e = 0; e < V; ++e)
              if (ocol[q] + e >= 0 && ocol[q] + e < nx) agent_store(buf + ooff[q] + cs * e, r.v[e]);
          }
          orow[q] += B;
          ooff[q] += mstep;
        }
      }
      const int mh = M - 1 - a, i = lane - (NL - B);
      if (hasR && a < nwa && mh >= 0 && mh < nmac && i >= 0) {
#pragma unroll
        for (int k = 0; k < Q; ++k) {
          const int rho = B * mh + i - 3 - (NL - 1) - 2 * (Q * a + k);
          if (row_ok(rho)) agent_store(halo_out + (int64_t)(Q * a + k) * ny + rho, hist[k]);
        }
      }
    }
    // ---- requests for the next time
    const int polled = agent_load(myfl);
    Vec xin[kItems];
    R xedge = R(0), xh = R(0);
    const bool need_in = M + 1 < nmac;
    const int mh = M + 1 - a;
    const bool need_h = a < nwa && mh >= 0 && mh < nmac && lane < (Q + 1) * B;
    const int hs = lane / B, hi = lane % B;
    if (need_in) {
#pragma unroll
      for (int q = 0; q < kItems; ++q) {
#pragma unroll
        for (int e = 0; e < V; ++e) {
          xin[q].v[e] = R(0);
          if (row_ok(irow[q]) && icol[q] + e >= 0 && icol[q] + e < nx)
            xin[q].v[e] = agent_load(in + ioff[q] + cs * e);
        }
        irow[q] += B;
        ioff[q] += mstep;
      }
      if (tid < B && row_ok(erow) && C0 >= 0 && C0 < nx) xedge = agent_load(in + eoff);
      erow += B;
      eoff += mstep;
    }
    if (need_h && hasL) {
      const int K = Q * a - 1 + hs, rho = B * mh + hi - 2 - 2 * K;
      if (K >= 0 && row_ok(rho)) xh = agent_load(halo_in + (int64_t)K * ny + rho);
    }
    // ---- this time's clocks
    const int mu = M - a;
    if (a < nwa && mu >= 0 && mu < nmac) {
      const int rmin = B * mu - 2 - (NL - 1) - 2 * (Q * a + Q - 1), rmax = B * mu + B - 3 - 2 * Q * a;
      using T = std::true_type;
      using F = std::false_type;
      using Z = std::integral_constant<int, 0>;
      using Starts = std::integral_constant<int, ADJ ? 1 : 0>;
      using Ends = std::integral_constant<int, 2>;
      if (rmin < 2 || rmax > ny - 3)
        clocks(T{}, T{}, Ends{}, mu, rd, wr);
      else if (!cols_in && ends)
        clocks(T{}, F{}, Ends{}, mu, rd, wr);
      else if (!cols_in && starts)
        clocks(T{}, F{}, Starts{}, mu, rd, wr);
      else if (!cols_in)
        clocks(T{}, F{}, Z{}, mu, rd, wr);
      else if (ends)
        clocks(F{}, F{}, Ends{}, mu, rd, wr);
      else if (starts)
        clocks(F{}, F{}, Starts{}, mu, rd, wr);
      else
        clocks(F{}, F{}, Z{}, mu, rd, wr);
    }
    // ---- the requests have arrived and the stores above are done
    gp_wait_memory();
    if (need_in) {
#pragma unroll
      for (int q = 0; q < kItems; ++q) {
        const int id = tid + q * kGpThreads, i = id % B, l = (id / B + i) % NL;
        sm.ring[0][wr][i][l + 1] = xin[q];
      }
      if (tid < B) sm.ring[0][wr][tid][0].v[V - 1] = xedge;
    }
    if (need_h) {
      if (hs > 0)
        sm.edge[a][wr][hi][hs - 1] = xh;
      else if (a > 0)
        sm.ring[a][wr][hi][0].v[V - 1] = xh;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      seen[q] = max(seen[q], __builtin_amdgcn_readlane(polled, q));
    __syncthreads();
    if (tid == 0 && M >= 0) agent_store(self, M + 1);
  }
}

}  // namespace
}  // namespace adst
