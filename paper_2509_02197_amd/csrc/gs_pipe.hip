// In-place Gauss-Seidel sweeps and reverse sweeps as one persistent launch.
//
// gauss_seidel.hip states the step, its reverse and the processing
// coordinates (each point needs the new values of its previous row and
// element and the old values of itself, its next row and next element). It
// runs them as one launch per wavefront level, so a run takes hundreds of
// dependent launches of 9 to 27 us, each bound by a tile's load latency and
// 32-step chain. Here the same order of point updates runs as a pipeline
// inside one launch, and the state passes through memory once per group of
// 8 or 16 phases (a phase is a sweep, or a fused reverse sweep). f64, 100
// sweeps and their reverse: 400 x 400 7.4 -> 1.07 ms, 4096 x 4096 26.4 ->
// 6.8 ms. What bounds it now is the pipeline's length (rows, plus 88 clocks
// a strip and about 80 a group) times the clock of the slowest strip, the
// ones at the sides, of which about half is arithmetic and half the waits,
// barrier and address work of a macro step.
//
// Skew. A lane owns 16 bytes of a row (V elements) and walks the rows, one
// clock a row; lane l is one row behind lane l-1, phase k two rows behind
// phase k-1. A strip's columns also move one element to the left with every
// phase: in processing columns, element e of lane l in phase k is C0 - k +
// l*V + e. Then all that a lane reads in phase k is its own or its left
// neighbour's: its row's old values are elements -1 .. V-1 of phase k-1, that
// is the left lane's last one and its own, shifted by one; so are the next
// row's; the previous element is the left lane's last one of phase k. One
// lane shift of one value a phase and clock serves all of it (a shift
// instruction issues in 5.5 cycles, an f64 addition in 5, an integer one in
// 2.3). A wave carries kGpQ = 2 phases in registers, a workgroup 4 or 8
// waves, each one macro step (kGpB = 8 clocks, one barrier) after the one
// before, which hands its last phase over through LDS. Four phases a wave
// and four waves took 1.32 and 7.4 ms for the two sizes above.
//
// Strips and groups. Because the columns move left with the phases, a strip
// needs nothing from the strip right of it: it reads from its left neighbour
// one value per row and phase (the neighbour's last lane, through the halo
// buffer in the caller's scratch) and from the group before what that group
// stored into the state. Workgroup (G, J) therefore waits only for (G-1, J),
// (G-1, J-1) and (G, J-1), and, before it writes over the halo slots of group
// G-2, for their reader (G-2, J+1). Workgroups draw (G, J) from a ticket, by
// G + column and then G, the order in which they can start: all four have
// smaller tickets, so they have started when this one starts, and every wait
// ends whatever number of workgroups the chip holds at once (one a CU).
//
// Progress. A workgroup publishes the number of macro times it has finished:
// at time M it stores the results of time M-1, requests its inputs of time
// M+1 and computes time M (wave a macro step M-a); then every wave waits for
// its memory operations, the workgroup meets at a barrier and one thread
// stores M+1. Values that workgroups exchange (state, halo, progress) are
// read and written with agent-scope atomic accesses, which the per-XCD caches
// do not hold back, so the wait and barrier before the progress store are
// all the ordering needed. Lane l of phase k is on row c-2-l-2k at clock c.
// With requests of clocks up to c = B*(M+2)-1 to make, a reader waits for
// these counts: the state from (G-1, J) was computed 2S-1 clocks later than
// the reader's clock (S phases a group), enters the output ring a clock
// later, is stored in the macro time after that one, by wave waves-1, and is
// seen in the next: (c+2S)/B + waves + 1; the column left of the strip, from
// (G-1, J-1), 64 clocks later; the left strip's last lane is 63 clocks behind
// lane 0: (c+64)/B + 2. The halo slots a time M writes were read 64 clocks
// before. The state is updated in place: (G, J) stores a row at least ten
// times after (G, J-1) read the last column it needs of it, because it waits
// for (G, J-1) to be that far ahead, and (G, J+1) and (G-1, J+1) read only
// columns right of all that (G, J) writes.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "adst.h"
#include "gs_pipe.h"
#include "kernels.h"

namespace adst {
namespace {

// Phases of one launch: bounds the halo buffer's extra strips (a strip moves
// one column per phase) and the number of progress counters.
constexpr int kGpMaxPhases = 256;

// Waves of a workgroup: eight, or four where that still gives every
// workgroup at work at once a CU of its own (one fits a CU by its LDS). Half
// the phases a group make a clock half as long on the CU, which shortens
// the chain of a small grid (400 x 400 f64, T = 100: 1.26 -> 1.08 ms), but
// twice the groups; with more of them at work than CUs the chip is short of
// places (4096 x 4096: 6.7 ms with eight waves, 8.7 with four). A strip starts
// 88 clocks after its left neighbour and works for about ny + 112, so a group
// has a few strips at work at a time. With all its strips counted, wide
// grids of few rows took eight waves (reverse sweeps, eight, four, level
// launches: 64 x 20000 f64, T = 10, 9.2, 6.3, 6.9 ms; 300 x 100000 f32, T = 20,
// 25.5, 19.9, 24.6; 48 x 5000 f64, T = 100, 2.85, 2.01, 5.70); 33 shapes of 48
// to 4000 rows, T = 8 to 200, in both types: none slower.
constexpr int kGpWide = 8, kGpNarrow = 4, kGpCus = 256;

struct GpGeom {
  int64_t ngroups, ncol, nj;
  uint64_t flag_bytes, bytes;  // flags; flags and halo
};

GpGeom gp_geom(const StepShape& s, int nph, int nwaves) {
  GpGeom g{};
  const int64_t isz = s.dtype == ADST_F64 ? 8 : 4, nc = kGpLanes * 16 / isz, S = kGpQ * nwaves;
  g.ngroups = (nph + S - 1) / S;
  for (int64_t k = 0; k < g.ngroups; ++k) {  // as j_lo and j_hi of the kernel
    const int64_t nw = (std::min(S, nph - k * S) + kGpQ - 1) / kGpQ;
    const int64_t lo = k * S / nc, hi = (s.nx - 1 + k * S + nw * kGpQ - 1) / nc;
    g.ncol = std::max(g.ncol, hi - lo + 1);
    g.nj = hi + 1;
  }
  g.flag_bytes = (uint64_t(g.ngroups) * g.ncol + 1) * kGpFlagInts * sizeof(int);
  g.bytes = g.flag_bytes + uint64_t(std::min<int64_t>(2, g.ngroups)) * g.nj * S * uint64_t(s.ny) * isz;
  return g;
}

int gp_waves(const StepShape& s, int nph) {
  const GpGeom g = gp_geom(s, nph, kGpNarrow);
  const int64_t at_work = std::min<int64_t>(g.ncol, (int64_t(s.ny) + 112) / 88 + 2);
  return g.ngroups * at_work <= kGpCus ? kGpNarrow : kGpWide;
}

// Whether launches of up to kGpMaxPhases phases can run the shape; where not,
// the level launches do. The kernel's rows, columns and macro times are
// 32-bit: they reach a few hundred beyond the grid's extent. A launch has
// fewer than 2^32 work-items (HIP refuses more: 3 x 160,000,000 f64 with 100
// phases would have 1.04 of that many).
constexpr int32_t kGpMaxExtent = INT32_MAX - 4 * kGpMaxPhases;
bool gp_fits(const StepShape& s, int nph) {
  if (s.nx > kGpMaxExtent || s.ny > kGpMaxExtent) return false;
  for (const int nw : {kGpNarrow, kGpWide}) {
    const GpGeom g = gp_geom(s, nph, nw);
    if (uint64_t(g.ngroups) * g.ncol * kGpLanes * nw >= (uint64_t(1) << 32)) return false;
  }
  return true;
}

template <class R, bool ADJ>
hipError_t gp_run(const StepShape& s, R* buf, const R* src, int phases, void* scratch,
                  hipStream_t st) {
  for (int ph = 0; ph < phases; ph += kGpMaxPhases) {
    const int n = std::min(kGpMaxPhases, phases - ph), nw = gp_waves(s, n);
    const GpGeom g = gp_geom(s, n, nw);
    const hipError_t z = launch_fill_zero(scratch, (int64_t)g.flag_bytes, st);
    if (z != hipSuccess) return z;
    const GpArgs a{buf, ph == 0 ? src : buf, static_cast<int*>(scratch),
                   static_cast<char*>(scratch) + g.flag_bytes, s.nx, s.ny, n, ph, phases,
                   (int)g.ngroups, (int)g.ncol, (int)g.nj};
    const dim3 grid((unsigned)(g.ngroups * g.ncol)), block(kGpLanes * nw);
    if (nw == kGpNarrow)
      gs_pipe<R, ADJ, kGpNarrow><<<grid, block, 0, st>>>(a, R(s.p0));
    else
      gs_pipe<R, ADJ, kGpWide><<<grid, block, 0, st>>>(a, R(s.p0));
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace

// The halo is two groups' phases by rows for every strip: on wide grids a
// quarter of an f64 state and an eighth of an f32 one with eight waves, half
// that with four (4096 x 4096, T = 100: 34.6 of 134 MB, 4.5 of 67), but a
// strip however narrow the grid is and one more per 128 or 256 phases it has
// moved left by. Grids of fewer than 16 columns would need several states (3
// columns f64, T = 200: 10), and run the level launches beyond this bound
// (1,000,000 rows of 4 f64, T = 20: 210 ms forward as one launch, 258 as
// levels).
uint64_t gp_most_bytes(const StepShape& s) {
  const uint64_t state = uint64_t(s.nx) * s.ny * (s.dtype == ADST_F64 ? 8 : 4);
  return std::max<uint64_t>(2 * state + (64 << 10), 1 << 20);
}

// gp_waves picks eight waves only above some number of phases: a run of
// fewer phases never needs more than this.
uint64_t gs_pipe_bytes(const StepShape& s, int32_t sweeps) {
  if (sweeps <= 0) return 0;
  const int phases = (int)std::min<int64_t>(int64_t(sweeps) + 1, kGpMaxPhases);
  if (!gp_fits(s, phases)) return 0;
  uint64_t bytes = gp_geom(s, phases, kGpNarrow).bytes;
  if (gp_waves(s, phases) == kGpWide) bytes = std::max(bytes, gp_geom(s, phases, kGpWide).bytes);
  return bytes <= gp_most_bytes(s) ? bytes : 0;
}

// Whether a run takes the persistent launch where it has the scratch for it.
// A forward run of a few sweeps may be shorter as levels, in f32 above all,
// where a strip is twice as wide and its clock longer: the launch takes about
// 10 us and, for each of its clocks, 0.24 us in f64 and 0.30 to 0.34 in f32, as
// the rows grow in number (0.21 and 0.26 where it is one strip); a level of
// that few tiles of aligned rows takes 9 us (of others a third more). Forward
// runs as one launch and as levels, us: 5000 x 5000 f32 one sweep 2366 and
// 1978, three 2386 and 2078, eight 2399 and 2488; 2048 x 2048 f32 five 1000 and
// 908; 400 x 400 f32 one 187 and 161, three 189 and 218; 1501 x 2003 f32 one
// 767 and 1046; 32 x 32 f64 one 34 and 29, two 33 and 53; 400 x 400 f64 one 184
// and 207. The reverse sweeps were the faster as one launch at all sizes (0.31
// to 0.97).
bool gs_takes_pipe(const StepShape& s, bool adjoint, int32_t sweeps) {
  const bool f64 = s.dtype == ADST_F64;
  if (adjoint || sweeps > 6 || s.nx % (f64 ? 2 : 4) != 0) return true;
  const int64_t strips = gp_geom(s, 1, kGpNarrow).ncol, clocks = int64_t(s.ny) + 76 + 88 * (strips - 1);
  const double clock = strips == 1 ? (f64 ? 0.21 : 0.26)
                       : f64      ? 0.24
                                  : 0.30 + 0.04 * std::min(1.0, s.ny / 1000.0);
  return 9.0 * double(gs_kernel_launches(s, false, sweeps)) >= 10.0 + clock * double(clocks);
}

GsPipeCost gs_pipe_cost(const StepShape& s, bool adjoint, int32_t sweeps) {
  GsPipeCost c;
  const int64_t isz = s.dtype == ADST_F64 ? 8 : 4, phases = int64_t(sweeps) + (adjoint ? 1 : 0);
  for (int64_t ph = 0; ph < phases; ph += kGpMaxPhases) {
    const int n = (int)std::min<int64_t>(kGpMaxPhases, phases - ph), nw = gp_waves(s, n);
    const GpGeom g = gp_geom(s, n, nw);
    ++c.launches;
    // the state in and out per group; the halo's values written and read once
    c.bytes += 2 * isz * s.ny * (uint64_t(g.ngroups) * s.nx + uint64_t(n) * (g.ncol - 1));
  }
  return c;
}

hipError_t gs_pipe_forward(const StepShape& s, const void* src, void* dst, int32_t sweeps,
                           void* scratch, hipStream_t st) {
  if (s.dtype == ADST_F64)
    return gp_run<double, false>(s, static_cast<double*>(dst), static_cast<const double*>(src),
                                 sweeps, scratch, st);
  return gp_run<float, false>(s, static_cast<float*>(dst), static_cast<const float*>(src), sweeps,
                              scratch, st);
}

hipError_t gs_pipe_adjoint(const StepShape& s, void* g, int32_t sweeps, void* scratch,
                           hipStream_t st) {
  if (s.dtype == ADST_F64)
    return gp_run<double, true>(s, static_cast<double*>(g), static_cast<const double*>(g),
                                sweeps + 1, scratch, st);
  return gp_run<float, true>(s, static_cast<float*>(g), static_cast<const float*>(g), sweeps + 1,
                             scratch, st);
}

}  // namespace adst
