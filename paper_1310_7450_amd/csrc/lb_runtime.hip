// Host runtime and C ABI of lbnlm: parameter resolution, workspace layout,
// strip work lists, captured step graphs, convergence checks, observation
// and state transfer. See include/lb.h for the contract of every entry point.
#include "lb.h"
#include "lb_internal.h"

#include <algorithm>
#include <array>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <limits>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <vector>

using namespace lbnlm;

// Scratch of the allocation-free observation (lb_observe_noalloc): the
// per-strip partials, per-row profiles and per-channel scalars of one
// observation and the gathered result live in this file-scope device array
// instead of the handle's workspace. Each GPU the library runs on holds its
// own copy until the process ends; every call on that GPU shares it.
constexpr size_t kNoallocScratchBytes = size_t(16) << 20;
static __device__ __align__(256) double scratch[kNoallocScratchBytes / sizeof(double)];

namespace {

constexpr int kDefaultK = 1000;
constexpr size_t kAlign = 256;
constexpr size_t kStageNodes = 4096;  // 320 KB
constexpr size_t kHostStressNodes = 1 << 15;  // converted on the host (8 x 4096 FP32: 68 us, on the GPU 143)
#ifndef LB_WG_WAVES
#define LB_WG_WAVES 4
#endif
constexpr int kWaves = LB_WG_WAVES;  // wavefronts (strips) per workgroup


size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// D2Q9 velocities and rest weights, host side (layout conversion only).
constexpr int HCX[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
constexpr int HCY[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
constexpr int HOPP[9] = {0, 3, 4, 1, 2, 7, 8, 5, 6};
inline double hweight(int i) { return i == 0 ? 4.0 / 9.0 : (i < 5 ? 1.0 / 9.0 : 1.0 / 36.0); }

struct Layout {
  long long plane = 0;       // nodes per state buffer (multiple of the tile)
  int esize = 8;             // bytes per element
  int total_rows = 0;
  int total_part = 0;
  int max_strips = 0;
  int n_tiles = 0;  // tiles of the tiled step (stress force, or FP64 strip-class channels)
  size_t off_state[2] = {0, 0}, off_ch = 0, off_strips = 0, off_astrips = 0, off_rstrips = 0, off_part = 0,
         off_prof = 0, off_prev = 0, off_scal = 0, off_uref = 0, bytes = 0;
  size_t off_stress[2] = {0, 0};  // viscoelastic model only
  size_t off_saf_u = 0, off_saf_t = 0;  // stress-as-force scratch (u~, Sigma^nN)
  size_t off_tiles = 0;                 // tiles of the tiled step
  // two steps per launch: strips of the other channels for captured blocks
  // (and their reverse), and the two-step strips
  size_t off_bstrips = 0, off_brstrips = 0, off_tstrips = 0;
  size_t off_blk = 0;     // boxes of the channels that run many steps per launch
  size_t off_gpb = 0, off_gpm = 0;  // boxes of the pressure-driven channels, one and many steps per launch
  // staging of every state of at most kStageNodes, and (FP32) of one where the
  // other buffer holds too few rows of it (see store_state)
  size_t off_stage = 0, stage = 0;
  size_t off_btiles = 0;  // tiles of the tiled channels without two-step strips
  int strip_cap = 0;      // entries of each one-step strip list
  int max_two = 0;
  long long max_boxes = 0;
  std::vector<char> blk_ok;  // how each channel uses boxes (kNoBoxes, kBoxes, kPressureBoxes)
  std::vector<ChanDev> ch;
};

std::string validate(const lb_channel *c, int n, const lb_options *o) {
  if (!c || n <= 0) return "no channels";
  if (!o) return "options are NULL";
  if (o->precision != LB_FP64 && o->precision != LB_FP32_SHIFTED) return "unknown precision";
  if (o->obs_every < 0 || (o->obs_every > 0 && (o->obs_every < 2 || (o->obs_every & 1))))
    return "obs_every must be 0 or an even number >= 2";
  if (o->strip_rows < 0 || o->strip_rows > 4096) return "strip_rows out of range";
  if (!(o->steady_tol >= 0) || !std::isfinite(o->steady_tol)) return "steady_tol must be >= 0";
  if (o->viscoelastic != 0 && o->viscoelastic != 1) return "viscoelastic must be 0 or 1";
  if (o->stress_force != 0 && o->stress_force != 1) return "stress_force must be 0 or 1";
  if (o->steps_per_sweep < 0 || o->steps_per_sweep > 2) return "steps_per_sweep must be 0, 1 or 2";
  if (o->stress_force && (o->precision != LB_FP64 || o->viscoelastic))
    return "stress_force needs FP64 and the instantaneous model";
  for (int i = 0; i < n; ++i) {
    const lb_channel &q = c[i];
    char buf[160];
    auto bad = [&](const char *what) {
      snprintf(buf, sizeof buf, "channel %d: %s", i, what);
      return std::string(buf);
    };
    if (q.nx < 1 || q.ny < 1) return bad("nx and ny must be >= 1");
    if ((long long)q.nx * q.ny > (1LL << 31)) return bad("too many nodes");
    if (!(q.tau_lb > 0.5) || !std::isfinite(q.tau_lb)) return bad("tau_lb must be > 1/2");
    if (!(q.G >= 0) || !std::isfinite(q.G)) return bad("G must be >= 0");
    if (!(q.tau0 > 0)) return bad("tau0 must be > 0");
    if (!(q.gamma_c > 0)) return bad("gamma_c must be > 0");
    if (!std::isfinite(q.force)) return bad("force must be finite");
    if (!std::isfinite(q.eps)) return bad("eps must be finite");
    if (!(q.visc_split >= 0 && q.visc_split <= 1)) return bad("visc_split must be in [0,1]");
    if (q.visc_split > 0 && std::isinf(q.tau0)) return bad("visc_split > 0 needs a finite tau0");
    if (!(std::fabs(q.wall_velocity) < 0.3)) return bad("wall_velocity must be finite with |u_w| < 0.3");
    if (!std::isfinite(q.pressure_gradient)) return bad("pressure_gradient must be finite");
    if (q.nn_pressure != 0 && q.nn_pressure != 1) return bad("nn_pressure must be 0 or 1");
    if (q.top_wall != LB_WALL_HALFWAY && q.top_wall != LB_WALL_ZOU_HE) return bad("unknown top_wall");
    if (q.top_wall == LB_WALL_ZOU_HE && (q.ny < 2 || q.pressure_gradient != 0 || o->stress_force))
      return bad("a Zou-He top wall needs ny >= 2, no pressure_gradient and no stress_force");
    if (q.pressure_gradient != 0 && (q.force != 0 || q.wall_velocity != 0 || q.nx < 2 || q.nn_pressure))
      return bad("pressure_gradient needs force = 0, wall_velocity = 0, nx >= 2 and nn_pressure = 0");
    if (q.pressure_gradient != 0 && o->stress_force) return bad("pressure_gradient is not combined with stress_force");
    if (o->stress_force && q.nn_pressure) return bad("stress_force needs nn_pressure = 0");
    if (o->stress_force && align_up((size_t)q.nx * q.ny, kTile) * kPlanes > 0xffffffffull)
      return bad("stress_force needs nx * ny <= 429,496,704 per channel");
  }
  return "";
}

// Separation closure and viscosity split of the channel parameters.
void resolve(const lb_channel &q, ChanDev &d) {
  const double eta_s = (q.tau_lb - 0.5) / 3.0;
  const double tau = q.tau0 * std::pow(10.0, std::min(q.eps, 0.0) / 0.05);
  const double Ginf = q.G * (1.0 + std::sqrt(std::max(q.eps, 0.0)));
  const double lgt = q.visc_split > 0 ? q.visc_split * Ginf * tau : 0.0;
  const double tau_eff = 0.5 + 3.0 * (eta_s + lgt);
  d.t = 0;
  d.t_startup = q.t_startup;
  d.nx = q.nx;
  d.ny = q.ny;
  d.active = 1;
  d.g = q.force;
  d.omega = 1.0 / tau_eff;
  d.kf = 1.0 - 0.5 / tau_eff;
  d.sp = -4.5 / tau_eff;
  d.G = Ginf;
  d.inv_tau = std::isinf(tau) ? 0.0 : 1.0 / tau;
  d.inv_gc = 1.0 / q.gamma_c;
  d.lgt = lgt;
  d.uw = q.wall_velocity;
  d.gpbc = q.pressure_gradient != 0 ? kGpbcPass : 0;
  d.pd = (q.nx + 1) * q.pressure_gradient;
  d.nnp = q.nn_pressure;
  d.zh = q.top_wall == LB_WALL_ZOU_HE;
}

// Term the pull adds to population i of a top-row node at step t: the link
// reflected at the moving half-way wall during step t - 1 gained
// -2 a c_x u_w / cs2 (a and c of the outgoing population opp(i)); only i = 7,
// 8 are affected (none at a Zou-He wall, which completes them instead).
double wall_pull_term(const lb_channel &q, int i, long long t) {
  const double uw = (q.top_wall == LB_WALL_HALFWAY && t >= 1 && t - 1 < q.t_startup) ? q.wall_velocity : 0.0;
  const int o = HOPP[i];
  return -6.0 * hweight(o) * HCX[o] * uw;
}

int strip_rows_for(int cls, int nx, int ny, int requested) {
  if (is_strip_class(cls)) {
    int s = requested > 0 ? requested : 16;
    return std::max(1, std::min(s, ny));
  }
  const int tyw = 64 / nx;
  int s = requested > 0 ? requested : std::max(64, tyw);
  s = (s + tyw - 1) / tyw * tyw;
  return s;
}

// Strips of one channel in row-band order: the strips of one band of rows
// are consecutive (x neighbours, which share cache lines at their edges,
// land on the same XCD), and bands follow each other upwards.
// With stack set, vector-sweep strips come in stacks of kWaves bands at one
// x, so that one workgroup (one CU) holds vertically adjacent strips, and odd
// bands march against the step's direction: two neighbouring strips then
// reach the rows they share (each one's halo and prefetch overrun) at the
// same time, and the second read hits in cache. That pays while a state
// buffer fits the last-level cache (measured: +1.4 points of HBM peak on
// 4096 x 1024 FP32); on larger states the row-band order of x neighbours is
// faster (-1.3 points with stacks on 16 x 8192 x 2048).
void add_strips(int ci, const ChanDev &d, int esize, int srows, bool stack, std::vector<Strip> &out) {
  const int cls = width_class(d.nx, esize);
  const int w = strip_cols(cls, esize);
  const int nxs = is_strip_class(cls) ? (d.nx + w - 1) / w : 1;
  const int nb = (d.ny + srows - 1) / srows;
  if (cls == kVecClass && stack) {
    for (int b0 = 0; b0 < nb; b0 += kWaves)
      for (int xs = 0; xs < nxs; ++xs)
        for (int b = b0; b < std::min(b0 + kWaves, nb); ++b)
          out.push_back(Strip{ci, xs * w, b * srows, std::min((b + 1) * srows, d.ny), b & 1});
    return;
  }
  for (int b = 0; b < nb; ++b)
    for (int xs = 0; xs < nxs; ++xs)
      out.push_back(Strip{ci, xs * w, b * srows, std::min((b + 1) * srows, d.ny), 0});
}

// Two steps per launch (sweep_vec2_kernel) for the blocks of captured steps:
// vector-class channels without the pressure drive (whose column pass runs
// between steps), with either stress model and any top wall, with blocks a
// multiple of four steps (a block is then an even number of two-step launches
// and returns the state to its buffer, as one-step launches do).
bool two_step_handle(const lb_options *o, int K) {
  return o->steps_per_sweep != 1 && !o->stress_force && K % 4 == 0;
}
bool two_step_channel(const lb_channel &c, int esize) {
  // (a row's slots in 32 bits)
  return width_class(c.nx, esize) == kVecClass && c.pressure_gradient == 0 &&
         align_up((size_t)c.nx, kTile) * kPlanes <= 0xffffffffull;
}
// The widths of 32 and 64 columns of the instantaneous model take two steps per
// launch too (sweep_narrow2_kernel), without the pressure drive.
bool narrow_two_step_channel(const lb_options *o, const lb_channel &c) {
  return !o->viscoelastic && (c.nx == 32 || c.nx == 64) && c.pressure_gradient == 0;
}
// Channels whose steps run in boxes (sweep_block_kernel), many per launch or,
// with the pressure drive, one: with either stress model and any top wall,
// while the handle's channels of the same kind hold few enough nodes. A small
// lattice is bound by the latency of its launches, which boxes take once for
// several steps; a large one by instruction issue, of which the boxes' halos
// cost more than the halos of strips. Measured, us per step, boxes against
// the path they replace:
//  * aligned widths (vector class; two steps per launch): FP32 512 x 512 6.4
//    against 19.4, 1024 x 768 15.8 / 17.9, 1024 x 1024 20.2 / 17.8; FP64
//    1024 x 512 18.0 / 23.8, 1024 x 768 26.4 / 24.2, and about the same with
//    the time-integrated stress;
//  * other widths above 64: FP32 (one step per launch) 200 x 20 2.0 / 14.4,
//    1000 x 300 7.6 / 19.8, 4000 x 2000 181 / 211; FP64 (tiles) 200 x 20
//    2.1 / 6.3, 1000 x 300 11.1 / 12.0, 1000 x 500 18.0 / 16.5, but
//    time-integrated 4000 x 2000 278 / 308;
//  * the pressure drive, one step per launch with the boundary columns in it
//    (FP64): 64 x 32 5.9 / 45 (a strip march and a column pass), 1000 x 320
//    18.8 / 26.0, 1000 x 1000 45 / 67;
//  * narrow widths, whose boxes need no columns beside them: 8 x 64 1.1 / 4.7
//    (FP64 1.4 / 3.9), 256 ragged channels of 8 columns 5.3 / 13.2 (8.4 /
//    22.1), 8 x 262144 18.8 / 40.4; from 32 columns on a box holds few rows:
//    64 x 8192 10.8 / 14.6 (FP64 17.3 / 15.1), 64 x 65536 92 / 73;
//  * the stress as a force (FP64; tiles): 8 x 64 1.9 / 9.9, 143 x 43 3.2 / 7.6,
//    512 x 64 4.4 / 7.9, 1000 x 100 5.7 / 8.5, 512 x 300 8.9 / 10.3, 500 x 500
//    14.1 / 11.8.
// FP64 with the pressure drive, one step per launch: every box at a period's end
// sums whole columns, whose lines are read once for each of them, so that the
// work grows with the height squared, summed over the channels (column_work); the
// column pass takes its channels at the same time. Boxes against strips and the
// pass, us per step: 100 x 5000 174 / 264, 100 x 7500 420 / 353; 16 x 10000 186 /
// 368, 16 x 15800 1775 / 612; 4 x 31600 154 / 340, 4 x 100000 6800 / 980; 12
// channels, the tallest 12 x 19529 and 50 x 4963, the others in boxes and these
// by the pass 904 to 1187, all by the pass 814.
constexpr double kColumnWork = 4e10;
double column_work(const lb_channel &c) {
  return (double)c.ny * std::min(c.nx, 70) * ((double)c.ny * std::min(c.nx, 16));
}
// That holds for launches of several steps. One step per launch leaves a box
// its halo and its loads: above the further limits the one-step sweeps are
// faster, and take blocks whose length leaves a plan one step (K / 2 without a
// divisor that pays) and single steps off the block boundaries. Measured, us
// per step, boxes against one-step sweeps:
//  * such blocks (K = 1006): FP32 aligned 1024 x 500 15.6 / 17.3, 1024 x 700
//    17.4 / 16.5 (time-integrated 1024 x 850 21.7 / 22.6); FP64 aligned 256 x
//    128 4.2 / 5.0, 384 x 256 6.5 / 5.8, other widths 359 x 381 7.1 / 8.5, 500 x
//    450 10.8 / 9.8, but 1000 x 100 6.5 / 5.7;
//  * steps one by one, boxes planned for more: FP32 aligned 1024 x 500 19.0 /
//    18.8, 1024 x 600 20.8 / 18.4 (time-integrated 21.6 / 22.9, 1024 x 700 24.0
//    / 23.1), other widths 2000 x 1000 54.2 / 55.6, 3000 x 1000 78.6 / 62.9, 369 x
//    11206 142 / 149; FP64 aligned 256 x 256 7.6 / 7.8, 384 x 256 8.9 / 8.4, other
//    widths 500 x 300 9.8 / 10.1, 500 x 450 14.0 / 11.6, 1000 x 100 8.7 / 8.1;
//  * short runs of steps off the boundaries, FP32 aligned 1024 x 700 15.7 /
//    17.3, 1024 x 850 18.3 / 17.9; FP64 512 x 512 10.4 / 11.7, 768 x 512 14.8 /
//    13.8 (time-integrated 15.6 / 16.3, 4096 x 120 22.6 / 18.2);
//  * 64 x 16000 FP32 25.9 / 23.0, 64 x 8192 14.9 / 21.3.
// Strips of 64 columns and tiles of 64 x 8 nodes do more than a narrow ragged
// channel needs; up to 96 columns, where they do a quarter more, such channels
// have the limits of several steps throughout (66 x 4000 FP64 12.6 / 16.2, 11 x
// 281389 FP32 79 / 342; 62 x 6605 FP64 time-integrated 25.8 / 17.6), and
// the further limits of the others grow as the sweeps' nodes (63 FP64 channels
// of 4 to 490 rows, 178,921 nodes, 18.2 / 30.2).
// The pressure drive, where a channel's height keeps it to one step per launch:
// the sweeps it competes with are faster on wide channels, the column pass
// slower on tall ones. FP64, all such channels together: 2000 x 64 8.3 / 10.7,
// 4000 x 64 15.5 / 14.6, 2000 x 128 16.7 / 16.8, 8000 x 128 40.3 / 35.0, 4000 x
// 256 40.1 / 39.4, 1000 x 1000 45 / 67, 100 of 64 x 64 26.1 / 23.2; FP32 aligned
// 512 x 512 27.0 / 39.0, 4096 x 200 27.5 / 26.3, 1024 x 1000 65 / 60. Blocks
// that leave short channels one step (FP64, K = 1006): 8000 x 40 16.0 / 16.6,
// 16000 x 40 28.0 / 23.7, 40000 x 24 32.7 / 31.4.
enum BoxKind {
  ALIGNED, OTHER, RAGGED, NARROW, NARROW_WIDE, PRESSURE, PRESSURE_RAGGED, PRESSURE_SHORT, FORCE, BOX_KINDS
};
struct BoxLimits {
  long long steps;      // most nodes of a kind in boxes of several steps,
  long long one;        // in boxes of one step,
  long long call_one;   // in boxes for a single step off the block boundaries,
  long long call;       // or several
};
// The nodes of a kind in a handle, those its sweeps step (whole strips, FP64
// whole tiles), its tallest and widest channel, and whether any is of the vector
// class.
struct BoxNodes {
  long long nodes = 0, swept = 0;
  int tallest = 0, widest = 0;
  bool aligned = false;
};
BoxLimits box_limits(const lb_options *o, int kind, const BoxNodes &all) {
  const bool fp32 = o->precision == LB_FP32_SHIFTED, ve = o->viscoelastic;
  const long long always = std::numeric_limits<long long>::max(), M = 1 << 20;
  auto same = [](long long n) { return BoxLimits{n, n, n, n}; };
  // the limits against the one-step sweeps, by what these step
  auto swept = [&](BoxLimits l) {
    const double f = all.nodes > 0 ? (double)all.swept / all.nodes : 1.0;
    return BoxLimits{l.steps, (long long)(l.one * f), (long long)(l.call_one * f), (long long)(l.call * f)};
  };
  switch (kind) {
    case ALIGNED:
      if (fp32) return ve ? BoxLimits{7 * M / 8, 7 * M / 8, 5 * M / 8, 7 * M / 8}
                          : BoxLimits{7 * M / 8, M / 2, M / 2, 3 * M / 4};
      return swept(BoxLimits{5 * M / 8, 3 * M / 64, 5 * M / 64, ve ? 7 * M / 16 : 5 * M / 16});
    case OTHER: {
      const bool wide = all.widest > 512;
      if (fp32) return swept(BoxLimits{8 * M, 8 * M, wide ? 2 * M : 8 * M, 8 * M});
      const long long steps = ve ? 8 * M : 3 * M / 10;
      return swept(wide ? BoxLimits{steps, M / 16, M / 16, steps}
                        : BoxLimits{steps, 9 * M / 64, 5 * M / 32, steps});
    }
    case RAGGED: return same(fp32 || ve ? 8 * M : 3 * M / 10);
    case NARROW_WIDE:
      if (fp32 && !ve) return BoxLimits{M, 15 * M / 16, 15 * M / 16, M};
      return same(ve ? always : M / 4);
    case PRESSURE: return same(fp32 ? (all.aligned ? 3 * M / 4 : M) : std::min(M, 2000ll * all.tallest));
    case PRESSURE_RAGGED: return same(M);
    case PRESSURE_SHORT:
      return BoxLimits{M, fp32 ? M : std::min(M, std::max(M / 8, 10000ll * all.tallest)), M, M};
    case FORCE:  // (one step, 400 x 400 8.8 / 11.2, 1024 x 147 13.5 / 10.3, 1 x 44747 and 2560 x 9 8.6 / 55)
      return all.widest > 512 && all.swept < 5 * all.nodes / 4 ? BoxLimits{5 * M / 32, M / 16, M / 16, 5 * M / 32}
                                                               : same(5 * M / 32);
    default: return same(always);
  }
}
// A channel with the pressure drive of few enough rows, or small enough for one
// box, for boxes of whole columns.
bool short_pressure(const lb_channel &c) { return c.ny <= 48 || (long long)c.nx * c.ny <= 1024; }
// The kind of a channel, or -1 if no box takes it.
int box_kind(const lb_options *o, const lb_channel &c, int esize) {
  const bool gp = c.pressure_gradient != 0;  // one step per launch in either setting
  if (o->steps_per_sweep == 1 && !gp) return -1;
  const size_t N = (size_t)c.nx * c.ny;
  if (align_up(N, kTile) * kPlanes > 0xffffffffull) return -1;  // 32-bit slots in a channel
  const int cls = width_class(c.nx, esize);
  const bool ragged = is_strip_class(cls) && c.nx <= 96 && (c.nx + 63) / 64 * 64 >= 5 * c.nx / 4;
  return o->stress_force         ? FORCE
         : gp                    ? (short_pressure(c) ? PRESSURE_SHORT : ragged ? PRESSURE_RAGGED : PRESSURE)
         : ragged                ? RAGGED
         : cls == kVecClass      ? ALIGNED
         : is_strip_class(cls)   ? OTHER
         : c.nx > 16             ? NARROW_WIDE
                                 : NARROW;
}
// values of block_channels: not in boxes; many steps per launch; pressure drive
enum { kNoBoxes = 0, kBoxes = 1, kPressureBoxes = 2 };
// The channels whose kind's nodes in the handle do not exceed this limit.
std::vector<char> block_channels(const lb_options *o, const lb_channel *c, int n, int esize,
                                 long long BoxLimits::*limit) {
  std::vector<int> kind(n);
  BoxNodes all[BOX_KINDS];
  auto tall = [&](int i) { return kind[i] == PRESSURE || kind[i] == PRESSURE_RAGGED; };
  double work = 0;
  for (int i = 0; i < n; ++i) {
    kind[i] = box_kind(o, c[i], esize);
    if (tall(i)) work += column_work(c[i]);
  }
  for (int i = 0; i < n; ++i) {
    if (esize == 8 && work > kColumnWork && tall(i)) kind[i] = -1;
    if (kind[i] < 0) continue;
    BoxNodes &k = all[kind[i]];
    k.nodes += (long long)c[i].nx * c[i].ny;
    k.tallest = std::max(k.tallest, c[i].ny);
    k.widest = std::max(k.widest, c[i].nx);
    const int rows = o->stress_force ? kSafTileY : esize == 8 ? kMainTileY : 1;
    k.swept += (long long)((c[i].nx + 63) / 64 * 64) * ((c[i].ny + rows - 1) / rows * rows);
    k.aligned = k.aligned || width_class(c[i].nx, esize) == kVecClass;
  }
  std::vector<char> ok(n, kNoBoxes);
  for (int i = 0; i < n; ++i)
    if (kind[i] >= 0 && all[kind[i]].nodes <= box_limits(o, kind[i], all[kind[i]]).*limit)
      ok[i] = c[i].pressure_gradient != 0 ? kPressureBoxes : kBoxes;
  // with the pressure drive also all kinds together; the short channels stay
  // (42 FP64 channels of two million nodes 340 us per step in the sweeps, with
  // those of up to 96 columns in boxes 477)
  long long pressure = 0;
  for (int i = 0; i < n; ++i)
    if (ok[i] == kPressureBoxes) pressure += (long long)c[i].nx * c[i].ny;
  for (int i = 0; i < n && pressure > 1 << 20; ++i)
    if (ok[i] == kPressureBoxes && kind[i] != PRESSURE_SHORT) ok[i] = kNoBoxes;
  return ok;
}
bool two_step_wall(const lb_channel &c) { return c.top_wall == LB_WALL_ZOU_HE || c.wall_velocity != 0; }
// Stored columns of the two-step strips of a width: at most two_step_cols,
// in multiples of two_step_unit columns, as even as possible.
std::vector<int> two_step_cuts(int nx, int npl, bool fp32) {
  const int U = two_step_unit(fp32), cols = two_step_cols(npl, fp32);
  const int units = nx / U, m = (nx + cols - 1) / cols;
  std::vector<int> x(1, 0);
  for (int i = 0; i < m; ++i) x.push_back(x.back() + U * (units / m + (i < units % m)));
  return x;
}
// Rows per two-step strip: whole rounds of resident strips cost each
// strip's rows plus its four extra rows of step t and about two rows of
// start-up, so the height minimises rounds x (rows + 6) over 16..56 rows.
// From four rounds on, workgroups that finish early let the next ones
// start, so the cost is the strips' rows (each plus 6) over the slots (the
// tallest strips then win: 16 x 8192 x 2048 at 56 rows 108.7-108.9k MLUPS,
// at 50 rows, the whole-round choice, 107.3k).
int two_step_rows(const std::vector<lb_channel> &chans, int npl, bool fp32, int slots) {
  int best = 16;
  double best_cost = 1e300;
  for (int H = 16; H <= kTwoStepMaxRows; ++H) {
    long long S = 0, work = 0;
    for (const lb_channel &c : chans) {
      const long long cuts = (long long)(two_step_cuts(c.nx, npl, fp32).size() - 1), full = c.ny / H, rem = c.ny % H;
      S += cuts * (full + (rem > 0));
      work += cuts * (full * (H + 6) + (rem > 0 ? rem + 6 : 0));
    }
    const double r = (double)S / std::max(slots, 1);
    const double cost = r < 4.0 ? std::ceil(r) * (H + 6) : (double)work / std::max(slots, 1);
    if (S > 0 && cost < best_cost) {
      best_cost = cost;
      best = H;
    }
  }
  return best;
}
// Rows per narrow two-step strip: one height R for every narrow channel
// (1, 2, 4, a multiple of 8 up to 64, or a power of two; a channel's
// strips take it rounded up to its row group), the smallest whose strips
// all fit the GPU's resident workgroups at once (slots), so that the strips
// are as short as one round allows; not above the requested height when
// one is given; within the room left in the strip list. (Measured where the
// kernel took 16 to 256 channels of 8 columns and 32 to 512 rows, which step in
// boxes now: among powers of two this height was the fastest in every case, a
// second round or strips twice as tall costing 10-55% per step; the multiples
// of 8 gained a further 14% with all 256 channels active, at 48 rows against
// 64, and lost 2% with 64 active, at 24 rows against 32.)
// a channel's rows per strip for height R: R rounded up to its row group
int narrow_rows(int R, int nx) {
  const int g = 64 / nx;
  return (std::max(R, g) + g - 1) / g * g;
}
int narrow_two_step_rows(const std::vector<lb_channel> &chans, long long slots, int requested, long long room) {
  // candidate heights: 1, 2, 4, every multiple of 8 up to 64, then powers
  // of two
  std::vector<int> cand = {1, 2, 4};
  for (int m = 8; m <= 64; m += 8) cand.push_back(m);
  for (int R = 128; R <= (1 << 30); R *= 2) {
    cand.push_back(R);
    if (R == (1 << 30)) break;
  }
  int last_fit = 0;  // the tallest height so far within the room
  for (const int R : cand) {
    if (requested > 0 && R > requested && last_fit > 0) return last_fit;
    long long S = 0;
    for (const lb_channel &c : chans) {
      const int rows = narrow_rows(R, c.nx);
      S += (c.ny + rows - 1) / rows;
    }
    if (S > room) continue;
    if (S <= slots) return R;
    last_fit = R;
  }
  return last_fit > 0 ? last_fit : 1 << 30;
}
// Many steps per launch on boxes (sweep_block_kernel): the box shape of one
// channel and the launch's steps and threads.
struct BoxShape {
  int ow, oh;  // box width and height
};
struct BoxPlan {
  int S = 0, threads = 0;  // S = 0: no plan
  std::vector<BoxShape> shape;
};
// Largest boxes whose region (box and a halo of reach S nodes, clipped at the
// walls; none across a box of the whole width) holds at most cap nodes: the
// whole width if that fits, all rows, or cut both ways, whichever repeats the
// fewest halo nodes. False if not even one node fits. With the pressure drive
// a launch of several steps needs whole columns, whose density it takes every
// step: boxes of all rows, in channels of at most 48 (above, most of a region
// is halo) or of one box. Measured with that limit off, FP64 us per step, many
// steps per launch against one: 64 x 32 3.2 / 5.9, 8000 x 20 5.3 / 13.2, 20000
// x 30 22.9 / 47.4, 1000 x 48 4.6 / 6.3, 8 x 64 2.4 / 5.1, but 64 x 64 6.4 /
// 6.8, 500 x 100 8.9 / 7.2, 4000 x 64 20.9 / 15.8.
bool box_shape(const lb_channel &c, int S, int reach, int cap, BoxShape &best) {
  const int h = 2 * reach * S;  // halo nodes in one direction, both sides
  double eff = 0;
  auto even = [](int n, int w) { return (n + (n + w - 1) / w - 1) / ((n + w - 1) / w); };
  auto offer = [&](int ow, int oh) {
    if (ow < 1 || oh < 1) return;
    ow = even(c.nx, std::min(ow, c.nx));
    oh = even(c.ny, std::min(oh, c.ny));
    const long long cw = ow >= c.nx ? c.nx : ow + h, rh = oh >= c.ny ? c.ny : std::min(oh + h, c.ny);
    if (cw * rh > cap) return;
    const double e = (double)ow * oh / (double)(cw * rh);
    if (e > eff) {
      eff = e;
      best = BoxShape{ow, oh};
    }
  };
  const bool columns = c.pressure_gradient != 0 && S > 1;
  if (c.nx <= cap) {
    if ((long long)c.nx * c.ny <= cap) offer(c.nx, c.ny);
    if (!columns) offer(c.nx, cap / c.nx - h);
  }
  if (columns) {
    if (c.ny <= 48) offer(cap / c.ny - h, c.ny);
    return eff > 0;
  }
  if (c.nx <= 64) return eff > 0;  // cutting such a row only adds halo
  if (c.ny <= cap) offer(cap / c.ny - h, c.ny);
  for (int ow = 4; ow + h <= cap; ow += (ow < 32 ? 4 : 16)) offer(ow, cap / (ow + h) - h);
  return eff > 0;
}
// wavefronts of a region at work in step s of S (see the kernel's node order;
// columns: boxes cut by columns alone are in column order)
int box_waves(const lb_channel &c, BoxShape b, int S, int step_reach, int s, bool columns) {
  const int reach = step_reach * (S - s) - 1, halo = 2 * step_reach * S;
  const bool whole = b.ow >= c.nx;
  const int cw = whole ? c.nx : b.ow + halo;
  const int rows = std::min(b.oh + 2 * reach, c.ny);
  if (columns && !whole && std::min(b.oh + halo, c.ny) == c.ny) return ((b.ow + 2 * reach) * c.ny + 63) / 64 + 1;
  return (rows * cw + 63) / 64;
}
void add_boxes(int ci, const lb_channel &c, BoxShape b, bool columns, std::vector<Strip> &out) {
  for (int y0 = 0; y0 < c.ny; y0 += b.oh)
    for (int x0 = 0; x0 < c.nx; x0 += b.ow)
      out.push_back(Strip{ci, x0, y0, std::min(y0 + b.oh, c.ny), columns, std::min(x0 + b.ow, c.nx)});
}
// Orders a list so that its items run in this order all over the GPU, where the
// kernels hand every XCD a contiguous part of it: boxes that sum the columns of a
// tall channel, long next to others, would all share one (28 FP64 channels of 2
// to 4114 rows 140 us per step, spread 69; with fewer boxes than CUs the
// neighbours an XCD's L2 holds count more, 14 of 2 to 921 rows 10.9, spread 13.9).
void spread_over_xcds(std::vector<Strip> &list) {
  const std::vector<Strip> in(list);
  const size_t n = in.size(), q = n >> 3, rem = n & 7;
  for (size_t w = 0; w < n; ++w) {
    const size_t j = w & 7;
    list[j * q + std::min(j, rem) + (w >> 3)] = in[w];
  }
}
long long box_count(const lb_channel &c, BoxShape b) {
  return (long long)((c.nx + b.ow - 1) / b.ow) * ((c.ny + b.oh - 1) / b.oh);
}
// The plan of least estimated time per step. A launch takes, in us,
// launch + rounds (start + S (step + wave v m)) + (S busy V + load R) / CUs
// for its rounds of resident workgroups, v wavefronts per SIMD of the largest
// box at work, m boxes sharing a CU, V wavefronts at work and R wavefronts of
// the regions in all; part/8 of the threads hold the largest region. The
// constants are fitted to 700 launches (one 8 x 64 channel to 1024 x 512 nodes
// and 256 ragged 8-wide channels, S 1 to 20; mean error 12% FP32, 9% FP64): the
// plan picked was within 6% of the best measured one in every case. S divides
// K / 2, so that a captured block is an even number of launches and leaves the
// state in its buffer.
BoxPlan plan_boxes(const std::vector<lb_channel> &chans, int K, bool fp32, bool stress_force, int cus, long long room) {
  BoxPlan best;
  double best_us = 1e300;
  const double launch = fp32 ? 2.7 : 2.0, start = fp32 ? 0.13 : 0.63, step = fp32 ? 0.38 : stress_force ? 0.9 : 0.59,
               wave = fp32 ? 0.29 : stress_force ? 0.6 : 0.47, busy = fp32 ? 0.032 : 0.0, load = fp32 ? 0.2 : 0.22;
  const int reach = stress_force ? 3 : 2;  // nodes a step reaches
  // the channels' shapes, each once with its number
  std::vector<const lb_channel *> shaped;
  std::vector<double> number;
  std::vector<int> which;
  std::map<std::array<int, 3>, int> seen;
  bool pressure = false;
  for (const lb_channel &c : chans) {
    const bool gp = c.pressure_gradient != 0;
    pressure = pressure || gp;
    const auto [it, added] = seen.try_emplace({c.nx, c.ny, gp}, (int)shaped.size());
    if (added) {
      shaped.push_back(&c);
      number.push_back(0);
    }
    which.push_back(it->second);
    number[it->second] += 1;
  }
  struct Fit {
    std::vector<BoxShape> shape;  // by shape of a channel; empty: not every one has a box
    double W = 0, R = 0, V = 0, vmax = 0;
  };
  std::vector<BoxShape> best_shape;
  for (int S = 1; S <= K / 2 && S <= 64; ++S) {  // (beyond 64 a launch's own time no longer counts)
    if ((K / 2) % S) continue;
    std::map<int, Fit> fits;  // by largest region
    for (int th = 256; th <= 1024; th *= 2) {
      const int resident = (fp32 && !pressure ? 24 : 16) * 64 / th;  // workgroups of a CU, by registers
      for (int part : {8, 6, 4, 3, 2}) {
        const auto [it, added] = fits.try_emplace(th * part / 8);
        Fit &f = it->second;
        for (size_t i = 0; added && i < shaped.size(); ++i) {
          const lb_channel &c = *shaped[i];
          BoxShape b;
          if (!box_shape(c, S, reach, th * part / 8, b)) {
            f.shape.clear();
            break;
          }
          f.shape.push_back(b);
          f.W += number[i] * (double)box_count(c, b);
        }
        // (one step per launch goes by rows, but the estimate was fitted so)
        const bool columns = S == 1 || f.W <= kColumnOrderBoxes;
        for (size_t i = 0; added && i < f.shape.size(); ++i) {
          const lb_channel &c = *shaped[i];
          const BoxShape b = f.shape[i];
          const double w = number[i] * (double)box_count(c, b);
          const int v0 = box_waves(c, b, S, reach, 0, columns);
          const double v = 0.5 * (v0 + box_waves(c, b, S, reach, S - 1, columns));
          f.R += w * v0;
          f.V += w * v;
          f.vmax = std::max(f.vmax, v);
        }
        if (f.shape.empty() || f.W > (double)room) continue;
        const double slots = (double)resident * cus, rounds = std::ceil(f.W / slots);
        const double m = f.W <= slots ? std::ceil(f.W / cus) : 1.3;
        const double us =
            (launch + rounds * (start + S * (step + wave * m * f.vmax / 4)) + (S * busy * f.V + load * f.R) / cus) / S;
        if (us < best_us) {
          best_us = us;
          best.S = S;
          best.threads = th;
          best_shape = f.shape;
        }
      }
    }
  }
  for (size_t i = 0; best.S && i < chans.size(); ++i) best.shape.push_back(best_shape[which[i]]);
  return best;
}
// Strips of one channel, band by band. With flip odd bands march against the
// others, so that two neighbouring bands are at their common boundary at the
// same time and read its rows from memory once: for the time-integrated
// model (4096 x 1024, us per step, without and with: FP32 51.9 / 50.0, FP64
// 91.6 / 91.6), not for the others (FP32 41.0 / 41.9, FP64 70.8 / 71.4, though
// 12% and 8% less is read there from beyond the L2).
void add_two_step_strips(int ci, const lb_channel &c, int npl, bool fp32, int H, bool flip, std::vector<Strip> &out) {
  const std::vector<int> x = two_step_cuts(c.nx, npl, fp32);
  for (int y0 = 0; y0 < c.ny; y0 += H)
    for (size_t s = 0; s + 1 < x.size(); ++s)
      out.push_back(Strip{ci, x[s], y0, std::min(y0 + H, c.ny), flip ? (y0 / H) & 1 : 0, x[s + 1]});
}

// The tiled step: the fused stress-force kernel for every channel of a
// stress-force handle; the FP64 tile sweep for FP64 channels of the strip
// classes whose slots fit 32-bit offsets (the others keep the strip sweeps).
#ifndef LB_TILE_SWEEP
#define LB_TILE_SWEEP 1
#endif
struct TileShape {
  int tx, ty;
};
TileShape tile_shape(const lb_options *o) {
  return o->stress_force ? TileShape{kSafTileX, kSafTileY} : TileShape{kMainTileX, kMainTileY};
}
bool tiled(const lb_options *o, const lb_channel &c) {
  if (o->stress_force) return true;
  return LB_TILE_SWEEP && o->precision == LB_FP64 && is_strip_class(width_class(c.nx, 8)) &&
         align_up((size_t)c.nx * c.ny, kTile) * kPlanes <= 0xffffffffull;
}
// Tiles of channel i. The kernels hand each of the 8 XCDs a contiguous run
// of the list: the tile columns of a channel are split into 8 groups, each
// group listed band by band, so that an XCD's tiles have their horizontal
// and vertical neighbours (which share halo populations) on the same L2.
void add_tiles(int i, const lb_channel &c, TileShape ts, std::vector<Strip> &out) {
  const int cols = (c.nx + ts.tx - 1) / ts.tx;
  for (int g = 0; g < 8; ++g)
    for (int y0 = 0; y0 < c.ny; y0 += ts.ty)
      for (int cx = g * cols / 8; cx < (g + 1) * cols / 8; ++cx)
        out.push_back(Strip{i, cx * ts.tx, y0, std::min(y0 + ts.ty, c.ny), 0});
}

// A state buffer larger than the last-level cache: the sweeps stream it
// (nontemporal stores)
bool streamed(const Layout &L) { return (long long)kPlanes * L.plane * L.esize > kNontemporalBytes; }

Layout make_layout(const lb_channel *c, int n, const lb_options *o) {
  Layout L;
  L.esize = (o->precision == LB_FP32_SHIFTED) ? 4 : 8;
  L.ch.resize(n);
  long long node = 0;
  int rows = 0, part = 0, strips = 0;
  for (int i = 0; i < n; ++i) {
    ChanDev &d = L.ch[i];
    resolve(c[i], d);
    d.off = node;
    node += (long long)align_up((size_t)c[i].nx * c[i].ny, 64);
    d.row_off = rows;
    rows += c[i].ny;
    const int cls = width_class(c[i].nx, L.esize);
    const int w = strip_cols(cls, L.esize);
    d.nxs = is_strip_class(cls) ? (c[i].nx + w - 1) / w : 1;
    d.poff = part;
    part += d.nxs * c[i].ny;
    const int srows = strip_rows_for(cls, c[i].nx, c[i].ny, o->strip_rows);
    strips += d.nxs * ((c[i].ny + srows - 1) / srows);
  }
  // room for the active set's smaller strips when few channels are left
  // (fewer than twice the SIMDs of any GPU this runs on, see upload_strips)
  strips = std::max(strips, 4096 + 2 * n);
  L.strip_cap = strips;
  L.plane = (long long)align_up((size_t)std::max<long long>(node, kTile), kTile);
  L.total_rows = rows;
  L.total_part = part;
  L.max_strips = strips;
  size_t at = 0;
  auto take = [&](size_t bytes) {
    size_t p = at;
    at = align_up(at + bytes, kAlign);
    return p;
  };
  const size_t state = (size_t)kPlanes * L.plane * L.esize;
  L.off_state[0] = take(state);
  L.off_state[1] = take(state);
  L.off_ch = take(sizeof(ChanDev) * n);
  L.off_strips = take(sizeof(Strip) * strips);
  L.off_astrips = take(sizeof(Strip) * strips);
  L.off_rstrips = take(sizeof(Strip) * strips);
  L.off_part = take(sizeof(double) * OF_COUNT * part);
  L.off_prof = take(sizeof(double) * OF_COUNT * rows);
  L.off_prev = take(sizeof(double) * rows);
  L.off_scal = take(sizeof(double) * CS_COUNT * n);
  L.off_uref = take(sizeof(float) * rows);
  if (o->viscoelastic) {
    const size_t stress = (size_t)kStressPlanes * L.plane * L.esize;
    L.off_stress[0] = take(stress);
    L.off_stress[1] = take(stress);
  }
  if (o->stress_force) {
    L.off_saf_u = take(sizeof(double) * 2 * L.plane);
    L.off_saf_t = take(sizeof(double) * 3 * L.plane);
  }
  const TileShape ts = tile_shape(o);
  for (int i = 0; i < n; ++i)
    if (tiled(o, c[i])) L.n_tiles += ((c[i].nx + ts.tx - 1) / ts.tx) * ((c[i].ny + ts.ty - 1) / ts.ty);
  L.off_tiles = take(sizeof(Strip) * L.n_tiles);
  L.off_bstrips = take(sizeof(Strip) * strips);
  L.off_brstrips = take(sizeof(Strip) * strips);
  const int min_rows = o->strip_rows > 0 ? std::min(o->strip_rows, 16) : 16;
  const int npl = two_step_npl(L.esize == 4, streamed(L), o->viscoelastic);
  for (int i = 0; i < n && two_step_handle(o, o->obs_every > 0 ? o->obs_every : kDefaultK); ++i)
    if (two_step_channel(c[i], L.esize))
      L.max_two += (int)(two_step_cuts(c[i].nx, npl, L.esize == 4).size() - 1) * ((c[i].ny + min_rows - 1) / min_rows);
  L.off_btiles = take(sizeof(Strip) * std::max(L.n_tiles, 1));
  // boxes of 64 nodes, or 4096 boxes and two per channel, in handles with
  // channels that step in them
  L.blk_ok = block_channels(o, c, n, L.esize, &BoxLimits::steps);
  L.max_boxes = std::max<long long>(4096 + 2ll * n, L.plane / 64);
  auto boxes = [&](char kind) {
    return std::count(L.blk_ok.begin(), L.blk_ok.end(), kind) ? sizeof(Strip) * L.max_boxes : 0;
  };
  L.off_blk = take(boxes(kBoxes));
  L.off_gpb = take(boxes(kPressureBoxes));
  L.off_gpm = take(boxes(kPressureBoxes));
  L.off_tstrips = take(sizeof(Strip) * std::max(L.max_two, 1));
  for (int i = 0; i < n; ++i) {
    const size_t N = (size_t)c[i].nx * c[i].ny;
    const size_t nodes = N <= kStageNodes ? N
                         : L.esize == 4 && c[i].ny < 6 ? (size_t)c[i].nx * std::min(c[i].ny, 3) : 0;
    L.stage = std::max(L.stage, sizeof(double) * kPlanes * nodes);
  }
  L.off_stage = take(L.stage);
  L.bytes = at;
  return L;
}

}  // namespace

struct lb_handle {
  Layout L;
  lb_options opt{};
  int n_ch = 0;
  int K = kDefaultK;
  std::vector<lb_channel> in;
  char *ws = nullptr;
  void *buf[2] = {nullptr, nullptr};
  ChanDev *dch = nullptr;
  Strip *dall = nullptr;     // every channel, for observation
  Strip *dact = nullptr;     // active channels, for stepping
  Strip *dact_rev = nullptr; // the same, each class group in reverse order
  double *dpart = nullptr, *dprof = nullptr, *dprev = nullptr, *dscal = nullptr;
  float *duref = nullptr;    // FP32: reference velocity of every row
  void *sbuf[2] = {nullptr, nullptr};  // viscoelastic model: stress buffers (same parity as buf)
  double *saf_u = nullptr, *saf_t = nullptr;  // stress-as-force scratch
  Strip *tiles = nullptr;                     // tiles of the tiled step (every tiled channel)
  // strips grouped by width class: [begin, begin + count) in the arrays
  int all_begin[kClasses] = {0}, all_count[kClasses] = {0};
  int act_begin[kClasses] = {0}, act_count[kClasses] = {0};
  Strip *dbact = nullptr, *dbact_rev = nullptr;  // captured blocks: active channels without two-step strips
  Strip *dtwo = nullptr;                        // two-step strips of the active channels
  int bact_begin[kClasses] = {0}, bact_count[kClasses] = {0};
  // the active channels that step in boxes
  enum { kMany, kPressure, kPressureMany, kBoxLists };
  struct BoxList {
    Strip *d = nullptr;
    int n = 0, S = 0, threads = 0;  // boxes, steps per launch (0: no list), threads
    BoxPlan all;                    // the plan of all channels of the kind
  };
  BoxList boxes[kBoxLists];  // captured blocks; every other step with the pressure drive; captured blocks with it
  int n_tiles = 0;           // tiles of the one-step tile list
  int only = -1;               // the box list that holds every active channel, if one does,
  bool both = false;           // or whether two hold them
  bool blk_all = false;        // every active channel runs many steps per launch in boxes
  // off the block boundaries boxes take single steps, or several at a time, of
  // the channels that run many steps in them
  bool box_one = false, box_several = false;
  std::vector<char> blk_ok;    // how each channel uses boxes (kNoBoxes, kBoxes, kPressureBoxes)
  int cus = 256;
  // captured blocks: the narrow two-step strips of each width, after the
  // others in dbact
  int n2_begin[kClasses] = {0}, n2_count[kClasses] = {0};
  int two_count = 0;
  bool two_only = false;  // every active channel has two-step strips
  bool two_wall = false;  // some two-step strip's channel has a moving or Zou-He top wall
  Strip *btiles = nullptr;  // captured blocks: tiles of the tiled channels without two-step strips
  int n_btiles = 0;
  bool two_step = false;     // captured blocks pair their steps where eligible
  int slots = 1024;          // two-step strips resident at once on the GPU
  int simds = 1024;          // SIMDs of the GPU (four per CU)
  long long n2slots = 1536;  // narrow two-step strips resident at once
  int cur = 0;               // buffer holding the current state
  hipStream_t stream = nullptr, cap = nullptr;
  bool own_stream = false;
  hipGraphExec_t graph[2] = {nullptr, nullptr};
  bool obs_valid = false;
  std::vector<double> hprof, hscal;
  std::vector<long long> t;  // host mirror of every channel's step
  std::vector<int> active;
  int n_checks = 0;
  int since_block = 0;       // steps since the last block boundary (handle clock)
  bool gpbc_pass = false;    // some channel's pressure drive takes the column pass after every step,
  bool gpbc_boxes = false;   // or after steps launched alone (column_pass_takes)
  bool any_zh = false;       // some channel has a Zou-He top wall
  int device = -1;           // the GPU current at lb_create
  double *noalloc = nullptr; // that GPU's copy of `scratch` (device address)
  hipError_t noalloc_err = hipSuccess;
  std::string err;
};

namespace {

lb_status fail(lb_handle *h, lb_status s, const std::string &msg) {
  if (h) h->err = msg;
  return s;
}

lb_status hipfail(lb_handle *h, hipError_t e, const char *where) {
  return fail(h, LB_EHIP, std::string(where) + ": " + hipGetErrorString(e));
}

#define HIPCHECK(h, call)                                  \
  do {                                                     \
    hipError_t e_ = (call);                                \
    if (e_ != hipSuccess) return hipfail((h), e_, #call);  \
  } while (0)

void group_strips(const std::vector<Strip> &s, const std::vector<ChanDev> &ch, int esize,
                  std::vector<Strip> &out, int begin[kClasses], int count[kClasses]) {
  out.clear();
  out.reserve(s.size());
  std::vector<int> cls(ch.size());
  for (size_t i = 0; i < ch.size(); ++i) cls[i] = width_class(ch[i].nx, esize);
  for (int c = 0; c < kClasses; ++c) {
    begin[c] = (int)out.size();
    if (std::count(cls.begin(), cls.end(), c))
      for (const Strip &x : s)
        if (cls[x.ch] == c) out.push_back(x);
    count[c] = (int)out.size() - begin[c];
  }
}

// captured blocks run some channels many steps per launch
bool many_steps(const lb_handle *h) {
  return h->boxes[lb_handle::kMany].S || h->boxes[lb_handle::kPressureMany].S;
}
// Plan of a box list. With the pressure drive: one step per launch, and as
// many as pay in captured blocks.
BoxPlan box_list_plan(const lb_handle *h, int list, const std::vector<lb_channel> &chans) {
  const bool one = list == lb_handle::kPressure || h->opt.steps_per_sweep == 1;
  return plan_boxes(chans, one ? 2 : h->K, h->L.esize == 4, h->opt.stress_force, h->cus, h->L.max_boxes);
}

lb_status upload_strips(lb_handle *h, bool all) {
  std::vector<Strip> raw, grouped;
  // stacks while a state buffer fits the last-level cache (the stores are
  // then cached, see sweep_args)
  const bool stack = !streamed(h->L);
  // Strip heights of the active set: the requested (or default) ones, all
  // divided alike while the active channels make fewer strips than the GPU
  // has SIMDs (down to a kernel's row group for the narrow widths, 4 rows
  // otherwise), so that a few small channels left still spread over the
  // GPU. A node's arithmetic does not depend on the strip it falls in.
  int div = 1;
  auto rows_of = [&](int i) {
    const ChanDev &d = h->L.ch[i];
    const int cls = width_class(d.nx, h->L.esize);
    const int base = strip_rows_for(cls, d.nx, d.ny, h->opt.strip_rows);
    if (is_strip_class(cls)) return std::max(std::min(base, 4), base / div);
    const int tyw = 64 / d.nx;
    const int r = std::max(tyw, base / div);
    return (r + tyw - 1) / tyw * tyw;
  };
  if (!all) {
    auto count = [&]() {
      long long S = 0;
      for (int i = 0; i < h->n_ch; ++i) {
        if (!h->active[i] || h->blk_ok[i] == kPressureBoxes || tiled(&h->opt, h->in[i])) continue;
        const ChanDev &d = h->L.ch[i];
        const int cls = width_class(d.nx, h->L.esize);
        const int w = strip_cols(cls, h->L.esize);
        S += (long long)(is_strip_class(cls) ? (d.nx + w - 1) / w : 1) * ((d.ny + rows_of(i) - 1) / rows_of(i));
      }
      return S;
    };
    for (long long S = count(); S > 0 && S < h->simds && div < 64;) {
      div *= 2;
      const long long S2 = count();
      if (S2 > h->L.strip_cap) {  // no room
        div /= 2;
        break;
      }
      S = S2;
    }
  }
  for (int i = 0; i < h->n_ch; ++i) {
    if (!all && (!h->active[i] || h->blk_ok[i] == kPressureBoxes || tiled(&h->opt, h->in[i]))) continue;
    const ChanDev &d = h->L.ch[i];
    add_strips(i, d, h->L.esize,
               all ? strip_rows_for(width_class(d.nx, h->L.esize), d.nx, d.ny, h->opt.strip_rows) : rows_of(i),
               stack, raw);
  }
  if (all) {
    group_strips(raw, h->L.ch, h->L.esize, grouped, h->all_begin, h->all_count);
    if (!grouped.empty())
      HIPCHECK(h, hipMemcpyAsync(h->dall, grouped.data(), grouped.size() * sizeof(Strip),
                                 hipMemcpyHostToDevice, h->stream));
  } else {
    group_strips(raw, h->L.ch, h->L.esize, grouped, h->act_begin, h->act_count);
    std::vector<Strip> rev(grouped);
    for (int c = 0; c < kClasses; ++c)
      std::reverse(rev.begin() + h->act_begin[c], rev.begin() + h->act_begin[c] + h->act_count[c]);
    if (!grouped.empty()) {
      HIPCHECK(h, hipMemcpyAsync(h->dact, grouped.data(), grouped.size() * sizeof(Strip),
                                 hipMemcpyHostToDevice, h->stream));
      HIPCHECK(h, hipMemcpyAsync(h->dact_rev, rev.data(), rev.size() * sizeof(Strip), hipMemcpyHostToDevice,
                                 h->stream));
    }
    // captured blocks: two-step strips for the eligible active channels, the
    // one-step strips of the others
    std::vector<Strip> braw, bgrouped, two, n2raw, n2grouped, lists[lb_handle::kBoxLists];
    bool wall = false;
    // boxes of the channels that step in them
    for (int l = 0; l < lb_handle::kBoxLists; ++l) {
      lb_handle::BoxList &list = h->boxes[l];
      list.n = list.S = 0;
      std::vector<lb_channel> chans;
      std::vector<int> ids;
      for (int i = 0; i < h->n_ch; ++i)
        if (h->active[i] && h->blk_ok[i] == (l == lb_handle::kMany ? kBoxes : kPressureBoxes)) {
          chans.push_back(h->in[i]);
          ids.push_back(i);
        }
      if (ids.empty()) continue;
      const BoxPlan p = list.all.shape.size() == ids.size() ? list.all : box_list_plan(h, l, chans);
      if (l == lb_handle::kPressureMany && p.S <= 1) continue;
      if (p.S == 0) return fail(h, LB_ENOMEM, "no box plan fits its workspace");
      std::vector<size_t> order(ids.size());
      for (size_t j = 0; j < ids.size(); ++j) order[j] = j;
      int tallest = 0;
      long long total = 0;
      for (size_t j = 0; j < ids.size(); ++j) {
        tallest = std::max(tallest, chans[j].ny);
        total += box_count(chans[j], p.shape[j]);
      }
      const bool sums = l == lb_handle::kPressure && h->L.esize == 8 && tallest > 256 && ids.size() > 1 && total > h->cus;
      if (sums)
        std::stable_sort(order.begin(), order.end(), [&](size_t a, size_t b) { return chans[a].ny > chans[b].ny; });
      for (size_t j : order)
        add_boxes(ids[j], chans[j], p.shape[j], p.S > 1 && total <= kColumnOrderBoxes, lists[l]);
      if (sums) spread_over_xcds(lists[l]);
      if ((long long)lists[l].size() > h->L.max_boxes) return fail(h, LB_ENOMEM, "box list exceeds its workspace");
      HIPCHECK(h, hipMemcpyAsync(list.d, lists[l].data(), lists[l].size() * sizeof(Strip), hipMemcpyHostToDevice,
                                 h->stream));
      list.S = p.S;
      list.threads = p.threads;
      list.n = (int)lists[l].size();
    }
    h->blk_all = h->both = true;
    h->only = -1;
    for (int i = 0; i < h->n_ch; ++i) {
      if (!h->active[i]) continue;
      if (h->blk_ok[i] == kNoBoxes) h->both = false;
      const int l = h->blk_ok[i] == kBoxes ? lb_handle::kMany : lb_handle::kPressureMany;
      if (h->blk_ok[i] == kNoBoxes || !h->boxes[l].S) h->blk_all = false;
      h->only = h->only < 0 || h->only == l ? l : lb_handle::kBoxLists;
    }
    if (h->only != lb_handle::kBoxLists) h->both = false;
    if (!h->blk_all || h->only == lb_handle::kBoxLists) h->only = -1;
    if (h->two_step || many_steps(h)) {
      const int es = h->L.esize;
      std::vector<lb_channel> elig, nelig;
      for (int i = 0; i < h->n_ch; ++i) {
        if (!h->active[i] || h->blk_ok[i] || !h->two_step) continue;
        if (two_step_channel(h->in[i], es)) elig.push_back(h->in[i]);
        else if (narrow_two_step_channel(&h->opt, h->in[i])) nelig.push_back(h->in[i]);
      }
      const int npl = two_step_npl(es == 4, streamed(h->L), h->opt.viscoelastic);
      const int H = h->opt.strip_rows > 0 ? std::min(h->opt.strip_rows, kTwoStepMaxRows)
                                          : two_step_rows(elig, npl, es == 4, h->slots);
      for (int i = 0; i < h->n_ch; ++i) {
        if (!h->active[i] || h->blk_ok[i]) continue;
        if (h->two_step && two_step_channel(h->in[i], es)) {
          add_two_step_strips(i, h->in[i], npl, es == 4, H, h->opt.viscoelastic, two);
          wall = wall || two_step_wall(h->in[i]);
        } else if (!(h->two_step && narrow_two_step_channel(&h->opt, h->in[i])) && !tiled(&h->opt, h->in[i])) {
          add_strips(i, h->L.ch[i], es, rows_of(i), stack, braw);
        }
      }
      // the narrow ones, in what room the list has left
      if (!nelig.empty()) {
        const int R2 = narrow_two_step_rows(nelig, h->n2slots, h->opt.strip_rows,
                                            h->L.strip_cap - (long long)braw.size());
        for (int i = 0; i < h->n_ch; ++i)
          if (h->active[i] && !h->blk_ok[i] && narrow_two_step_channel(&h->opt, h->in[i]))
            add_strips(i, h->L.ch[i], es, narrow_rows(R2, h->in[i].nx), stack, n2raw);
      }
    }
    group_strips(braw, h->L.ch, h->L.esize, bgrouped, h->bact_begin, h->bact_count);
    std::vector<Strip> brev(bgrouped);
    for (int c = 0; c < kClasses; ++c)
      std::reverse(brev.begin() + h->bact_begin[c], brev.begin() + h->bact_begin[c] + h->bact_count[c]);
    // the narrow two-step strips follow in dbact
    group_strips(n2raw, h->L.ch, h->L.esize, n2grouped, h->n2_begin, h->n2_count);
    for (int c = 0; c < kClasses; ++c) h->n2_begin[c] += (int)bgrouped.size();
    bgrouped.insert(bgrouped.end(), n2grouped.begin(), n2grouped.end());
    if ((long long)bgrouped.size() > h->L.strip_cap) return fail(h, LB_ENOMEM, "block strip list exceeds its workspace");
    if (!bgrouped.empty()) {
      HIPCHECK(h, hipMemcpyAsync(h->dbact, bgrouped.data(), bgrouped.size() * sizeof(Strip), hipMemcpyHostToDevice,
                                 h->stream));
      HIPCHECK(h, hipMemcpyAsync(h->dbact_rev, brev.data(), brev.size() * sizeof(Strip), hipMemcpyHostToDevice,
                                 h->stream));
    }
    if ((int)two.size() > h->L.max_two) return fail(h, LB_ENOMEM, "two-step strip list exceeds its workspace");
    h->two_count = (int)two.size();
    // (an FP64 state of up to 0.8 million nodes goes faster through the tiles:
    // 1024 x 700 22.2 us per step, two per launch 24.2; 1024 x 900 26.9 / 24.7)
    h->two_only = h->two_step && (h->L.esize == 4 || h->opt.viscoelastic || h->L.plane >= 3 << 18);
    for (int i = 0; i < h->n_ch; ++i)
      if (h->active[i] && (h->blk_ok[i] || !two_step_channel(h->in[i], h->L.esize))) h->two_only = false;
    h->two_wall = wall;
    if (!two.empty())
      HIPCHECK(h, hipMemcpyAsync(h->dtwo, two.data(), two.size() * sizeof(Strip), hipMemcpyHostToDevice, h->stream));
    // the host vectors die here: make the copies complete first
    HIPCHECK(h, hipStreamSynchronize(h->stream));
  }
  // the host vector dies here: make the copy complete first
  HIPCHECK(h, hipStreamSynchronize(h->stream));
  return LB_OK;
}

SweepArgs sweep_args(lb_handle *h, const Strip *strips, int begin, int count, int src, int k) {
  SweepArgs a{};
  a.A = h->buf[src];
  a.B = h->buf[src ^ 1];
  a.plane = h->L.plane;
  a.strips = strips + begin;
  a.ch = h->dch;
  a.part = h->dpart;
  a.n_strips = count;
  a.n_wg = (count + kWaves - 1) / kWaves;
  a.k = k;
  a.nt = streamed(h->L);
  a.uref = h->duref;
  a.ve = h->opt.viscoelastic;
  a.zh = h->any_zh;
  a.SA = h->sbuf[src];
  a.SB = h->sbuf[src ^ 1];
  return a;
}

// Enqueues S steps of the channels of a box list, if there are any (from
// buffer src, step offset k).
lb_status enqueue_boxes(lb_handle *h, int which, int src, int k, int S, hipStream_t s) {
  const lb_handle::BoxList &l = h->boxes[which];
  if (!l.n) return LB_OK;
  SweepArgs a = sweep_args(h, l.d, 0, l.n, src, k);
  a.n_wg = l.n;  // one box per workgroup
  const bool fp32 = h->opt.precision == LB_FP32_SHIFTED;
  const bool gpbc = which == lb_handle::kPressureMany || (which == lb_handle::kPressure && !fp32);
  HIPCHECK(h, launch_blocks(fp32, gpbc, h->opt.stress_force, l.threads, a, S, s));
  return LB_OK;
}

// Enqueues two steps of the channels with two-step strips, if there are any
// (from buffer src, step offset k).
lb_status enqueue_two_step(lb_handle *h, int src, int k, hipStream_t s) {
  if (!h->two_count) return LB_OK;
  SweepArgs a = sweep_args(h, h->dtwo, 0, h->two_count, src, k);
  a.wall = h->two_wall;
  a.down = (src == 1);
  a.n_wg = h->two_count;  // one strip per workgroup (a wavefront per stage)
  HIPCHECK(h, launch_two_step(h->opt.precision == LB_FP32_SHIFTED, a, s));
  return LB_OK;
}

// Enqueues what a step of the pressure-driven channels needs beside the sweeps:
// their boxes, unless (boxed) the block takes them many steps at once, and the
// inlet/outlet column pass on the state just written, where the step leaves it.
lb_status enqueue_pressure(lb_handle *h, int src, int k, hipStream_t s, bool boxed) {
  if (!boxed) {
    const lb_status st = enqueue_boxes(h, lb_handle::kPressure, src, k, 1, s);
    if (st != LB_OK) return st;
  }
  if (h->gpbc_pass || (h->gpbc_boxes && !boxed))
    HIPCHECK(h, launch_gpbc(h->opt.precision == LB_FP32_SHIFTED, h->buf[src ^ 1], h->dch, h->n_ch, k, h->duref,
                            boxed, s));
  return LB_OK;
}

// Enqueues the sweeps of one step (source buffer src, step offset k), over
// every active channel or (block) over those without two-step strips.
lb_status enqueue_step(lb_handle *h, int src, int k, hipStream_t s, bool block = false) {
  if (h->opt.stress_force) {
    HIPCHECK(h, launch_saf_fused(static_cast<const double *>(h->buf[src]), static_cast<double *>(h->buf[src ^ 1]),
                                 h->dch, block ? h->btiles : h->tiles, block ? h->n_btiles : h->n_tiles, k,
                                 streamed(h->L), src == 1, s));
    return LB_OK;
  }
  Strip *tl = block ? h->btiles : h->tiles;
  const int ntl = block ? h->n_btiles : h->n_tiles;
  if (ntl) {
    SweepArgs a = sweep_args(h, tl, 0, ntl, src, k);
    a.down = (src == 1);
    HIPCHECK(h, launch_tiles(a, s));
  }
  const int *begin = block ? h->bact_begin : h->act_begin, *count = block ? h->bact_count : h->act_count;
  Strip *fwd = block ? h->dbact : h->dact, *rev = block ? h->dbact_rev : h->dact_rev;
  for (int c = 0; c < kClasses; ++c) {
    if (!count[c]) continue;
    // Serpentine order: steps reading buffer 0 take the strips in order and
    // march them upwards, steps reading buffer 1 take them in reverse and
    // march downwards (flipped strips of a stack the other way in both), so
    // that every step starts on what the previous step wrote last, the
    // likeliest to still sit in the last-level cache (MALL).
    SweepArgs a = sweep_args(h, src == 0 ? fwd : rev, begin[c], count[c], src, k);
    a.down = (src == 1);
    HIPCHECK(h, launch_sweep(h->opt.precision == LB_FP32_SHIFTED, c, false, a, s));
  }
  return enqueue_pressure(h, src, k, s, block && h->boxes[lb_handle::kPressureMany].S);
}

// The observation of the current state: per-row, per-strip partials into
// part, then the per-channel reduction into prof and scal (and, with
// update_residual, the residual history in the workspace).
lb_status enqueue_observe_into(lb_handle *h, double *part, double *prof, double *scal, int update_residual,
                               int steps_since) {
  if (h->opt.stress_force) {
    HIPCHECK(h, launch_saf_observe(static_cast<const double *>(h->buf[h->cur]), h->dch, h->n_ch, h->L.plane,
                                   h->L.total_rows, h->saf_u, h->saf_t, part, h->stream));
  }
  for (int c = 0; c < kClasses && !h->opt.stress_force; ++c) {
    if (!h->all_count[c]) continue;
    SweepArgs a = sweep_args(h, h->dall, h->all_begin[c], h->all_count[c], h->cur, 0);
    a.part = part;
    HIPCHECK(h, launch_sweep(h->opt.precision == LB_FP32_SHIFTED, c, true, a, h->stream));
  }
  HIPCHECK(h, launch_reduce(h->dch, h->n_ch, part, prof, h->dprev, scal, h->duref, update_residual, steps_since,
                            h->stream));
  return LB_OK;
}

lb_status enqueue_observe(lb_handle *h, int update_residual, int steps_since) {
  return enqueue_observe_into(h, h->dpart, h->dprof, h->dscal, update_residual, steps_since);
}

void drop_graphs(lb_handle *h) {
  for (int p = 0; p < 2; ++p)
    if (h->graph[p]) {
      (void)hipGraphExecDestroy(h->graph[p]);
      h->graph[p] = nullptr;
    }
}

// Captures K steps starting from buffer src, followed by the step-counter
// advance, as one graph (K is even, so the state returns to buffer src).
lb_status capture(lb_handle *h, int src) {
  hipGraph_t g = nullptr;
  HIPCHECK(h, hipStreamBeginCapture(h->cap, hipStreamCaptureModeRelaxed));
  lb_status st = LB_OK;
  if (h->two_step || many_steps(h)) {
    // the boxes: K / S launches, an even number
    for (int l : {lb_handle::kMany, lb_handle::kPressureMany}) {
      const int S = h->boxes[l].S;
      for (int k = 0, j = 0; S && k < h->K && st == LB_OK; k += S, ++j)
        st = enqueue_boxes(h, l, src ^ (j & 1), k, S, h->cap);
    }
    // pairs of steps: one two-step launch for the eligible channels (its
    // j-th launch reads buffer src ^ (j & 1) and writes the other one), and
    // the one-step launches of the others
    for (int k = 0; k < h->K && st == LB_OK && !h->blk_all; k += 2) {
      st = enqueue_two_step(h, src ^ ((k / 2) & 1), k, h->cap);
      for (int c = 0; c < kClasses && st == LB_OK; ++c) {
        if (!h->n2_count[c]) continue;
        SweepArgs a = sweep_args(h, h->dbact, h->n2_begin[c], h->n2_count[c], src ^ ((k / 2) & 1), k);
        a.n_wg = h->n2_count[c];  // one strip per workgroup (a wavefront per stage)
        hipError_t e = launch_narrow_two_step(h->opt.precision == LB_FP32_SHIFTED, 1 << c, a, h->cap);
        if (e != hipSuccess) st = hipfail(h, e, "launch_narrow_two_step");
      }
      if (st == LB_OK) st = enqueue_step(h, src, k, h->cap, true);
      if (st == LB_OK) st = enqueue_step(h, src ^ 1, k + 1, h->cap, true);
    }
  } else {
    for (int k = 0; k < h->K && st == LB_OK; ++k) st = enqueue_step(h, src ^ (k & 1), k, h->cap);
  }
  if (st == LB_OK) {
    hipError_t e = launch_advance(h->dch, h->n_ch, h->K, h->cap);
    if (e != hipSuccess) st = hipfail(h, e, "launch_advance");
  }
  hipError_t e = hipStreamEndCapture(h->cap, &g);
  if (st != LB_OK) {
    if (g) (void)hipGraphDestroy(g);
    return st;
  }
  if (e != hipSuccess) return hipfail(h, e, "hipStreamEndCapture");
  e = hipGraphInstantiate(&h->graph[src], g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  if (e != hipSuccess) return hipfail(h, e, "hipGraphInstantiate");
  return LB_OK;
}

lb_status read_observation(lb_handle *h) {
  if (h->obs_valid) return LB_OK;
  lb_status st = enqueue_observe(h, 0, 0);
  if (st != LB_OK) return st;
  h->hprof.resize((size_t)h->L.total_rows * OF_COUNT);
  h->hscal.resize((size_t)h->n_ch * CS_COUNT);
  HIPCHECK(h, hipMemcpyAsync(h->hprof.data(), h->dprof, h->hprof.size() * sizeof(double),
                             hipMemcpyDeviceToHost, h->stream));
  HIPCHECK(h, hipMemcpyAsync(h->hscal.data(), h->dscal, h->hscal.size() * sizeof(double),
                             hipMemcpyDeviceToHost, h->stream));
  HIPCHECK(h, hipStreamSynchronize(h->stream));
  h->obs_valid = true;
  return LB_OK;
}

// Copies channel ch's tiles (and stress tiles) from the current buffer to
// the other one. A frozen channel is no longer swept, so both buffers must
// hold its state: later steps of odd length change which buffer is current.
lb_status mirror_state(lb_handle *h, int ch) {
  const ChanDev &d = h->L.ch[ch];
  const size_t Npad = align_up((size_t)d.nx * d.ny, kTile), es = h->L.esize;
  const size_t off = (size_t)slot(0, d.off) * es;
  HIPCHECK(h, hipMemcpyAsync(static_cast<char *>(h->buf[h->cur ^ 1]) + off,
                             static_cast<const char *>(h->buf[h->cur]) + off, kPlanes * Npad * es,
                             hipMemcpyDeviceToDevice, h->stream));
  return LB_OK;
}
lb_status mirror_stress(lb_handle *h, int ch) {
  if (!h->sbuf[0]) return LB_OK;
  const ChanDev &d = h->L.ch[ch];
  const size_t Npad = align_up((size_t)d.nx * d.ny, kTile), es = h->L.esize;
  const size_t off = (size_t)sslot(0, d.off) * es;
  HIPCHECK(h, hipMemcpyAsync(static_cast<char *>(h->sbuf[h->cur ^ 1]) + off,
                             static_cast<const char *>(h->sbuf[h->cur]) + off, kStressPlanes * Npad * es,
                             hipMemcpyDeviceToDevice, h->stream));
  return LB_OK;
}
lb_status mirror_channel(lb_handle *h, int ch) {
  const lb_status st = mirror_state(h, ch);
  return st == LB_OK ? mirror_stress(h, ch) : st;
}

// Convergence check after a graph: residuals of all channels, freeze the
// converged ones and rebuild the active work list.
lb_status check_steady(lb_handle *h) {
  const int first = (h->n_checks == 0);
  lb_status st = enqueue_observe(h, 1, h->K);
  if (st != LB_OK) return st;
  h->n_checks++;
  h->hscal.resize((size_t)h->n_ch * CS_COUNT);
  h->hprof.resize((size_t)h->L.total_rows * OF_COUNT);
  HIPCHECK(h, hipMemcpyAsync(h->hscal.data(), h->dscal, h->hscal.size() * sizeof(double),
                             hipMemcpyDeviceToHost, h->stream));
  HIPCHECK(h, hipMemcpyAsync(h->hprof.data(), h->dprof, h->hprof.size() * sizeof(double),
                             hipMemcpyDeviceToHost, h->stream));
  HIPCHECK(h, hipStreamSynchronize(h->stream));
  h->obs_valid = true;
  // NaN/Inf first: report it before anything is frozen, so that host and
  // device keep the same active channels and step counters
  for (int i = 0; i < h->n_ch; ++i)
    if (h->active[i] && h->hscal[(size_t)i * CS_COUNT + CS_NAN] != 0.0) {
      char buf[96];
      snprintf(buf, sizeof buf, "NaN/Inf seen in channel %d during a convergence check", i);
      return fail(h, LB_EUNSTABLE, buf);
    }
  bool changed = false;
  for (int i = 0; i < h->n_ch; ++i) {
    if (!h->active[i]) continue;
    const double *s = &h->hscal[(size_t)i * CS_COUNT];
    if (!first && s[CS_RESIDUAL] < h->opt.steady_tol) {
      h->active[i] = 0;
      h->L.ch[i].active = 0;
      changed = true;
      lb_status m = mirror_channel(h, i);
      if (m != LB_OK) return m;
    }
  }
  if (changed) {
    // publish the active flags and the new work list, then recapture
    std::vector<ChanDev> cur(h->n_ch);
    HIPCHECK(h, hipMemcpyAsync(cur.data(), h->dch, sizeof(ChanDev) * h->n_ch, hipMemcpyDeviceToHost, h->stream));
    HIPCHECK(h, hipStreamSynchronize(h->stream));
    for (int i = 0; i < h->n_ch; ++i) cur[i].active = h->active[i];
    HIPCHECK(h, hipMemcpyAsync(h->dch, cur.data(), sizeof(ChanDev) * h->n_ch, hipMemcpyHostToDevice, h->stream));
    HIPCHECK(h, hipStreamSynchronize(h->stream));
    lb_status u = upload_strips(h, false);
    if (u != LB_OK) return u;
    drop_graphs(h);
  }
  return LB_OK;
}

// FP32 storage: moves every active row's reference velocity to its current
// mean u_x. Needs the observation of the current state in dprof (taken here
// unless the convergence check just took it).
lb_status rereference(lb_handle *h, bool observed) {
  if (h->opt.precision != LB_FP32_SHIFTED) return LB_OK;
  if (!observed) {
    lb_status st = enqueue_observe(h, 0, 0);
    if (st != LB_OK) return st;
  }
  HIPCHECK(h, launch_rereference(static_cast<float *>(h->buf[h->cur]), h->dch, h->n_ch, h->L.total_rows, h->dprof,
                                 h->duref, h->stream));
  return LB_OK;
}

// ---- state and stress between the storage and the layout of the C ABI -----
//
// lb_get_state, lb_set_state, lb_set_profile and the stress calls convert on
// the GPU; what crosses the host link is the caller's FP64 array, staged in
// the other state buffer, which mirror_state then makes equal to the current
// one again (small states in an area of their own; a small stress is read
// through the host). The link bounds it: the copies of the 24 MB of
// 1000 x 300 nodes take 0.7 ms in and 1.4 ms out (pageable memory). Set, 200
// FP32 steps and read take 5.4 ms there, with host loops over the nodes 24.1.
// Every value is formed by the operations, in the order, of the definition in
// FP64 (no contraction).

__device__ __forceinline__ double weight(int i) { return i == 0 ? 4.0 / 9.0 : (i < 5 ? 1.0 / 9.0 : 1.0 / 36.0); }
// E_i(u) of the FP32 storage: the velocity part of the equilibrium at
// density 1, a_i (3 c_ix u + (9/2 c_ix^2 - 3/2) u^2).
__device__ __forceinline__ double ref_eq(int i, double u) {
#pragma clang fp contract(off)
  const double cx = HCX[i];
  return weight(i) * (3.0 * cx * u + (4.5 * cx * cx - 1.5) * u * u);
}
// What a layout conversion has to know of its channel.
struct StateArgs {
  int nx, ny;
  int zh;                // top wall: Zou-He, with the wall velocity and force of the step
  double uw, fx;
  double wall[3];        // what the pull adds to a top-row node's populations 4, 7 and 8
};
__device__ __forceinline__ double wall_term(const StateArgs &a, int i) { return a.wall[i == 4 ? 0 : i - 6]; }
// Zou-He completion (the steps' zou_he_top) of a top-row node: no flow
// through the wall, n4 = n2, and the diagonals such that (m + f/2)/s is the
// wall velocity.
__device__ __forceinline__ void complete_top(const StateArgs &a, double f[9]) {
#pragma clang fp contract(off)
  const double s = (f[0] + f[1] + f[3]) + 2.0 * (f[2] + f[5] + f[6]);
  const double d87 = (s * a.uw - 0.5 * a.fx) - ((f[1] - f[3]) + (f[5] - f[6]));
  f[4] = f[2];
  f[8] = 0.5 * ((f[5] + f[6]) + d87);
  f[7] = 0.5 * ((f[5] + f[6]) - d87);
}

// Planes [p0, p1) of the state (populations after the pull; 9 is the previous
// trace), FP64, plane by plane at out, one node per thread. src: the
// channel's first slot; uref: the reference velocity of its rows (FP32).
template <typename T>
__global__ void unpack_state_kernel(const T *__restrict__ src, const float *__restrict__ uref,
                                    double *__restrict__ out, StateArgs a, int p0, int p1) {
#pragma clang fp contract(off)
  const long long N = (long long)a.nx * a.ny, id = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (id >= N) return;
  const int y = (int)(id / a.nx), x = (int)(id - (long long)y * a.nx);
  // FP32 slots hold n - a_i - E_i(u_ref) of the row the slot belongs to
  auto at = [&](int p, int xs, int ys) -> double {
    const double v = src[slot(p, (long long)ys * a.nx + xs)];
    return sizeof(T) == 4 ? v + weight(p) + ref_eq(p, uref[ys]) : v;
  };
  const bool top = a.zh && y == a.ny - 1;
  double f[9];
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    f[i] = 0;
    if (!top && (i < p0 || i >= p1)) continue;
    const int ys = y - HCY[i];
    int xs = x - HCX[i];
    xs = xs < 0 ? a.nx - 1 : (xs >= a.nx ? 0 : xs);
    if (ys < 0)
      f[i] = at(HOPP[i], x, y);
    else if (ys >= a.ny)
      f[i] = at(HOPP[i], x, y) + wall_term(a, i);
    else
      f[i] = at(i, xs, ys);
  }
  if (top) complete_top(a, f);
#pragma unroll
  for (int i = 0; i < 9; ++i)
    if (i >= p0 && i < p1) out[(i - p0) * N + id] = f[i];
  if (p1 == 10) out[(9 - p0) * N + id] = src[slot(9, id)];
}

// Stores rows [r0, r1) of a state, a row at a time per workgroup: every slot
// from the (node, population) it feeds (the inverse of the pull). src: rows
// [s0, s0 + srows) of the ten planes, plane by plane; one column stands for
// all if !cols. A Zou-He top wall replaces what enters its row from above.
// FP32: the row's reference velocity becomes the row mean of u_x (0 where
// that is not a finite velocity), summed from x = 0 on. Starts the channel's
// residual history anew and sets its step counter.
template <typename T>
__global__ void pack_state_kernel(T *__restrict__ dst, const double *__restrict__ src, StateArgs a, int r0, int r1,
                                  int s0, int srows, int cols, float *__restrict__ uref, double *__restrict__ prev,
                                  long long *__restrict__ step, long long t) {
#pragma clang fp contract(off)
  __shared__ double su[256];
  const long long width = cols ? a.nx : 1, plane = width * srows;
  auto at = [&](int p, int x, int ys) { return src[p * plane + (ys - s0) * width + (cols ? x : 0)]; };
  for (int y = r0 + (int)blockIdx.x; y < r1; y += gridDim.x) {
    const bool top = y == a.ny - 1;
    auto node = [&](int x, double f[9]) {
#pragma unroll
      for (int i = 0; i < 9; ++i) f[i] = at(i, x, y);
      if (a.zh && top) complete_top(a, f);
    };
    float ur = 0.0f;
    if constexpr (sizeof(T) == 4) {
      double sum = 0;
      for (int x0 = 0; x0 < a.nx; x0 += blockDim.x) {
        const int x = x0 + (int)threadIdx.x;
        if (x < a.nx) {
          double f[9], rho = 0, jx = 0;
          node(x, f);
#pragma unroll
          for (int i = 0; i < 9; ++i) {
            rho += f[i];
            jx += HCX[i] * f[i];
          }
          su[threadIdx.x] = jx / rho;
        }
        __syncthreads();
        const int n = min((int)blockDim.x, a.nx - x0);
        for (int k = 0; k < n; ++k) sum += su[k];
        __syncthreads();
      }
      const double u = sum / a.nx;
      if (isfinite(u) && fabs(u) <= 1.0) ur = (float)u;
      if (threadIdx.x == 0) uref[y] = ur;
    }
    if (threadIdx.x == 0) {
      prev[y] = __longlong_as_double(0x7ff8000000000000ll);
      if (y == 0) *step = t;
    }
    for (int x = threadIdx.x; x < a.nx; x += blockDim.x) {
      const long long id = (long long)y * a.nx + x;
      double f[9];
      node(x, f);
#pragma unroll
      for (int j = 0; j < 9; ++j) {
        const int yd = y + HCY[j];
        int xd = x + HCX[j];
        xd = xd < 0 ? a.nx - 1 : (xd >= a.nx ? 0 : xd);
        double v;
        if (yd < 0)
          v = f[HOPP[j]];
        else if (yd >= a.ny)
          v = f[HOPP[j]] - wall_term(a, HOPP[j]);
        else
          v = at(j, xd, yd);
        dst[slot(j, id)] = sizeof(T) == 4 ? (T)(v - weight(j) - ref_eq(j, ur)) : (T)v;
      }
      dst[slot(9, id)] = (T)at(9, x, y);
    }
  }
}

// The stored stress to and from the C ABI's layout.
template <typename T>
__global__ void unpack_stress_kernel(const T *__restrict__ src, double *__restrict__ out, long long N) {
  const long long id = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (id >= N) return;
  for (int p = 0; p < kStressPlanes; ++p) out[p * N + id] = src[sslot(p, id)];
}
template <typename T>
__global__ void pack_stress_kernel(T *__restrict__ dst, const double *__restrict__ in, long long N) {
  const long long id = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (id >= N) return;
  for (int p = 0; p < kStressPlanes; ++p) dst[sslot(p, id)] = (T)in[p * N + id];
}

StateArgs state_args(const lb_handle *h, int ch, long long t) {
  const ChanDev &d = h->L.ch[ch];
  const lb_channel &q = h->in[ch];
  return StateArgs{d.nx, d.ny, d.zh, t < q.t_startup ? q.wall_velocity : 0.0, t < q.t_startup ? q.force : 0.0,
                   {wall_pull_term(q, 4, t), wall_pull_term(q, 7, t), wall_pull_term(q, 8, t)}};
}

// lb_set_state from pops[9][ny][width] and P[ny][width], where one column
// (width 1) stands for all. As many rows at a time as the staging holds, with
// the rows next to them.
lb_status store_state(lb_handle *h, int ch, const double *pops, const double *P, bool cols, long long t) {
  const ChanDev &d = h->L.ch[ch];
  const int es = h->L.esize;
  const size_t width = cols ? d.nx : 1, N = width * d.ny, Npad = align_up((size_t)d.nx * d.ny, kTile);
  char *dst = static_cast<char *>(h->buf[h->cur]) + (size_t)slot(0, d.off) * es;
  char *other = static_cast<char *>(h->buf[h->cur ^ 1]) + (size_t)slot(0, d.off) * es;
  const size_t row = sizeof(double) * kPlanes * width, other_rows = kPlanes * Npad * es / row,
               stage_rows = h->L.stage / row;
  double *stage = reinterpret_cast<double *>(other_rows >= (size_t)d.ny || other_rows >= stage_rows
                                                 ? other : h->ws + h->L.off_stage);
  const int cap = (int)std::min<size_t>(std::max(other_rows, stage_rows), d.ny);
  if (cap < d.ny && cap < 3) return fail(h, LB_ENOMEM, "no room to stage a row of the state");
  const int step = cap == d.ny ? d.ny : cap - 2;
  const StateArgs a = state_args(h, ch, t);
  const unsigned threads = (unsigned)std::min<size_t>(256, align_up(d.nx, 64));
  for (int r0 = 0; r0 < d.ny; r0 += step) {
    const int r1 = std::min(r0 + step, d.ny), s0 = std::max(r0 - 1, 0), srows = std::min(r1 + 1, d.ny) - s0;
    const size_t plane = width * srows;
    if (srows == d.ny) {
      HIPCHECK(h, hipMemcpyAsync(stage, pops, sizeof(double) * 9 * N, hipMemcpyHostToDevice, h->stream));
    } else {
      for (int i = 0; i < 9; ++i)
        HIPCHECK(h, hipMemcpyAsync(stage + i * plane, pops + i * N + s0 * width, sizeof(double) * plane,
                                   hipMemcpyHostToDevice, h->stream));
    }
    HIPCHECK(h, hipMemcpyAsync(stage + 9 * plane, P + s0 * width, sizeof(double) * plane, hipMemcpyHostToDevice,
                               h->stream));
    auto pack = [&](auto *to) {
      hipLaunchKernelGGL(pack_state_kernel, dim3(std::min(r1 - r0, 1 << 20)), dim3(threads), 0, h->stream, to,
                         static_cast<const double *>(stage), a, r0, r1, s0, srows, (int)cols, h->duref + d.row_off,
                         h->dprev + d.row_off, &h->dch[ch].t, t);
    };
    if (es == 8)
      pack(reinterpret_cast<double *>(dst));
    else
      pack(reinterpret_cast<float *>(dst));
    HIPCHECK(h, hipGetLastError());
  }
  // both buffers: a frozen channel is read from whichever is current later
  const lb_status m = mirror_channel(h, ch);
  if (m != LB_OK) return m;
  HIPCHECK(h, hipStreamSynchronize(h->stream));
  h->t[ch] = t;
  h->obs_valid = false;
  return LB_OK;
}

lb_status fill_rest(lb_handle *h, int which);

// Device address of `scratch` on GPU dev, looked up once per device (with
// that device current, as the caller of lb_create leaves it) and kept for
// the life of the process. In host code the array's name is only a stand-in
// for the symbol: kernels and copies take this address.
constexpr int kMaxDevices = 64;
std::mutex g_noalloc_mu;
double *g_noalloc[kMaxDevices] = {};

hipError_t noalloc_scratch(int dev, double **out) {
  std::lock_guard<std::mutex> lock(g_noalloc_mu);
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  if (!g_noalloc[dev]) {
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_noalloc[dev] = static_cast<double *>(p);
  }
  *out = g_noalloc[dev];
  return hipSuccess;
}

// Observable `what` of channel c as lb_observe reports it, from the reduced
// profiles (prof, [row][OF_COUNT]) or scalars (scal, [channel][CS_COUNT]),
// into out (ny doubles, or one). One thread per row.
__global__ void gather_observable_kernel(const ChanDev *ch, int c, int what, const double *prof,
                                         const double *scal, double *out) {
  const ChanDev d = ch[c];
  const int y = blockIdx.x * blockDim.x + threadIdx.x;
  if (what >= 32) {
    if (y != 0) return;
    const double *s = scal + (long long)c * CS_COUNT;
    double v = 0.0;
    switch (what) {
      case LB_OBS_MASS: v = (double)((long long)d.nx * d.ny) + s[CS_MASS_DEV]; break;
      case LB_OBS_MOMX: v = s[CS_MOMX]; break;
      case LB_OBS_FLUX: v = s[CS_FLUX]; break;
      case LB_OBS_WALL_DRAG: v = s[CS_DRAG]; break;
      case LB_OBS_UMID: v = s[CS_UMID]; break;
      case LB_OBS_NAN: v = s[CS_NAN]; break;
      default: break;
    }
    out[0] = v;
    return;
  }
  if (y >= d.ny) return;
  const double *r = prof + ((long long)d.row_off + y) * OF_COUNT;
  double v = 0.0;
  switch (what) {
    case LB_OBS_UX: v = r[OF_UX]; break;
    case LB_OBS_UY: v = r[OF_UY]; break;
    case LB_OBS_SXX: v = r[OF_SXX]; break;
    case LB_OBS_SXY: v = r[OF_SXY]; break;
    case LB_OBS_SYY: v = r[OF_SYY]; break;
    case LB_OBS_N1: v = r[OF_SXX] - r[OF_SYY]; break;
    case LB_OBS_PRESSURE: v = (1.0 + r[OF_RHOE_DEV]) / 3.0; break;
    case LB_OBS_KXY: v = r[OF_KXY]; break;
    case LB_OBS_TRT: v = r[OF_TRT]; break;
    case LB_OBS_KXX: v = r[OF_KXX]; break;
    default: break;
  }
  out[y] = v;
}

}  // namespace

extern "C" {

const char *lb_status_string(int32_t s) {
  switch (s) {
    case LB_OK: return "LB_OK";
    case LB_EINVAL: return "LB_EINVAL";
    case LB_ENOMEM: return "LB_ENOMEM";
    case LB_EHIP: return "LB_EHIP";
    case LB_EUNSTABLE: return "LB_EUNSTABLE";
    case LB_ESTATE: return "LB_ESTATE";
    default: return "unknown status";
  }
}

const char *lb_last_error(const lb_handle *h) { return h ? h->err.c_str() : "NULL handle"; }

lb_status lb_workspace_bytes(const lb_channel *c, int32_t n, const lb_options *o, size_t *bytes) {
  if (!bytes) return LB_EINVAL;
  if (!validate(c, n, o).empty()) return LB_EINVAL;
  *bytes = make_layout(c, n, o).bytes;
  return LB_OK;
}

lb_status lb_create(const lb_channel *c, int32_t n, const lb_options *o, void *ws, size_t ws_bytes,
                    void *stream, lb_handle **out) {
  if (!out) return LB_EINVAL;
  *out = nullptr;
  if (!validate(c, n, o).empty()) return LB_EINVAL;
  if (!ws || (reinterpret_cast<uintptr_t>(ws) % kAlign)) return LB_EINVAL;
  lb_handle *h = new (std::nothrow) lb_handle();
  if (!h) return LB_ENOMEM;
  h->L = make_layout(c, n, o);
  if (ws_bytes < h->L.bytes) {
    delete h;
    return LB_ENOMEM;
  }
  h->opt = *o;
  h->n_ch = n;
  for (int i = 0; i < n; ++i) {
    h->any_zh = h->any_zh || h->L.ch[i].zh;
  }
  h->K = o->obs_every > 0 ? o->obs_every : kDefaultK;
  h->in.assign(c, c + n);
  h->ws = static_cast<char *>(ws);
  h->buf[0] = h->ws + h->L.off_state[0];
  h->buf[1] = h->ws + h->L.off_state[1];
  h->dch = reinterpret_cast<ChanDev *>(h->ws + h->L.off_ch);
  h->tiles = reinterpret_cast<Strip *>(h->ws + h->L.off_tiles);
  h->dall = reinterpret_cast<Strip *>(h->ws + h->L.off_strips);
  h->dact = reinterpret_cast<Strip *>(h->ws + h->L.off_astrips);
  h->dact_rev = reinterpret_cast<Strip *>(h->ws + h->L.off_rstrips);
  h->dbact = reinterpret_cast<Strip *>(h->ws + h->L.off_bstrips);
  h->dbact_rev = reinterpret_cast<Strip *>(h->ws + h->L.off_brstrips);
  h->dtwo = reinterpret_cast<Strip *>(h->ws + h->L.off_tstrips);
  h->btiles = reinterpret_cast<Strip *>(h->ws + h->L.off_btiles);
  h->boxes[lb_handle::kMany].d = reinterpret_cast<Strip *>(h->ws + h->L.off_blk);
  h->boxes[lb_handle::kPressure].d = reinterpret_cast<Strip *>(h->ws + h->L.off_gpb);
  h->boxes[lb_handle::kPressureMany].d = reinterpret_cast<Strip *>(h->ws + h->L.off_gpm);
  h->two_step = false;
  for (int i = 0; i < n && two_step_handle(o, h->K); ++i)
    h->two_step = h->two_step || two_step_channel(c[i], h->L.esize) || narrow_two_step_channel(o, c[i]);
  h->dpart = reinterpret_cast<double *>(h->ws + h->L.off_part);
  h->dprof = reinterpret_cast<double *>(h->ws + h->L.off_prof);
  h->dprev = reinterpret_cast<double *>(h->ws + h->L.off_prev);
  h->dscal = reinterpret_cast<double *>(h->ws + h->L.off_scal);
  h->duref = reinterpret_cast<float *>(h->ws + h->L.off_uref);
  if (o->viscoelastic) {
    h->sbuf[0] = h->ws + h->L.off_stress[0];
    h->sbuf[1] = h->ws + h->L.off_stress[1];
  }
  if (o->stress_force) {
    h->saf_u = reinterpret_cast<double *>(h->ws + h->L.off_saf_u);
    h->saf_t = reinterpret_cast<double *>(h->ws + h->L.off_saf_t);
  }
  h->t.assign(n, 0);
  h->active.assign(n, 1);
  auto bail = [&](lb_status s) {
    if (h->cap) (void)hipStreamDestroy(h->cap);
    if (h->own_stream && h->stream) (void)hipStreamDestroy(h->stream);
    delete h;
    return s;
  };
  if (stream) {
    h->stream = static_cast<hipStream_t>(stream);
  } else {
    if (hipStreamCreateWithFlags(&h->stream, hipStreamNonBlocking) != hipSuccess) return bail(LB_EHIP);
    h->own_stream = true;
  }
  if (hipStreamCreateWithFlags(&h->cap, hipStreamNonBlocking) != hipSuccess) return bail(LB_EHIP);
  {
    // strips of the two-step sweep resident at once
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
      return bail(LB_EHIP);
    // four and more strips on a CU in even numbers: each is two wavefronts, and
    // an odd one leaves two SIMDs with a wavefront more than the others
    // (time-integrated FP32, 4096 x 1024: five strips 54.5 us, four 52.0)
    int per_cu = two_step_blocks_per_cu(o->precision == LB_FP32_SHIFTED, streamed(h->L), o->viscoelastic);
    if (per_cu >= 4) per_cu &= ~1;
    h->slots = per_cu * std::max(cus, 1);
    h->simds = 4 * std::max(cus, 1);
    h->cus = std::max(cus, 1);
    h->n2slots = (long long)narrow_two_step_blocks_per_cu(o->precision == LB_FP32_SHIFTED) * std::max(cus, 1);
  }
  // channels that step in boxes; where blocks leave a kind's plan one step,
  // those within its limit
  h->blk_ok = h->L.blk_ok;
  const std::vector<char> one = block_channels(o, c, n, h->L.esize, &BoxLimits::one);
  auto plan = [&](int l) -> BoxPlan & {
    const char kind = l == lb_handle::kMany ? kBoxes : kPressureBoxes;
    std::vector<lb_channel> chans;
    for (int i = 0; i < n; ++i)
      if (h->blk_ok[i] == kind) chans.push_back(c[i]);
    // (a plan for all is one for those still active later)
    BoxPlan &p = h->boxes[l].all;
    p = chans.empty() ? BoxPlan() : box_list_plan(h, l, chans);
    return p;
  };
  for (int l : {lb_handle::kMany, lb_handle::kPressureMany}) {
    const char kind = l == lb_handle::kMany ? kBoxes : kPressureBoxes;
    if (plan(l).S > 1) continue;
    for (int i = 0; i < n; ++i)
      if (h->blk_ok[i] == kind) h->blk_ok[i] = one[i];
    plan(l);
  }
  plan(lb_handle::kPressure);
  for (char &k : h->blk_ok)
    if ((k == kBoxes && !h->boxes[lb_handle::kMany].all.S) ||
        (k == kPressureBoxes && !h->boxes[lb_handle::kPressure].all.S))
      k = kNoBoxes;
  {
    const std::vector<char> single = block_channels(o, c, n, h->L.esize, &BoxLimits::call_one),
                            several = block_channels(o, c, n, h->L.esize, &BoxLimits::call);
    // (a handle of several kinds steps in as many sweeps: boxes unless those
    // within no limit hold three quarters of the nodes. 26 FP64 channels 1 to
    // 14923 wide, 62%, step by step 53 us, in sweeps 213)
    double in_boxes = 0, beyond_one = 0, beyond_several = 0;
    for (int i = 0; i < n; ++i)
      if (h->blk_ok[i] == kBoxes) {
        const double nodes = (double)c[i].nx * c[i].ny;
        in_boxes += nodes;
        if (!single[i]) beyond_one += nodes;
        if (!several[i]) beyond_several += nodes;
      }
    h->box_one = beyond_one < 0.75 * in_boxes;
    h->box_several = beyond_several < 0.75 * in_boxes;
  }
  for (int i = 0; i < n; ++i) {
    ChanDev &d = h->L.ch[i];
    if (d.gpbc && h->blk_ok[i] == kPressureBoxes) d.gpbc = h->L.esize == 8 ? kGpbcStep : kGpbcBoxes;
    h->gpbc_pass = h->gpbc_pass || d.gpbc == kGpbcPass;
    h->gpbc_boxes = h->gpbc_boxes || d.gpbc == kGpbcBoxes;
  }
  if (hipMemcpyAsync(h->dch, h->L.ch.data(), sizeof(ChanDev) * n, hipMemcpyHostToDevice, h->stream) !=
      hipSuccess)
    return bail(LB_EHIP);
  std::vector<double> nanrows(std::max(1, h->L.total_rows), std::numeric_limits<double>::quiet_NaN());
  if (hipMemcpyAsync(h->dprev, nanrows.data(), sizeof(double) * h->L.total_rows, hipMemcpyHostToDevice,
                     h->stream) != hipSuccess)
    return bail(LB_EHIP);
  std::vector<float> zrows(std::max(1, h->L.total_rows), 0.0f);
  if (hipMemcpyAsync(h->duref, zrows.data(), sizeof(float) * h->L.total_rows, hipMemcpyHostToDevice, h->stream) !=
      hipSuccess)
    return bail(LB_EHIP);
  if (upload_strips(h, true) != LB_OK || upload_strips(h, false) != LB_OK) return bail(LB_EHIP);
  std::vector<Strip> tiles, btiles;  // kept until the synchronisation below
  for (int i = 0; i < n; ++i)
    if (tiled(o, c[i]) && h->blk_ok[i] != kPressureBoxes) {
      add_tiles(i, c[i], tile_shape(o), tiles);
      if (!h->blk_ok[i] && !(h->two_step && two_step_channel(c[i], h->L.esize)))
        add_tiles(i, c[i], tile_shape(o), btiles);
    }
  if (!tiles.empty() && hipMemcpyAsync(h->tiles, tiles.data(), sizeof(Strip) * tiles.size(),
                                       hipMemcpyHostToDevice, h->stream) != hipSuccess)
    return bail(LB_EHIP);
  h->n_tiles = (int)tiles.size();
  h->n_btiles = (int)btiles.size();
  if (!btiles.empty() && hipMemcpyAsync(h->btiles, btiles.data(), sizeof(Strip) * btiles.size(),
                                        hipMemcpyHostToDevice, h->stream) != hipSuccess)
    return bail(LB_EHIP);
  if (fill_rest(h, 0) != LB_OK || fill_rest(h, 1) != LB_OK) return bail(LB_EHIP);
  // zero stress at rest (outside any graph)
  for (int b = 0; b < 2; ++b)
    if (h->sbuf[b] &&
        hipMemsetAsync(h->sbuf[b], 0, (size_t)kStressPlanes * h->L.plane * h->L.esize, h->stream) != hipSuccess)
      return bail(LB_EHIP);
  if (hipStreamSynchronize(h->stream) != hipSuccess) return bail(LB_EHIP);
  // the allocation-free observation's scratch on this GPU (a failure here
  // is reported by lb_observe_noalloc, not by lb_create)
  h->noalloc_err = hipGetDevice(&h->device);
  if (h->noalloc_err == hipSuccess) h->noalloc_err = noalloc_scratch(h->device, &h->noalloc);
  *out = h;
  return LB_OK;
}

lb_status lb_destroy(lb_handle *h) {
  if (!h) return LB_OK;
  if (h->stream) (void)hipStreamSynchronize(h->stream);
  drop_graphs(h);
  if (h->cap) (void)hipStreamDestroy(h->cap);
  if (h->own_stream && h->stream) (void)hipStreamDestroy(h->stream);
  delete h;
  return LB_OK;
}

lb_status lb_step(lb_handle *h, int64_t n) {
  if (!h) return LB_EINVAL;
  if (n < 0) return fail(h, LB_EINVAL, "negative step count");
  h->obs_valid = false;
  int64_t left = n;
  // Every K steps of the handle's clock end a block: the convergence check
  // (if enabled) and, for FP32 storage, the move of the row reference
  // velocities. Whole blocks run as one graph; steps that start or end off
  // a block boundary are enqueued launch by launch, several steps each where
  // a kernel takes them. The boundaries do not depend on how the steps are
  // split over calls, and all kernels round alike, so neither does the result.
  while (left > 0) {
    bool any = false;
    for (int a : h->active) any |= (a != 0);
    if (!any) break;
    int m;
    if (h->since_block == 0 && left >= h->K) {
      if (!h->graph[h->cur]) {
        lb_status st = capture(h, h->cur);
        if (st != LB_OK) return st;
      }
      HIPCHECK(h, hipGraphLaunch(h->graph[h->cur], h->stream));
      m = h->K;
    } else {
      m = (int)std::min<int64_t>(left, h->K - h->since_block);
      int launches = 0;
      for (int k = 0; k < m; ++launches) {
        // boxes hold the halo of up to S steps; two steps per launch where
        // every channel takes them (the same results: no kernel's rounding
        // differs from another's)
        const int src = h->cur ^ (launches & 1);
        const int many = h->boxes[lb_handle::kMany].S, pressure = std::max(h->boxes[lb_handle::kPressureMany].S, 1);
        int S = std::min(h->only >= 0 ? h->boxes[h->only].S : h->both ? std::min(many, pressure) : 0, m - k);
        if ((h->both || h->only == lb_handle::kMany) && !(S > 1 ? h->box_several : h->box_one)) S = 0;
        const bool in_boxes = S > 0;
        if (!in_boxes) S = h->two_only ? std::min(2, m - k) : 1;
        lb_status st;
        if (in_boxes && h->both) {
          st = enqueue_boxes(h, lb_handle::kMany, src, k, S, h->stream);
          if (st == LB_OK)
            st = S > 1 ? enqueue_boxes(h, lb_handle::kPressureMany, src, k, S, h->stream)
                       : enqueue_pressure(h, src, k, h->stream, false);
        } else {
          st = in_boxes ? enqueue_boxes(h, h->only, src, k, S, h->stream)
               : S == 2 ? enqueue_two_step(h, src, k, h->stream)
                        : enqueue_step(h, src, k, h->stream);
        }
        if (st != LB_OK) return st;
        k += S;
      }
      HIPCHECK(h, launch_advance(h->dch, h->n_ch, m, h->stream));
      h->cur ^= (launches & 1);
    }
    for (int i = 0; i < h->n_ch; ++i)
      if (h->active[i]) h->t[i] += m;
    left -= m;
    h->since_block += m;
    h->obs_valid = false;
    if (h->since_block == h->K) {
      h->since_block = 0;
      bool observed = false;
      if (h->opt.steady_tol > 0) {
        lb_status st = check_steady(h);
        if (st != LB_OK) return st;
        observed = true;
      }
      lb_status st = rereference(h, observed);
      if (st != LB_OK) return st;
      h->obs_valid = false;
    }
  }
  h->obs_valid = false;
  return LB_OK;
}

lb_status lb_observe(lb_handle *h, int32_t ch, int32_t what, double *out, size_t n) {
  if (!h) return LB_EINVAL;
  if (ch < 0 || ch >= h->n_ch || !out) return fail(h, LB_EINVAL, "bad channel or output");
  const ChanDev &d = h->L.ch[ch];
  if (what == LB_OBS_STEP) {
    if (n < 1) return fail(h, LB_EINVAL, "output too small");
    out[0] = (double)h->t[ch];
    return LB_OK;
  }
  if (what == LB_OBS_ACTIVE) {
    if (n < 1) return fail(h, LB_EINVAL, "output too small");
    out[0] = h->active[ch];
    return LB_OK;
  }
  lb_status st = read_observation(h);
  if (st != LB_OK) return st;
  const double *s = &h->hscal[(size_t)ch * CS_COUNT];
  const double *pr = &h->hprof[(size_t)d.row_off * OF_COUNT];
  const long long N = (long long)d.nx * d.ny;
  if (what >= 32) {
    if (n < 1) return fail(h, LB_EINVAL, "output too small");
    switch (what) {
      case LB_OBS_MASS: out[0] = (double)N + s[CS_MASS_DEV]; return LB_OK;
      case LB_OBS_MOMX: out[0] = s[CS_MOMX]; return LB_OK;
      case LB_OBS_FLUX: out[0] = s[CS_FLUX]; return LB_OK;
      case LB_OBS_WALL_DRAG: out[0] = s[CS_DRAG]; return LB_OK;
      case LB_OBS_UMID: out[0] = s[CS_UMID]; return LB_OK;
      case LB_OBS_RESIDUAL: {
        // residual is only meaningful after two checks
        out[0] = h->n_checks >= 2 ? s[CS_RESIDUAL] : INFINITY;
        return LB_OK;
      }
      case LB_OBS_NAN: out[0] = s[CS_NAN]; return LB_OK;
      default: return fail(h, LB_EINVAL, "unknown observable");
    }
  }
  if (n < (size_t)d.ny) return fail(h, LB_EINVAL, "output shorter than ny");
  for (int y = 0; y < d.ny; ++y) {
    const double *r = pr + (size_t)y * OF_COUNT;
    double v;
    switch (what) {
      case LB_OBS_UX: v = r[OF_UX]; break;
      case LB_OBS_UY: v = r[OF_UY]; break;
      case LB_OBS_SXX: v = r[OF_SXX]; break;
      case LB_OBS_SXY: v = r[OF_SXY]; break;
      case LB_OBS_SYY: v = r[OF_SYY]; break;
      case LB_OBS_N1: v = r[OF_SXX] - r[OF_SYY]; break;
      case LB_OBS_PRESSURE: v = (1.0 + r[OF_RHOE_DEV]) / 3.0; break;
      case LB_OBS_KXY: v = r[OF_KXY]; break;
      case LB_OBS_TRT: v = r[OF_TRT]; break;
      case LB_OBS_KXX: v = r[OF_KXX]; break;
      default: return fail(h, LB_EINVAL, "unknown observable");
    }
    out[y] = v;
  }
  return LB_OK;
}

lb_status lb_observe_noalloc(lb_handle *h, int32_t ch, int32_t what, double *out, size_t n) {
  if (!h) return LB_EINVAL;
  if (ch < 0 || ch >= h->n_ch || !out) return fail(h, LB_EINVAL, "bad channel or output");
  const ChanDev &d = h->L.ch[ch];
  if (what == LB_OBS_STEP || what == LB_OBS_ACTIVE) {
    if (n < 1) return fail(h, LB_EINVAL, "output too small");
    out[0] = what == LB_OBS_STEP ? (double)h->t[ch] : (double)h->active[ch];
    return LB_OK;
  }
  const bool scalar = what >= 32;
  const bool known = scalar ? (what >= LB_OBS_MASS && what <= LB_OBS_NAN) : (what >= LB_OBS_UX && what <= LB_OBS_KXX);
  if (!known) return fail(h, LB_EINVAL, "unknown observable");
  const size_t count = scalar ? 1 : (size_t)d.ny;
  if (n < count) return fail(h, LB_EINVAL, scalar ? "output too small" : "output shorter than ny");
  if (what == LB_OBS_RESIDUAL) {
    // the residual of the last convergence check, kept in the workspace
    if (h->n_checks < 2) {
      out[0] = INFINITY;
      return LB_OK;
    }
    HIPCHECK(h, hipMemcpyAsync(out, h->dscal + (size_t)ch * CS_COUNT + CS_RESIDUAL, sizeof(double),
                               hipMemcpyDeviceToHost, h->stream));
    HIPCHECK(h, hipStreamSynchronize(h->stream));
    return LB_OK;
  }
  if (h->opt.stress_force)
    return fail(h, LB_EINVAL, "lb_observe_noalloc: the stress-force observation needs per-node scratch (use lb_observe)");
  if (!h->noalloc) return hipfail(h, h->noalloc_err, "lb_observe_noalloc: scratch address");
  // partials, profiles, scalars and the gathered result, 256-byte aligned
  auto chunk = [](size_t doubles) { return align_up(doubles, kAlign / sizeof(double)); };
  const size_t n_part = chunk((size_t)OF_COUNT * h->L.total_part), n_prof = chunk((size_t)OF_COUNT * h->L.total_rows);
  const size_t n_scal = chunk((size_t)CS_COUNT * h->n_ch), n_out = chunk(count);
  const size_t need = (n_part + n_prof + n_scal + n_out) * sizeof(double);
  if (need > kNoallocScratchBytes) {
    char buf[200];
    snprintf(buf, sizeof buf,
             "lb_observe_noalloc: this handle's observation needs %zu bytes of scratch, more than its %zu "
             "(use lb_observe)", need, kNoallocScratchBytes);
    return fail(h, LB_EINVAL, buf);
  }
  double *part = h->noalloc, *prof = part + n_part, *scal = prof + n_prof, *res = scal + n_scal;
  lb_status st = enqueue_observe_into(h, part, prof, scal, 0, 0);
  if (st != LB_OK) return st;
  hipLaunchKernelGGL(gather_observable_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, h->stream,
                     h->dch, ch, what, prof, scal, res);
  HIPCHECK(h, hipGetLastError());
  HIPCHECK(h, hipMemcpyAsync(out, res, count * sizeof(double), hipMemcpyDeviceToHost, h->stream));
  HIPCHECK(h, hipStreamSynchronize(h->stream));
  return LB_OK;
}

lb_status lb_get_state(lb_handle *h, int32_t ch, double *pops, double *P) {
  if (!h) return LB_EINVAL;
  if (ch < 0 || ch >= h->n_ch || !pops || !P) return fail(h, LB_EINVAL, "bad channel or output");
  const ChanDev &d = h->L.ch[ch];
  const size_t N = (size_t)d.nx * d.ny;
  const int es = h->L.esize;
  // the channel's tiles are one contiguous block of each state buffer; that
  // of the other one holds 10 planes in FP64, or 5 where slots are FP32
  const char *src = static_cast<const char *>(h->buf[h->cur]) + (size_t)slot(0, d.off) * es;
  double *stage = reinterpret_cast<double *>(static_cast<char *>(h->buf[h->cur ^ 1]) + (size_t)slot(0, d.off) * es);
  const StateArgs a = state_args(h, ch, h->t[ch]);
  const dim3 grid((unsigned)((N + 255) / 256));
  auto unpack = [&](double *to, int p0, int p1) {
    if (es == 8)
      hipLaunchKernelGGL(unpack_state_kernel<double>, grid, dim3(256), 0, h->stream,
                         reinterpret_cast<const double *>(src), h->duref + d.row_off, to, a, p0, p1);
    else
      hipLaunchKernelGGL(unpack_state_kernel<float>, grid, dim3(256), 0, h->stream,
                         reinterpret_cast<const float *>(src), h->duref + d.row_off, to, a, p0, p1);
    return hipGetLastError();
  };
  if (N <= kStageNodes) {
    // small: by the staging area in one copy, the other buffer left alone (two
    // copies and the mirroring after them took 61 us for 64 x 32
    // FP64, this 41)
    double *small = reinterpret_cast<double *>(h->ws + h->L.off_stage);
    std::vector<double> out((size_t)kPlanes * N);
    HIPCHECK(h, unpack(small, 0, kPlanes));
    HIPCHECK(h, hipMemcpyAsync(out.data(), small, sizeof(double) * kPlanes * N, hipMemcpyDeviceToHost, h->stream));
    HIPCHECK(h, hipStreamSynchronize(h->stream));
    std::copy(out.begin(), out.begin() + 9 * N, pops);
    std::copy(out.begin() + 9 * N, out.end(), P);
    return LB_OK;
  }
  const int per = es == 8 ? kPlanes : kPlanes / 2;
  for (int p0 = 0; p0 < kPlanes; p0 += per) {
    const int p1 = p0 + per;
    HIPCHECK(h, unpack(stage, p0, p1));
    const int np = std::min(p1, 9) - p0;
    HIPCHECK(h, hipMemcpyAsync(pops + p0 * N, stage, sizeof(double) * np * N, hipMemcpyDeviceToHost, h->stream));
    if (p1 == kPlanes)
      HIPCHECK(h, hipMemcpyAsync(P, stage + np * N, sizeof(double) * N, hipMemcpyDeviceToHost, h->stream));
  }
  const lb_status m = mirror_channel(h, ch);
  if (m != LB_OK) return m;
  HIPCHECK(h, hipStreamSynchronize(h->stream));
  return LB_OK;
}

lb_status lb_set_state(lb_handle *h, int32_t ch, const double *pops_in, const double *P, int64_t t) {
  if (!h) return LB_EINVAL;
  if (ch < 0 || ch >= h->n_ch || !pops_in || !P || t < 0) return fail(h, LB_EINVAL, "bad arguments");
  return store_state(h, ch, pops_in, P, true, t);
}

lb_status lb_get_stress(lb_handle *h, int32_t ch, double *sigma) {
  if (!h) return LB_EINVAL;
  if (ch < 0 || ch >= h->n_ch || !sigma) return fail(h, LB_EINVAL, "bad channel or output");
  if (!h->opt.viscoelastic) return fail(h, LB_EINVAL, "the handle runs the instantaneous model (no stored stress)");
  const ChanDev &d = h->L.ch[ch];
  const size_t N = (size_t)d.nx * d.ny, Npad = align_up(N, kTile);
  const int es = h->L.esize;
  // the channel's stress tiles are one contiguous block of each buffer
  const char *src = static_cast<const char *>(h->sbuf[h->cur]) + (size_t)sslot(0, d.off) * es;
  if (N <= kHostStressNodes) {
    std::vector<char> raw(kStressPlanes * Npad * es);
    HIPCHECK(h, hipMemcpyAsync(raw.data(), src, raw.size(), hipMemcpyDeviceToHost, h->stream));
    HIPCHECK(h, hipStreamSynchronize(h->stream));
    for (int p = 0; p < kStressPlanes; ++p)
      for (size_t id = 0; id < N; ++id) {
        const size_t k = (size_t)sslot(p, (long long)id);
        sigma[p * N + id] = es == 8 ? reinterpret_cast<const double *>(raw.data())[k]
                                    : (double)reinterpret_cast<const float *>(raw.data())[k];
      }
    return LB_OK;
  }
  // staged where the other buffer holds the channel's state
  double *stage = reinterpret_cast<double *>(static_cast<char *>(h->buf[h->cur ^ 1]) + (size_t)slot(0, d.off) * es);
  const dim3 grid((unsigned)((N + 255) / 256));
  if (es == 8)
    hipLaunchKernelGGL(unpack_stress_kernel<double>, grid, dim3(256), 0, h->stream,
                       reinterpret_cast<const double *>(src), stage, (long long)N);
  else
    hipLaunchKernelGGL(unpack_stress_kernel<float>, grid, dim3(256), 0, h->stream,
                       reinterpret_cast<const float *>(src), stage, (long long)N);
  HIPCHECK(h, hipGetLastError());
  HIPCHECK(h, hipMemcpyAsync(sigma, stage, sizeof(double) * kStressPlanes * N, hipMemcpyDeviceToHost, h->stream));
  const lb_status m = mirror_state(h, ch);
  if (m != LB_OK) return m;
  HIPCHECK(h, hipStreamSynchronize(h->stream));
  return LB_OK;
}

lb_status lb_set_stress(lb_handle *h, int32_t ch, const double *sigma) {
  if (!h) return LB_EINVAL;
  if (ch < 0 || ch >= h->n_ch || !sigma) return fail(h, LB_EINVAL, "bad channel or input");
  if (!h->opt.viscoelastic) return fail(h, LB_EINVAL, "the handle runs the instantaneous model (no stored stress)");
  const ChanDev &d = h->L.ch[ch];
  const size_t N = (size_t)d.nx * d.ny;
  const int es = h->L.esize;
  char *dst = static_cast<char *>(h->sbuf[h->cur]) + (size_t)sslot(0, d.off) * es;
  // staged like a small state, or where the other buffer holds the channel's
  const bool small = N <= kStageNodes;
  char *other = static_cast<char *>(h->buf[h->cur ^ 1]) + (size_t)slot(0, d.off) * es;
  double *stage = reinterpret_cast<double *>(small ? h->ws + h->L.off_stage : other);
  const dim3 grid((unsigned)((N + 255) / 256));
  HIPCHECK(h, hipMemcpyAsync(stage, sigma, sizeof(double) * kStressPlanes * N, hipMemcpyHostToDevice, h->stream));
  if (es == 8)
    hipLaunchKernelGGL(pack_stress_kernel<double>, grid, dim3(256), 0, h->stream, reinterpret_cast<double *>(dst),
                       stage, (long long)N);
  else
    hipLaunchKernelGGL(pack_stress_kernel<float>, grid, dim3(256), 0, h->stream, reinterpret_cast<float *>(dst),
                       stage, (long long)N);
  HIPCHECK(h, hipGetLastError());
  const lb_status m = small ? mirror_stress(h, ch) : mirror_channel(h, ch);
  if (m != LB_OK) return m;
  HIPCHECK(h, hipStreamSynchronize(h->stream));
  h->obs_valid = false;
  return LB_OK;
}

lb_status lb_set_profile(lb_handle *h, int32_t ch, const double *ux, const double *n1, int32_t n_pts,
                         int32_t points) {
  if (!h) return LB_EINVAL;
  if (ch < 0 || ch >= h->n_ch || !ux || !n1 || n_pts < 1) return fail(h, LB_EINVAL, "bad arguments");
  if (points != LB_PROFILE_ROWS && points != LB_PROFILE_CHEBYSHEV) return fail(h, LB_EINVAL, "unknown point set");
  const ChanDev &d = h->L.ch[ch];
  if (points == LB_PROFILE_ROWS && n_pts != d.ny) return fail(h, LB_EINVAL, "row profile needs ny values");
  std::vector<double> u(d.ny), q(d.ny);
  if (points == LB_PROFILE_ROWS) {
    for (int y = 0; y < d.ny; ++y) {
      u[y] = ux[y];
      q[y] = n1[y];
    }
  } else {
    // barycentric interpolation on the Chebyshev-Gauss points
    // d_k = cos(pi (2k+1)/(2n)), weights (-1)^k sin(pi (2k+1)/(2n))
    const double H = 0.5 * d.ny, yc = 0.5 * (d.ny - 1);
    for (int y = 0; y < d.ny; ++y) {
      const double dd = (y - yc) / H;
      double num_u = 0, num_q = 0, den = 0;
      int hit = -1;
      for (int k = 0; k < n_pts; ++k) {
        const double th = M_PI * (2 * k + 1) / (2.0 * n_pts);
        const double dk = std::cos(th);
        if (dd == dk) {
          hit = k;
          break;
        }
        const double wk = ((k & 1) ? -1.0 : 1.0) * std::sin(th) / (dd - dk);
        num_u += wk * ux[k];
        num_q += wk * n1[k];
        den += wk;
      }
      u[y] = hit >= 0 ? ux[hit] : num_u / den;
      q[y] = hit >= 0 ? n1[hit] : num_q / den;
    }
  }
  // one column: every node of a row starts alike
  std::vector<double> pops((size_t)9 * d.ny);
  for (int y = 0; y < d.ny; ++y) {
    // with the flow-induced density the conserved mass is sum (s + 3/2 P);
    // without it, sum s
    const double rho = d.nnp ? 1.0 - 1.5 * q[y] : 1.0;
    const double usq = u[y] * u[y];
    for (int i = 0; i < 9; ++i) {
      const double cu = HCX[i] * u[y];
      pops[(size_t)i * d.ny + y] = hweight(i) * rho * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * usq);
    }
  }
  return store_state(h, ch, pops.data(), q.data(), false, h->t[ch]);
}

}  // extern "C"

namespace {

// Rest state: n_i = a_i (stored as 0 when shifted), previous trace 0.
template <typename T>
__global__ void fill_rest_kernel(T *p, long long n_slots, int shifted) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n_slots;
       i += (long long)gridDim.x * blockDim.x) {
    const int f = (int)((i / kTile) % kPlanes);
    p[i] = (f < 9 && !shifted) ? T(f == 0 ? 4.0 / 9.0 : (f < 5 ? 1.0 / 9.0 : 1.0 / 36.0)) : T(0);
  }
}

lb_status fill_rest(lb_handle *h, int which) {
  const long long n = (long long)kPlanes * h->L.plane;
  if (h->L.esize == 8)
    hipLaunchKernelGGL(fill_rest_kernel<double>, dim3(2048), dim3(256), 0, h->stream,
                       static_cast<double *>(h->buf[which]), n, 0);
  else
    hipLaunchKernelGGL(fill_rest_kernel<float>, dim3(2048), dim3(256), 0, h->stream,
                       static_cast<float *>(h->buf[which]), n, 1);
  HIPCHECK(h, hipGetLastError());
  return LB_OK;
}

}  // namespace
