// dirac_plan.hip -- plans, argument checking and the C ABI of libdirac.
// The operations are defined in include/libdirac.h; this file validates
// arguments, owns the scratch memory and sequences kernel launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <new>
#include <vector>

#include "../../include/libdirac.h"
#include "dirac_launch.h"
#include "dirac_pass_cost.h"
#include "dirac_trace.h"
#include "dirac_plan.h"

using namespace dirac;

namespace {

thread_local char g_err[512] = "";

int fail(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof g_err, fmt, ap);
  va_end(ap);
  return code;
}

int hip_fail(hipError_t e, const char* what) {
  return fail(DL_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

bool finite_pos(double v) { return std::isfinite(v) && v > 0.0; }

}  // namespace

namespace dirac {

int set_error(int code, const char* msg) { return fail(code, "%s", msg); }
int set_hip_error(hipError_t e, const char* what) { return hip_fail(e, what); }

int validate_grid(const dl_grid* g, double dx, double dt, double c, double m, int dtype, int bc,
                  int max_ndim, int shift) {
  if (!g) return fail(DL_ERR_ARG, "grid is NULL");
  if (g->ndim < 1 || g->ndim > max_ndim) return fail(DL_ERR_ARG, "ndim must be 1..%d", max_ndim);
  for (int d = 0; d < g->ndim; ++d) {
    if (g->n[d] < 2) return fail(DL_ERR_ARG, "n[%d] = %lld: need at least 2 cells", d,
                                 static_cast<long long>(g->n[d]));
    if (g->n[d] > (int64_t(1) << 31)) return fail(DL_ERR_ARG, "n[%d] too large", d);
    if (g->axis[d] < 0 || g->axis[d] > 2) return fail(DL_ERR_ARG, "axis[%d] must be 0, 1 or 2", d);
    if (d > 0 && g->axis[d] <= g->axis[d - 1])
      return fail(DL_ERR_ARG, "axis[] must increase with the grid dimension");
    if (!std::isfinite(g->xmin[d])) return fail(DL_ERR_ARG, "xmin[%d] not finite", d);
  }
  int64_t cells = 1;
  for (int d = 0; d < g->ndim; ++d) {
    if (cells > (int64_t(1) << 40) / g->n[d]) return fail(DL_ERR_ARG, "grid too large");
    cells *= g->n[d];
  }
  if (!finite_pos(dx) || !finite_pos(dt) || !finite_pos(c))
    return fail(DL_ERR_ARG, "dx, dt and c must be finite and positive");
  if (!std::isfinite(m) || m < 0.0) return fail(DL_ERR_ARG, "m must be finite and >= 0");
  if (dtype != DL_C64 && dtype != DL_C128) return fail(DL_ERR_DTYPE, "unknown dtype %d", dtype);
  if (bc != DL_BC_ZERO && bc != DL_BC_PERIODIC) return fail(DL_ERR_ARG, "unknown bc %d", bc);
  const double K = c * dt / dx;
  if (!(std::fabs(K - shift) <= 1e-12 * shift))
    return fail(DL_ERR_CFL, "c*dt/dx = %.17g: the characteristic shift needs c*dt = %d dx", K,
                shift);
  return DL_OK;
}

PhaseK make_phase(int ntransports, double dt, double c, double m, int mode, bool two_angles) {
  PhaseK k{};
  const double s = std::ldexp(1.0, -ntransports);
  const double mc2 = m * c * c;
  const double mu = mc2 * dt;
  k.eu_re = s * std::cos(mu);
  k.eu_im = -s * std::sin(mu);
  k.ed_re = s * std::cos(mu);
  k.ed_im = s * std::sin(mu);
  k.dt = dt;
  k.mc2 = mc2;
  k.scale = s;
  k.scale_f = static_cast<float>(s);
  k.mode = mode;
  k.two_angles = two_angles ? 1 : 0;
  return k;
}

int phase_mode(double m, const double* V) {
  if (V) return 2;
  return (m != 0.0) ? 1 : 0;
}

int axes_code(const dl_grid& g) {
  if (g.ndim == 1) return g.axis[0];
  if (g.ndim == 2) return 10 * g.axis[1] + g.axis[0];  // 10: (x,y) 20: (x,z) 21: (y,z)
  return 210;
}

// Tiling of the one-pass sweep: strips of `strip_width` x cells, march
// segments sized so that at most `target` waves (one full round of resident
// waves) are created, avoiding a partial second round.
void make_tiling(const dl_grid& g, int64_t target, int seg_override, SweepArgs& a, int& blocks,
                 int strip_width) {
  a.nx = g.n[0];
  a.ny = g.ndim > 1 ? g.n[1] : 1;
  a.nz = g.ndim > 2 ? g.n[2] : 1;
  a.nstrips = (a.nx + strip_width - 1) / strip_width;
  if (g.ndim == 1) {
    a.nseg = 1;
    a.H = 1;
    a.nyblk = 1;
    a.ntiles = a.nstrips;
  } else if (g.ndim == 2) {
    const int64_t ny = a.ny;
    int64_t H;
    if (seg_override > 0) {
      H = seg_override;
    } else {
      int64_t nseg = target / a.nstrips;
      if (nseg < 1) nseg = 1;
      H = (ny + nseg - 1) / nseg;
      if (H < 8) H = 8;
    }
    if (H > ny) H = ny;
    a.H = static_cast<int>(H);
    a.nseg = (ny + H - 1) / H;
    a.nyblk = 1;
    a.ntiles = a.nstrips * a.nseg;
  } else {
    const int TY = kTY3D_F32;  // overwritten by the caller for FP64
    (void)TY;
    a.ntiles = 0;
  }
  blocks = static_cast<int>((a.ntiles + 3) / 4);
  a.xcd_remap = (blocks % 8 == 0) ? 1 : 0;
  a.axes_code = axes_code(g);
}

// Time of a register-tile pass in us, from fits (rms error 4-9 %) to the
// passes of 1 to 12 steps (8 with a vector potential) on planes of 128^2 to
// 4096^2 (2048^2) cells, of alpha_x and alpha_y with a potential: it picks a plan's
// tile and depth (dirac_pass_cost.h, fitted to every phase mode and to thin planes,
// says whether a call takes them).  A compute unit's first tile takes t0 + t1 per transport
// pair, every further one n0 + n1 per transport pair.  Without a vector potential
// and with at most one workgroup per unit (rms error 2-5 %, 64^2 to 640^2), the
// loads of all workgroups add `load` on a full chip.
double tile_time(bool fp64, bool strang, bool field, TileKind kind, int halo, double tiles,
                 int cu_count) {
  struct Fit { double t0, t1, n0, n1; };
  struct One { double t0, t1, load; };
  static const One one[2][2][4] = {  // [fp64][strang][kind]
      {{{4.7, 0.68, 2.2}, {6.3, 1.03, 3.8}, {4.7, 0.36, 1.4}, {6.8, 0.64, 3.3}},
       {{4.8, 0.57, 2.8}, {5.8, 1.01, 3.5}, {4.6, 0.34, 1.3}, {6.5, 0.61, 3.1}}},
      {{{8.4, 0.69, 6.1}, {9.9, 0.92, 6.4}, {6.5, 0.40, 3.2}, {10.3, 0.77, 7.5}},
       {{8.3, 0.66, 5.7}, {10.8, 0.77, 5.8}, {6.3, 0.38, 3.1}, {10.1, 0.74, 6.5}}}};
  const double per_cu = (kind >= kTilePairs ? 2.0 : 1.0) * tiles / cu_count;
  if (!field && (per_cu <= 1.0 || kind >= kTilePairs)) {
    const One& f = one[fp64][strang][kind];
    return f.t0 + f.t1 * halo + f.load * per_cu;
  }
  static const Fit fits[2][2][2][2] = {  // [field][fp64][strang][kind]
      {{{{5.0, 0.74, 4.2, 0.28}, {7.1, 1.07, 6.4, 0.51}},
        {{5.1, 0.63, 5.2, 0.11}, {6.5, 1.04, 6.0, 0.43}}},
       {{{9.3, 0.79, 15.5, 0.0}, {11.1, 1.0, 10.9, 0.17}},
        {{8.8, 0.79, 14.8, 0.0}, {11.8, 0.89, 10.4, 0.18}}}},
      {{{{5.1, 1.63, 4.4, 0.76}, {7.7, 2.37, 9.1, 2.21}},
        {{0.0, 0.0, 0.0, 0.0}, {9.0, 1.59, 11.0, 1.28}}},
       {{{5.9, 1.79, 8.6, 0.92}, {12.2, 3.10, 18.1, 2.76}},
        {{0.0, 0.0, 0.0, 0.0}, {13.7, 2.01, 20.5, 1.52}}}}};
  const Fit& f = fits[field][fp64][strang][kind];
  const double more = std::max(0.0, (per_cu < 4.0 ? std::ceil(per_cu) : per_cu) - 1.0);
  return f.t0 + f.t1 * halo + more * (f.n0 + f.n1 * halo);
}

// 3-D tiling: strips of `strip_width` x cells by blocks of `ty` y rows, march
// segments along z.  A tile (a wave, or with per_block = 1 a workgroup) of a
// segment of H planes runs H + halo plane iterations; with `target` tiles
// resident at once, the segment count is the one that minimises (rounds of
// resident tiles) x (H + halo).  per_block: tiles per workgroup (4 or 1).
void make_tiling3d(const dl_grid& g, int ty, int strip_width, int halo, int64_t target,
                   int seg_override, SweepArgs& a, int& blocks, int per_block) {
  a.nx = g.n[0];
  a.ny = g.n[1];
  a.nz = g.n[2];
  a.nstrips = (a.nx + strip_width - 1) / strip_width;
  a.nyblk = (a.ny + ty - 1) / ty;
  const int64_t per_seg = a.nstrips * a.nyblk;
  int64_t H;
  if (seg_override > 0) {
    H = seg_override;
  } else {
    if (target < 1) target = 1;
    H = a.nz;
    int64_t best = -1;
    for (int64_t ns = 1; ns <= 4096 && ns <= a.nz; ++ns) {
      const int64_t h = (a.nz + ns - 1) / ns;
      if (h < 4 && ns > 1) break;
      const int64_t nseg = (a.nz + h - 1) / h;
      const int64_t rounds = (per_seg * nseg + target - 1) / target;
      const int64_t cost = rounds * (h + halo);
      if (best < 0 || cost < best) {
        best = cost;
        H = h;
      }
    }
  }
  if (H > a.nz) H = a.nz;
  a.H = static_cast<int>(H);
  a.nseg = (a.nz + H - 1) / H;
  a.ntiles = per_seg * a.nseg;
  if (per_block == 1) {  // one workgroup per tile, XCD-contiguous runs of tiles
    blocks = static_cast<int>((a.ntiles + 7) / 8 * 8);
    a.xcd_remap = 1;
  } else {
    blocks = static_cast<int>((a.ntiles + 3) / 4);
    a.xcd_remap = (blocks % 8 == 0) ? 1 : 0;
  }
  a.axes_code = 210;
}

}  // namespace dirac

// ===========================================================================
// plan
// ===========================================================================

// one-cell transports per step: one per axis (Sec. 2.1), or two per axis for
// the second-order step (Sec. 2.4)
int dirac::transports_per_step(dl_plan p) {
  if (p->strang && p->g.ndim == 3) return 8;  // A four times, B and C twice
  return (p->strang ? 2 : 1) * p->g.ndim;
}

// make the tilings of phase mode `mode` current
static void select_tiling(dl_plan p, int mode) {
  const PlanTiling& t = p->tiling[mode < 0 || mode > 4 ? 2 : mode];
  for (int d = 0; d < kMaxDepth; ++d) {
    p->sw[d] = t.a[d];
    p->bl[d] = t.b[d];
  }
}

// waves that can be resident at once for the sweep kernel of this plan
static int64_t resident_waves(dl_plan p, int mode, int depth) {
  if (p->waves_per_cu > 0) return int64_t(p->cu_count) * p->waves_per_cu;
  int occ = p->dry ? 0
                   : sweep_occupancy(p->fp64, p->strang, p->g.ndim, axes_code(p->g), mode, depth,
                                     p->nc);
  if (occ <= 0) occ = 2;
  return int64_t(occ) * 4 * p->cu_count;
}

// tiling of a register-tile pass of `steps` steps; false if the tile is too
// small for them
static bool tile_args(dl_plan p, bool field, TileKind kind, int steps, TileArgs& a) {
  if (field && p->strang && kind != kTileBig) return false;
  const bool pairs = kind >= kTilePairs;
  if (pairs && (field || axes_code(p->g) != 10)) return false;
  const TileShape t = tile_shape(p->fp64, kind, field);
  const int halo = steps * (p->strang ? 2 : 1);
  const int64_t w = 64 - 2 * halo, h = t.waves * t.rows - 2 * halo;
  if (w < 16 || h < (field ? 2 : 8)) return false;
  a.nx = p->g.n[0];
  a.ny = p->g.n[1];
  a.periodic = (p->bc == DL_BC_PERIODIC);
  a.steps = steps;
  a.halo = halo;
  a.nstrips = (a.nx + w - 1) / w;
  a.ntiles = a.nstrips * ((a.ny + h - 1) / h);
  a.xcd_remap = 1;
  a.axes_code = axes_code(p->g);
  // the pairs apart double the loads, the set-up and the workgroups: only where
  // each finds a compute unit of its own (256^2, FP32: 0.97 against 1.19 us per
  // step; 384^2 with two workgroups on some units 1.45 against 1.34), which takes
  // a few units to spare (64 rows, FP64, 12 steps: 242 workgroups on 256 units 22
  // us, 256 of them 52 us)
  if (pairs && 2 * a.ntiles > p->cu_count - p->cu_count / 20) return false;
  return a.ntiles <= INT32_MAX - 8;
}

// fitted time of a register-tile pass in us; negative: no such pass
static double tile_cost(dl_plan p, bool field, TileKind kind, int steps) {
  TileArgs a{};
  if (!tile_args(p, field, kind, steps, a)) return -1.0;
  return tile_time(p->fp64, p->strang, field, kind, a.halo, static_cast<double>(a.ntiles),
                   p->cu_count);
}

// The register tiles of 2-D plans whose passes are not capped or retiled by the
// caller; a call takes them where they are predicted to beat the marching passes
// (pass_list).  With FP32 state on planes of any size (per step, Lie, potential: 1.2
// against 4.1 us at 256^2, 4.6 against 6.7 us at 1024^2, 14.0 against 17.0 us at
// 2048^2), with FP64 state or a vector potential up to 600 thousand cells (768^2 FP64
// 5.5 against 6.4 us; 1024^2 9.1 against 8.7, second order 18.4 against 15.5; pulse,
// 768^2: FP32 9.0 against 11.1 us, FP64 14.1 against 14.8; 1024^2: 15.6 against 13.7
// and 24.2 against 18.7).  The tile and the depth are those of the least fitted time
// per step; small planes of alpha_x and alpha_y run the two pairs of a spinor apart
// (per step, Lie: 128^2 FP32 1.15 -> 0.81 us, FP64 1.57 -> 1.06; 512^2 FP64 3.5 -> 2.8).
constexpr int64_t kTileMaxCells = 600000;

static void choose_tile(dl_plan p) {
  p->tile_depth = p->tile_depth_field = 0;
  if (p->g.ndim != 2 || p->depth_limit < kMaxDepth || p->waves_per_cu > 0 || p->seg_override > 0)
    return;
  const bool few = p->g.n[0] * p->g.n[1] <= kTileMaxCells;
  for (int field = 0; field < 2; ++field) {
    if (!few && (p->fp64 || field)) continue;
    int& depth = field ? p->tile_depth_field : p->tile_depth;
    TileKind& in_kind = field ? p->tile_kind_field : p->tile_kind;
    double best = 0.0;
    for (TileKind kind : {kTileSmall, kTileBig, kTilePairs, kTilePairsBig})
      for (int k = 1; k <= kMaxTileDepth; ++k) {
        const double t = tile_cost(p, field != 0, kind, k);
        if (t > 0.0 && (depth == 0 || t / k < best)) {
          best = t / k;
          depth = k;
          in_kind = kind;
        }
      }
  }
}

// The split of a line into workgroups of `kind` for passes of up to `steps`
// steps: halo and own, and the workgroups (0: no such pass).  own is a whole
// number of cache lines, and passes that follow each other share the split, so
// the cells a workgroup reads were written through its own L2 (3e5 cells, FP32,
// passes of 3 and 2 steps split on their own: 8.6 and 7.9 us, of 2 and 2 5.9).
static int64_t line_blocks(dl_plan p, LineKind kind, int steps, LineArgs& a) {
  if (kind == kLineSplit && p->nc != 4) return 0;
  a.halo = steps * (p->strang ? 2 : 1);
  a.own = (line_span(line_waves(kind)) - 2 * a.halo) / 8 * 8;
  if (a.halo > kMaxLineHalo || a.own <= 0) return 0;
  const int64_t blocks = (p->g.n[0] + a.own - 1) / a.own;
  // the pairs apart load every cache line twice: only where compute units are
  // idle otherwise (at most two workgroups each; 4096 cells, FP64: 0.142
  // against 0.197 us per step, 65536: 0.297 against 0.303, 262144: no gain)
  if (kind == kLineSplit && 2 * blocks > 2 * int64_t(p->cu_count)) return 0;
  return blocks <= INT32_MAX ? blocks : 0;
}

// Fitted time of such a pass in us (rms error 5-10 %, 15 % for the pairs apart;
// lines of 1000 to 2^22 cells, 2 to 96 transports): a compute unit's first
// workgroup takes t0 + t1 per step, every further one n0 + n1 per step; at the
// least the state's bytes at 4.5 TB/s.  Negative: no such pass.
static double line_cost(dl_plan p, LineKind kind, int steps) {
  struct Fit { double t0, t1, n0, n1; };
  static const Fit all[2][2][3] = {  // [fp64][strang][kind]
      {{{2.66, 0.138, 0.29, 0.067}, {2.71, 0.330, 1.52, 0.261}, {3.15, 0.078, 0.51, 0.026}},
       {{2.81, 0.210, 0.26, 0.105}, {2.64, 0.522, 1.39, 0.404}, {3.04, 0.124, 0.43, 0.041}}},
      {{{3.03, 0.149, 1.02, 0.059}, {3.64, 0.361, 4.47, 0.232}, {3.52, 0.088, 1.10, 0.022}},
       {{2.99, 0.260, 0.95, 0.104}, {3.75, 0.601, 4.57, 0.394}, {3.20, 0.154, 1.05, 0.038}}}};
  static const Fit pair[2][2][2] = {
      {{{2.91, 0.076, 0.17, 0.031}, {2.84, 0.166, 0.88, 0.129}},
       {{2.83, 0.119, 0.16, 0.047}, {2.77, 0.266, 0.84, 0.195}}},
      {{{2.98, 0.081, 0.41, 0.031}, {3.27, 0.199, 2.04, 0.123}},
       {{2.94, 0.140, 0.39, 0.054}, {3.19, 0.337, 2.02, 0.206}}}};
  LineArgs a{};
  const int64_t blocks = line_blocks(p, kind, steps, a);
  if (blocks == 0) return -1.0;
  const Fit& f = p->nc == 4 ? all[p->fp64][p->strang][kind] : pair[p->fp64][p->strang][kind];
  const double per_cu =
      static_cast<double>(kind == kLineSplit ? 2 * blocks : blocks) / p->cu_count;
  const double more = std::max(0.0, (per_cu < 4.0 ? std::ceil(per_cu) : per_cu) - 1.0);
  return std::max(f.t0 + f.t1 * steps + more * (f.n0 + f.n1 * steps),
                  2.0 * static_cast<double>(p->state_bytes) / 4.5e6);
}

// the kind of least fitted time for a pass of `steps` steps; its time
static double line_best(dl_plan p, int steps, LineKind* kind) {
  double best = -1.0;
  for (int k = 0; k < 3; ++k) {
    const double t = line_cost(p, static_cast<LineKind>(k), steps);
    if (t > 0.0 && (best < 0.0 || t < best)) {
      best = t;
      *kind = static_cast<LineKind>(k);
    }
  }
  return best;
}

constexpr int64_t kLineFewCells = 200000;
constexpr int64_t kLineFewCellsPair = int64_t(1) << 20;

// Lines without a vector potential whose passes are not capped by the caller
// run register passes of the depth of least fitted time per step (whole
// exchanges, kLineSync transports); they beat the marching passes at every
// length (lowest order, FP32, per step: 1000 cells 0.13 us, 2^22 cells 6.8
// against 12.7 us; second order at 2^20 cells 2.9 us).
static void choose_line(dl_plan p) {
  p->line_depth = 0;
  if (p->g.ndim != 1 || p->depth_limit < kMaxDepth) return;
  const int per = kLineSync / (p->strang ? 2 : 1);
  double best = 0.0;
  for (int k = per; k <= kMaxLineHalo; k += per) {
    LineKind kind = kLineSmall;
    const double t = line_best(p, k, &kind);
    if (t > 0.0 && (p->line_depth == 0 || t / k < best)) {
      best = t / k;
      p->line_depth = k;
    }
  }
}

static int plan_tiling(dl_plan p) {
  p->list_mode = -1;
  p->rev_steps = -1;
  // fused steps per pass.  A periodic 2-D pass reaches one row per stage (one
  // per lowest-order step, two per second-order step) beyond a segment on each
  // side and wraps once, so the box needs at least twice that many rows.  A
  // 3-D pass fuses at most two steps; the rows and planes its stored cells
  // depend on lie at most two beyond the box, which one wrap reaches for any
  // box of two or more cells per axis.
  int depth = 1;
  if (p->g.ndim == 3) {
    if (p->strang)
      depth = p->depth_limit;  // second-order groups: a capped depth, else the whole call
    else if (p->g.n[0] < kMaxRow3DFused)
      depth = std::min(p->depth_limit, max_depth3d(p->fp64));
  } else {
    depth = std::min(p->depth_limit, max_depth(p->fp64, p->strang));
    const int stages_per_step = p->strang ? 2 : 1;
    if (p->g.ndim == 2 && p->bc == DL_BC_PERIODIC)
      while (depth > 1 && p->g.n[1] < 2 * stages_per_step * depth) --depth;
  }
  p->depth = depth;
  // with a vector potential: 3-D passes fuse or group steps as without a field
  p->depth_field =
      (p->g.ndim == 3) ? depth : std::min(depth, field_max_depth(p->fp64, p->strang));
  for (int mode = 0; mode < 5; ++mode) {
    PlanTiling& t = p->tiling[mode];
    if (p->g.ndim == 3) {
      const int m = std::min(mode, 3);  // a pulse runs the static field's kernels
      make_tiling3d(p->g, p->fp64 ? kTY3D_F64 : kTY3D_F32, 64, 2, resident_waves(p, m, 1),
                    p->seg_override, t.a[0], t.b[0], 4);
      if (depth >= 2)  // workgroup tiles: resident workgroups are the target
        make_tiling3d(p->g, p->fp64 ? kTY3D2_F64 : kTY3D2_F32, strip_width(2), 4,
                      resident_waves(p, m, 2) / 4, p->seg_override, t.a[1], t.b[1], 1);
    } else {
      for (int d = 1; d <= (mode >= 3 ? p->depth_field : depth); ++d)
        make_tiling(p->g, resident_waves(p, mode, d), p->seg_override, t.a[d - 1], t.b[d - 1],
                    strip_width(pass_xlanes(p->strang, d)));
    }
    for (int d = 0; d < kMaxDepth; ++d) t.a[d].periodic = (p->bc == DL_BC_PERIODIC);
  }
  select_tiling(p, 2);
  choose_tile(p);
  choose_line(p);
  // resident 1-D path: the whole line in one workgroup (4 cells per thread)
  // for all steps of a call.  One workgroup issues every step, so it only
  // beats the tiled passes when those pay a launch for every one or two
  // steps: it is used for plans that fuse at most 2 steps per pass.
  p->resident = false;
  if (p->g.ndim == 1 && p->allow_resident && !p->strang && depth <= 2) {
    const int64_t n = p->g.n[0];
    const int64_t threads = ((n + 4 * 64 - 1) / (4 * 64)) * 64;
    if (threads <= 1024 && (p->bc == DL_BC_ZERO || threads * 4 == n)) {
      p->resident = true;
      p->res_threads = static_cast<int>(threads);
    }
  }
  return DL_OK;
}

// Plans with register passes, whose calls often take an odd number of passes, get
// the third state buffer with the second, in one allocation, up to this size (2048^2
// FP32: 134 MB): allocated by the first such call it cost that call 30 to 300 us.
// Larger plans prefer an even count (even_passes) and allocate it on demand.
constexpr size_t kAltWithPlan = size_t(256) << 20;

static hipError_t alloc_states(dl_plan p) {
  const size_t at = (p->state_bytes + 255) / 256 * 256;
  if (p->g.ndim < 3 && (p->tile_depth > 0 || p->tile_depth_field > 0 || p->line_depth > 0) &&
      p->state_bytes <= kAltWithPlan) {
    if (hipMalloc(&p->tmp, at + p->state_bytes) == hipSuccess) {
      p->alt = static_cast<char*>(p->tmp) + at;
      p->alt_in_tmp = true;
      return hipSuccess;
    }
    (void)hipGetLastError();
    p->tmp = nullptr;
  }
  return hipMalloc(&p->tmp, p->state_bytes);
}

extern "C" int dl_plan_create(dl_plan* out, const dl_grid* g, double dx, double dt, double c,
                              double m, dl_dtype dtype, dl_bc bc, unsigned flags) {
  dirac::TraceRange trace_range("dl_plan_create");
  if (!out) return fail(DL_ERR_ARG, "out is NULL");
  *out = nullptr;
  const bool strang = (flags & DL_STRANG) != 0;
  // characteristic shift per step: one cell (lowest order), two cells (the
  // half steps of the 1-D / 2-D second-order step), four cells (the quarter
  // steps of A in the 3-D second-order step)
  const int shift = strang ? ((g && g->ndim == 3) ? 4 : 2) : 1;
  int rc = validate_grid(g, dx, dt, c, m, dtype, bc, 3, shift);
  if (rc) return rc;
  if (g->ndim == 3 && !(g->axis[0] == 0 && g->axis[1] == 1 && g->axis[2] == 2))
    return fail(DL_ERR_ARG, "3-D grids carry alpha_x, alpha_y, alpha_z in order");
  const bool pair = (flags & DL_BISPINOR) != 0;
  if (pair && g->ndim != 1) return fail(DL_ERR_ARG, "two-component states are 1-D lines");
  dl_plan p = new (std::nothrow) dl_plan_s();
  if (!p) return fail(DL_ERR_NOMEM, "host allocation failed");
  p->g = *g;
  for (int d = g->ndim; d < 3; ++d) {
    p->g.n[d] = 1;
    p->g.axis[d] = -1;
    p->g.xmin[d] = 0.0;
  }
  p->dx = dx;
  p->dt = dt;
  p->c = c;
  p->m = m;
  p->dtype = dtype;
  p->bc = bc;
  p->flags = flags;
  p->fp64 = (dtype == DL_C128);
  p->cells = 1;
  for (int d = 0; d < g->ndim; ++d) p->cells *= g->n[d];
  p->nc = pair ? 2 : 4;
  p->state_bytes = static_cast<size_t>(p->cells) * p->nc * (p->fp64 ? 16 : 8);
  p->dry = (flags & DL_DRY) != 0;
  p->use_graph = (flags & DL_GRAPH) != 0;
  p->strang = strang;
  plan_tiling(p);
  if (p->dry) {
    *out = p;
    return DL_OK;
  }
  hipError_t e = hipGetDevice(&p->device);
  if (e != hipSuccess) {
    delete p;
    return hip_fail(e, "hipGetDevice");
  }
  int ncu = 0;
  if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, p->device) == hipSuccess &&
      ncu > 0)
    p->cu_count = ncu;
  plan_tiling(p);
  const bool mid = strang && g->ndim == 3;  // the 3-D second-order step runs through a third buffer
  if (mid) dirac::strang3d_prepare(p->fp64);
  if (alloc_states(p) != hipSuccess ||
      (mid && hipMalloc(&p->tmp2, p->state_bytes) != hipSuccess) ||
      hipMalloc(&p->partials, sizeof(double) * 2 * 8 * kObsBlocks) != hipSuccess ||
      hipMalloc(&p->dres, sizeof(double) * 64) != hipSuccess ||
      hipHostMalloc(&p->hres, sizeof(double) * 64, hipHostMallocMapped) != hipSuccess ||
      hipHostGetDevicePointer(reinterpret_cast<void**>(&p->hres_dev), p->hres, 0) !=
          hipSuccess) {
    (void)hipGetLastError();
    dl_plan_destroy(p);
    return fail(DL_ERR_NOMEM, "device allocation of %zu bytes of scratch failed", p->state_bytes);
  }
  *out = p;
  return DL_OK;
}

void dl_plan_s::drop_graphs() {
  for (auto& ge : graphs) {
    if (ge.exec) (void)hipGraphExecDestroy(ge.exec);
  }
  graphs.clear();
}

extern "C" int dl_plan_destroy(dl_plan p) {
  if (!p) return DL_OK;
  if (p->is_batch) {
    if (!p->dry) (void)hipDeviceSynchronize();
    destroy_batch(p);
    delete p;
    return DL_OK;
  }
  if (!p->dry) {
    (void)hipDeviceSynchronize();
    p->drop_graphs();
    if (p->cap_stream) (void)hipStreamDestroy(p->cap_stream);
    if (p->tmp) (void)hipFree(p->tmp);
    if (p->tmp2) (void)hipFree(p->tmp2);
    if (p->proj) (void)hipFree(p->proj);
    if (p->partials) (void)hipFree(p->partials);
    if (p->dres) (void)hipFree(p->dres);
    if (p->hres) (void)hipHostFree(p->hres);
    if (p->tile_partials) (void)hipFree(p->tile_partials);
    if (p->alt && !p->alt_in_tmp) (void)hipFree(p->alt);
    (void)hipGetLastError();
  }
  delete p;
  return DL_OK;
}

namespace dirac {

int check_live(dl_plan p) {
  if (!p) return fail(DL_ERR_ARG, "plan is NULL");
  if (p->is_batch) return fail(DL_ERR_STATE, "a batch handle: use dl_batch_step");
  if (p->dry) return fail(DL_ERR_STATE, "dry plan: created with DL_DRY, no device work allowed");
  return DL_OK;
}

int check_state_ptr(const void* ptr, const char* name) {
  if (!ptr) return fail(DL_ERR_ARG, "%s is NULL", name);
  if (reinterpret_cast<uintptr_t>(ptr) % 16) return fail(DL_ERR_ALIGN, "%s not 16-byte aligned", name);
  return DL_OK;
}

int check_f64_ptr(const void* ptr, const char* name, bool nullable) {
  if (!ptr) return nullable ? DL_OK : fail(DL_ERR_ARG, "%s is NULL", name);
  if (reinterpret_cast<uintptr_t>(ptr) % 8) return fail(DL_ERR_ALIGN, "%s not 8-byte aligned", name);
  return DL_OK;
}

// the field integral factors of the next `n` steps of the call (1 unless a
// pulse is on)
static void set_pulse(dl_plan p, double* F, int n) {
  for (int s = 0; s < n; ++s)
    F[s] = p->pulse_on ? pulse_step_integral(p->pulse, s) : 1.0;
}

// one pass of `depth` fused steps src -> dst with the current phase and tiling
hipError_t launch_pass(dl_plan p, int depth, const void* src, void* dst, const double* V,
                       hipStream_t st) {
  if (p->g.ndim == 3) {
    SweepArgs a = p->sw[p->strang ? 0 : depth - 1];  // second-order passes size their own grids
    a.ph = p->ph;
    a.At = p->field;
    set_pulse(p, a.F, std::min(depth, kMaxFieldSteps));
    a.cells = p->cells;
    if (p->strang)
      return launch_strang3d(p->fp64, src, dst, p->tmp2, nullptr, V, a,
                             p->pulse_on ? &p->pulse : nullptr, depth, st);
    return launch_sweep3d(p->fp64, depth, src, dst, V, a, p->bl[depth - 1], st);
  }
  SweepArgs a = p->sw[depth - 1];
  a.ph = p->ph;
  a.At = p->field;
  set_pulse(p, a.F, std::min(depth, kMaxFieldSteps));
  a.cells = p->cells;
  a.nc = p->nc;
  return launch_sweep2d(p->fp64, p->strang, depth, src, dst, V, a, p->bl[depth - 1], st);
}

// the last pass of a dl_step_observables call: a lowest-order pass (2-D, or
// the two-step 3-D pass) that also leaves the observables sums of every wave
// in p->tile_partials
static hipError_t launch_pass_obs(dl_plan p, int depth, const void* src, void* dst,
                                  const double* V, const ObsArgs& o, hipStream_t st,
                                  int64_t* waves) {
  if (p->g.ndim == 3) {
    if (depth != 2) return hipErrorInvalidValue;
    SweepArgs a = p->sw[1];
    a.ph = p->ph;
    a.At = nullptr;
    a.cells = p->cells;
    *waves = a.ntiles * 4;  // four waves per workgroup tile
    return launch_sweep3d_obs(p->fp64, src, dst, V, a, o, p->tile_partials, p->bl[1], st);
  }
  SweepArgs a = p->sw[depth - 1];
  a.ph = p->ph;
  a.At = nullptr;
  a.cells = p->cells;
  a.nc = p->nc;
  *waves = a.ntiles;
  return launch_sweep2d_obs(p->fp64, depth, src, dst, V, a, o, p->tile_partials,
                            p->bl[depth - 1], st);
}

// one register pass of `steps` steps src -> dst over a 1-D line split for
// passes of up to `most` steps
static hipError_t launch_pass_line(dl_plan p, LineKind kind, int steps, int most,
                                   const void* src, void* dst, const double* V,
                                   hipStream_t st) {
  LineArgs a{};
  if (steps > most) return hipErrorInvalidValue;
  const int64_t blocks = line_blocks(p, kind, most, a);
  a.nx = p->g.n[0];
  a.periodic = (p->bc == DL_BC_PERIODIC);
  a.steps = steps;
  a.ph = p->ph;
  return launch_line(p->fp64, p->strang, kind, p->g.axis[0], p->nc, src, dst, V, a, blocks, st);
}

// one register-tile pass of `depth` steps src -> dst
static hipError_t launch_pass_tile(dl_plan p, int depth, const void* src, void* dst,
                                   const double* V, hipStream_t st) {
  TileArgs a{};
  const bool field = p->ph.mode >= 3;
  const TileKind kind = field ? p->tile_kind_field : p->tile_kind;
  if (!tile_args(p, field, kind, depth, a)) return hipErrorInvalidValue;
  a.ph = p->ph;
  a.At = p->field;
  a.cells = p->cells;
  if (p->pulse_on) set_pulse(p, a.F, depth);
  return launch_tile2d(p->fp64, p->strang, kind, src, dst, V, a, st);
}

// copying the state back from the plan's buffer: 9 us up to 25 MB, then 5.4 TB/s
static double copy_us(dl_plan p) {
  return std::max(9.0, 2.0 * static_cast<double>(p->state_bytes) / 5.4e6);
}

// passes for n steps where a pass has at most `depth`, `more` passes of the call
// following: a single one ends in the plan's buffer, so two shallower ones, unless
// copying the state back is cheaper; an odd count of three or more needs the third
// state buffer, so one more pass where the plan lacks it and that costs at most 3 %.
// time(steps): of a pass
template <class F>
static int64_t even_passes(dl_plan p, int64_t n, int depth, int more, F time) {
  const int64_t passes = (n + depth - 1) / depth;
  if (passes == n) return passes;
  if (passes + more == 1) {
    const int k = static_cast<int>(n);
    return time(k - k / 2) + time(k / 2) < time(k) + copy_us(p) ? 2 : 1;
  }
  if ((passes + more) % 2 == 0 || p->alt_in_tmp) return passes;
  auto us = [&](int64_t m) {
    const int d = static_cast<int>(n / m);
    const double deep = static_cast<double>(n % m);
    return (static_cast<double>(m) - deep) * time(d) + (deep > 0.0 ? deep * time(d + 1) : 0.0);
  };
  return us(passes + 1) <= 1.03 * us(passes) ? passes + 1 : passes;
}

// predicted time of a 2-D call's passes (dirac_pass_cost.h)
static double list_us(dl_plan p, const PassList& l) {
  const int mode = p->ph.mode;
  const TileKind kind = mode >= 3 ? p->tile_kind_field : p->tile_kind;
  const double cells = static_cast<double>(p->cells);
  double us = l.passes == 1 ? copy_us(p) : 0.0;
  for (int r = 0; r < l.n; ++r) {
    const int d = l.run[r].depth;
    double t = 0.0;
    if (l.run[r].kind == PassRun::kTile) {
      TileArgs a{};
      if (tile_args(p, mode >= 3, kind, d, a))
        t = tile_pass_us(p->fp64, p->strang, mode, kind, a.halo, static_cast<double>(a.ntiles),
                         cells, p->cu_count);
    } else {
      const SweepArgs& a = p->sw[d - 1];
      t = march_pass_us(p->fp64, p->strang, mode, d,
                        mode >= 3 ? field_max_depth(p->fp64, p->strang)
                                  : max_depth(p->fp64, p->strang),
                        a.H, static_cast<double>(a.ny) / static_cast<double>(a.nseg),
                        p->bl[d - 1], cells, p->cu_count);
    }
    us += t * static_cast<double>(l.run[r].count);
  }
  return us;
}

// `left` steps in marching passes, deepest first, appended to l
static void add_marching(PassList& l, int64_t left, int dmax) {
  for (int d = dmax; d >= 1; --d) {
    l.add(PassRun::kMarch, d, left / d);
    left %= d;
  }
}

// The passes of a call of `nsteps` steps with the current phase: register
// passes (1-D) or register tiles (2-D) where the plan uses them and, in 2-D, they are
// predicted to be the faster, marching passes for the rest, deepest first.  obs: the
// last pass is the marching pass that sums the observables (on 3-D plans a two-step
// one, after the single step of an odd count).
static PassList make_pass_list(dl_plan p, int64_t nsteps, bool obs) {
  PassList l;
  int64_t left = nsteps;
  const int dmax = (p->ph.mode >= 3) ? p->depth_field : p->depth;
  // (FP64 calls of two marching passes or one on long lines run those: a wave of
  // a register pass reads 64 cells to write 48, and short passes are bound by the
  // bytes; 10 steps: 1e6 cells 63 against 66 us, 4e6 228 against 240.  FP32 lines of
  // two components: two full marching passes of long lines only; 10 steps: 2^20 cells
  // 19.6 against 21.3, 2^22 63.5 against 67.8; 8 steps 20.4 against 19.1)
  const bool few = p->fp64 ? p->cells >= kLineFewCells && left <= 2 * dmax
                           : p->nc == 2 && p->cells >= kLineFewCellsPair && left == 2 * dmax;
  if (p->line_depth > 0 && p->ph.mode <= 2 && left > 0 && !few) {
    const int64_t passes = even_passes(p, left, p->line_depth, 0, [&](int k) {
      LineKind kind = kLineSmall;
      return line_best(p, k, &kind);
    });
    const int d = static_cast<int>(left / passes);  // passes of d + 1 and d steps
    l.line_steps = static_cast<int>((left + passes - 1) / passes);
    (void)line_best(p, l.line_steps, &l.line_kind);
    l.add(PassRun::kLine, d + 1, left % passes);
    l.add(PassRun::kLine, d, passes - left % passes);
    return l;
  }
  const bool field = p->ph.mode >= 3;
  const int tile = field ? p->tile_depth_field : p->tile_depth;
  const TileKind tkind = field ? p->tile_kind_field : p->tile_kind;
  const int64_t n = obs ? left - std::min<int64_t>(left, dmax) : left;  // steps tiles may take
  if (tile > 0 && n > 0) {
    const int64_t passes = even_passes(p, n, tile, left > n ? 1 : 0, [&](int k) {
      return tile_cost(p, field, tkind, k);
    });
    const int d = static_cast<int>(n / passes);  // passes of d + 1 and d steps
    l.add(PassRun::kTile, d + 1, n % passes);
    l.add(PassRun::kTile, d, passes - n % passes);
    add_marching(l, left - n, dmax);
    PassList m;
    add_marching(m, left, dmax);
    const double margin = l.passes == 1 || (p->fp64 && p->strang) ? 1.0 : 0.95;
    return list_us(p, m) < margin * list_us(p, l) ? m : l;
  }
  if (obs && p->g.ndim == 3 && p->depth == 2 && left % 2 == 1 && left > 1) {
    l.add(PassRun::kMarch, 1, 1);
    --left;
  }
  add_marching(l, left, dmax);
  return l;
}

// ... kept for the next call of the same kind (the choice takes the host 0.3 us)
static const PassList& pass_list(dl_plan p, int64_t nsteps, bool obs) {
  if (p->list_mode != p->ph.mode || p->list_steps != nsteps || p->list_obs != obs) {
    p->list = make_pass_list(p, nsteps, obs);
    p->list_mode = p->ph.mode;
    p->list_steps = nsteps;
    p->list_obs = obs;
  }
  return p->list;
}

// The plan's third state buffer: with it, an odd number (>= 3) of passes
// ends in psi (psi -> tmp -> alt -> tmp ... -> psi) instead of in tmp with a
// copy back.  Where it did not come with the plan (kAltWithPlan), allocated once,
// by the first call that needs it, and never while the stream is being captured;
// without it the copy stays.  n: passes
// of the call.
static void want_alt(dl_plan p, int64_t n, hipStream_t st) {
  if (p->alt || p->alt_failed) return;
  if (p->g.ndim == 3 && p->strang) return;  // second-order 3-D groups end in psi by themselves
  if (n < 3 || n % 2 == 0) return;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone) {
    (void)hipGetLastError();
    return;
  }
  if (hipMalloc(&p->alt, p->state_bytes) != hipSuccess) {
    (void)hipGetLastError();
    p->alt = nullptr;
    p->alt_failed = true;
  }
}

// enqueue `nsteps` steps starting from psi, in passes of the plan's depth
// (the remainder in shallower passes), alternating between psi and the plan's
// tmp buffer, or, for an odd number (>= 3) of passes when the plan holds its
// third buffer, through tmp and that buffer so that the last pass writes psi;
// returns the buffer that holds the result.  With `obs`, the last pass also
// sums the observables (launch_pass_obs; `obs_waves` receives the number of
// partials it writes).
hipError_t enqueue_steps(dl_plan p, void* psi, const double* V, int64_t nsteps, hipStream_t st,
                         void** result, const ObsArgs* obs = nullptr,
                         int64_t* obs_waves = nullptr) {
  if (p->g.ndim == 3 && p->strang && p->depth_limit >= kMaxDepth && nsteps > 0 && !obs) {
    // second-order 3-D steps: the whole call is one group, nsteps + 1 passes
    // in place through the plan's two scratch states (a cap on the depth
    // keeps groups of that many steps instead)
    SweepArgs a = p->sw[0];
    a.ph = p->ph;
    a.At = p->field;
    a.cells = p->cells;
    hipError_t e = launch_strang3d(p->fp64, psi, psi, p->tmp2, p->tmp, V, a,
                                   p->pulse_on ? &p->pulse : nullptr, nsteps, st);
    if (e != hipSuccess) return e;
    p->pulse.n0 += nsteps;
    p->ran.of[PassRun::kMarch] += nsteps + 1;
    *result = psi;
    return hipSuccess;
  }
  const PassList list = pass_list(p, nsteps, obs != nullptr);
  list.count(p->ran, 1);
  want_alt(p, list.passes, st);
  void* third = (list.passes >= 3 && list.passes % 2 == 1) ? p->alt : nullptr;
  void* in = psi;
  int64_t i = 0;
  for (int r = 0; r < list.n; ++r) {
    const PassRun& run = list.run[r];
    for (int64_t c = 0; c < run.count; ++c, ++i) {
      const bool last = i == list.passes - 1;
      void* out = third ? (last ? psi : (i % 2 == 0 ? p->tmp : third))
                        : (in == psi ? p->tmp : psi);
      hipError_t e;
      if (run.kind == PassRun::kLine)
        e = launch_pass_line(p, list.line_kind, run.depth, list.line_steps, in, out, V, st);
      else if (run.kind == PassRun::kTile)
        e = launch_pass_tile(p, run.depth, in, out, V, st);
      else if (obs && last)
        e = launch_pass_obs(p, run.depth, in, out, V, *obs, st, obs_waves);
      else
        e = launch_pass(p, run.depth, in, out, V, st);
      if (e != hipSuccess) return e;
      p->pulse.n0 += run.depth;  // the pulse's step index of the next pass
      in = out;
    }
  }
  *result = in;
  return hipSuccess;
}

}  // namespace dirac

// dst = src for n 16-byte words: a plain kernel rather than a copy node, so a
// captured graph holds kernels only
__global__ __launch_bounds__(256) void k_copy16(const uint4* __restrict__ src,
                                                uint4* __restrict__ dst, int64_t n) {
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride)
    dst[i] = src[i];
}

// `replays`: how often the call will launch it (for the plan's pass counts)
static hipError_t graph_for(dl_plan p, void* psi, const double* V, int64_t pairs,
                            int64_t replays, hipGraphExec_t* exec) {
  if (p->g.ndim == 3 && p->strang && p->depth_limit >= kMaxDepth)
    p->ran.of[PassRun::kMarch] += replays * (2 * pairs + 1);
  else
    pass_list(p, 2 * pairs, false).count(p->ran, replays);
  for (auto& ge : p->graphs) {
    if (ge.psi == psi && ge.V == V && ge.pairs == pairs && ge.mode == p->ph.mode) {
      *exec = ge.exec;
      return hipSuccess;
    }
  }
  const PassCount ran = p->ran;  // the capture itself runs nothing
  if (!p->cap_stream) {
    hipError_t e = hipStreamCreateWithFlags(&p->cap_stream, hipStreamNonBlocking);
    if (e != hipSuccess) return e;
  }
  want_alt(p, pass_list(p, 2 * pairs, false).passes, p->cap_stream);  // before the capture begins
  hipGraph_t graph = nullptr;
  hipError_t e = hipStreamBeginCapture(p->cap_stream, hipStreamCaptureModeThreadLocal);
  if (e != hipSuccess) return e;
  void* res = nullptr;
  hipError_t e2 = enqueue_steps(p, psi, V, 2 * pairs, p->cap_stream, &res);
  p->ran = ran;
  if (e2 == hipSuccess && res != psi) {
    // an odd number of passes ends in the plan's buffer: every replay must
    // leave the state in psi, where the next one starts
    const int64_t words = static_cast<int64_t>(p->state_bytes / 16);
    const int64_t blocks = std::min<int64_t>((words + 255) / 256, 8192);
    hipLaunchKernelGGL(k_copy16, dim3(static_cast<unsigned>(blocks)), dim3(256), 0,
                       p->cap_stream, static_cast<const uint4*>(res), static_cast<uint4*>(psi),
                       words);
    e2 = hipGetLastError();
  }
  e = hipStreamEndCapture(p->cap_stream, &graph);
  if (e2 != hipSuccess) {
    if (graph) (void)hipGraphDestroy(graph);
    return e2;
  }
  if (e != hipSuccess) return e;
  hipGraphExec_t ex = nullptr;
  e = hipGraphInstantiate(&ex, graph, nullptr, nullptr, 0);
  (void)hipGraphDestroy(graph);
  if (e != hipSuccess) return e;
  if (p->graphs.size() >= 8) p->drop_graphs();
  p->graphs.push_back(GraphEntry{psi, V, pairs, p->ph.mode, ex});
  *exec = ex;
  return hipSuccess;
}

// A call of a few lowest-order steps over a line that one workgroup holds, one cell
// per thread, runs in place in one launch instead of two register passes.  Enqueued one
// after the other the second launch bounds such calls: through the Python binding, at
// every length, width, phase mode and step count up to the limit, 6.2 to 7.0 us in place
// against 8.5 to 9.1 (FP32), 6.8 to 8.8 against 9.6 to 10.4 (FP64).  On the device alone
// the steps of one workgroup (0.25 us and 0.009 us per wave with FP32 state, 0.033 with
// FP64) overtake two passes: 10 steps on 1000 cells with a potential 6.7 against 5.9 us
// with four components and 6.5 against 5.4 with two, FP64, 5 steps, 8.7 against 6.1 and
// 7.2 against 5.3.  The limits are where that difference eats the launch (2.6 us).  A
// call that is being captured costs the host nothing on replay and takes the faster
// device time (fits to captured calls on 64 to 1024 cells, errors 2 to 4 %).
static bool short_line(dl_plan p, int64_t nsteps, hipStream_t st) {
  if (p->line_depth == 0 || p->strang || !p->allow_resident || p->g.n[0] > 1024 ||
      nsteps > (p->fp64 ? 5 : 10))
    return false;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &cs) != hipSuccess) {
    (void)hipGetLastError();
    cs = hipStreamCaptureStatusNone;
  }
  if (cs == hipStreamCaptureStatusNone) return true;
  struct Fit { double t0, wave, v0, v_wave, step, step_wave; };
  static const Fit whole[2][2] = {  // [fp64][two components]
      {{1.52, 0.033, 0.23, 0.021, 0.244, 0.009}, {1.50, 0.011, 0.21, 0.024, 0.252, 0.009}},
      {{1.45, 0.127, 0.50, 0.031, 0.238, 0.033}, {1.47, 0.021, 0.42, 0.048, 0.228, 0.032}}};
  static const Fit passes[2][2] = {
      {{3.88, 0.020, 0.67, 0.013, 0.080, 0.0}, {3.80, 0.026, 0.63, 0.004, 0.042, 0.0}},
      {{4.06, 0.029, 1.01, 0.014, 0.085, 0.0}, {3.87, 0.024, 0.84, 0.007, 0.047, 0.0}}};
  const double waves = static_cast<double>((p->g.n[0] + 63) / 64);
  auto us = [&](const Fit& f) {
    return f.t0 + f.wave * waves + (p->ph.mode == 2 ? f.v0 + f.v_wave * waves : 0.0) +
           static_cast<double>(nsteps) * (f.step + f.step_wave * waves);
  };
  return us(whole[p->fp64][p->nc == 2]) <= us(passes[p->fp64][p->nc == 2]);
}

extern "C" int dl_step(dl_plan p, void* psi, const double* V, int64_t nsteps, void* stream) {
  dirac::TraceRange trace_range("dl_step");
  int rc = check_live(p);
  if (rc) return rc;
  if ((rc = check_state_ptr(psi, "psi"))) return rc;
  if ((rc = check_f64_ptr(V, "V", true))) return rc;
  if (nsteps < 0) return fail(DL_ERR_ARG, "nsteps = %lld < 0", static_cast<long long>(nsteps));
  if (nsteps == 0) return DL_OK;
  p->ran = PassCount{};
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int mode = phase_mode(p->m, V);
  p->ph = make_phase(transports_per_step(p), p->dt, p->c, p->m, mode, p->fp64);
  p->field = nullptr;
  select_tiling(p, mode);
  const bool one = short_line(p, nsteps, st);
  if (p->resident || one) {
    ResidentArgs ra{};
    ra.n = p->g.n[0];
    ra.nsteps = nsteps;
    ra.periodic = (p->bc == DL_BC_PERIODIC);
    ra.ph = p->ph;
    ra.nc = p->nc;
    hipError_t e = launch_resident1d(p->fp64, p->g.axis[0], psi, V, ra, one ? 1 : 4,
                                     one ? static_cast<int>((p->g.n[0] + 63) / 64 * 64)
                                         : p->res_threads,
                                     st);
    p->ran.whole = 1;
    return e == hipSuccess ? DL_OK : hip_fail(e, "resident 1-D sweep launch");
  }
  int64_t done = 0;
  if (p->use_graph && nsteps >= 2 * p->graph_pairs) {
    hipGraphExec_t ex = nullptr;
    const int64_t reps = nsteps / (2 * p->graph_pairs);
    hipError_t e = graph_for(p, psi, V, p->graph_pairs, reps, &ex);
    if (e != hipSuccess) return hip_fail(e, "graph capture");
    for (int64_t r = 0; r < reps; ++r) {
      e = hipGraphLaunch(ex, st);
      if (e != hipSuccess) return hip_fail(e, "hipGraphLaunch");
    }
    done = reps * 2 * p->graph_pairs;
  }
  void* res = nullptr;
  hipError_t e = enqueue_steps(p, psi, V, nsteps - done, st, &res);
  if (e != hipSuccess) return hip_fail(e, "sweep launch");
  if (res != psi) {
    e = hipMemcpyAsync(psi, res, p->state_bytes, hipMemcpyDeviceToDevice, st);
    if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync");
  }
  return DL_OK;
}

extern "C" int dl_step_field(dl_plan p, void* psi, const double* V, const double* A,
                             int64_t nsteps, void* stream) {
  dirac::TraceRange trace_range("dl_step_field");
  int rc = check_live(p);
  if (rc) return rc;
  if (!A) return dl_step(p, psi, V, nsteps, stream);
  if ((rc = check_state_ptr(psi, "psi"))) return rc;
  if ((rc = check_f64_ptr(V, "V", true))) return rc;
  if ((rc = check_f64_ptr(A, "A", false))) return rc;
  if (p->nc != 4) return fail(DL_ERR_ARG, "a vector potential couples all four components");
  if (nsteps < 0) return fail(DL_ERR_ARG, "nsteps = %lld < 0", static_cast<long long>(nsteps));
  if (nsteps == 0) return DL_OK;
  hipStream_t st = static_cast<hipStream_t>(stream);
  p->ran = PassCount{};
  p->ph = make_phase(transports_per_step(p), p->dt, p->c, p->m, 3, p->fp64);
  p->field = A;
  select_tiling(p, 3);
  void* res = nullptr;
  hipError_t e = enqueue_steps(p, psi, V, nsteps, st, &res);
  p->field = nullptr;
  if (e != hipSuccess) return hip_fail(e, "sweep launch");
  if (res != psi) {
    e = hipMemcpyAsync(psi, res, p->state_bytes, hipMemcpyDeviceToDevice, st);
    if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync");
  }
  return DL_OK;
}

extern "C" int dl_step_pulse(dl_plan p, void* psi, const double* V, const double* P,
                             const dl_pulse* pulse, double t0, int64_t nsteps, void* stream) {
  dirac::TraceRange trace_range("dl_step_pulse");
  int rc = check_live(p);
  if (rc) return rc;
  if ((rc = check_state_ptr(psi, "psi"))) return rc;
  if ((rc = check_f64_ptr(V, "V", true))) return rc;
  if ((rc = check_f64_ptr(P, "P", false))) return rc;
  if (!pulse) return fail(DL_ERR_ARG, "pulse is NULL");
  const double pv[5] = {pulse->omega, pulse->phase, pulse->t_on, pulse->t_flat, pulse->t_off};
  for (double v : pv)
    if (!std::isfinite(v)) return fail(DL_ERR_ARG, "pulse parameters must be finite");
  if (pulse->t_on < 0.0 || pulse->t_flat < 0.0 || pulse->t_off < 0.0)
    return fail(DL_ERR_ARG, "pulse durations must be >= 0");
  if (!std::isfinite(t0)) return fail(DL_ERR_ARG, "t0 must be finite");
  if (p->nc != 4) return fail(DL_ERR_ARG, "a vector potential couples all four components");
  if (nsteps < 0) return fail(DL_ERR_ARG, "nsteps = %lld < 0", static_cast<long long>(nsteps));
  if (nsteps == 0) return DL_OK;
  hipStream_t st = static_cast<hipStream_t>(stream);
  // 1-D / 2-D: phase mode 4 forms each step's field integral in the pass; 3-D
  // passes run the static-field kernels with At = F P, F of each step
  const int mode = (p->g.ndim == 3) ? 3 : 4;
  p->ran = PassCount{};
  p->ph = make_phase(transports_per_step(p), p->dt, p->c, p->m, mode, p->fp64);
  p->field = P;
  p->pulse = PulseK{pulse->omega, pulse->phase, pulse->t_on, pulse->t_flat, pulse->t_off,
                    t0, p->dt, 0};
  p->pulse_on = true;
  select_tiling(p, mode);
  void* res = nullptr;
  hipError_t e = enqueue_steps(p, psi, V, nsteps, st, &res);
  p->field = nullptr;
  p->pulse_on = false;
  if (e != hipSuccess) return hip_fail(e, "sweep launch");
  if (res != psi) {
    e = hipMemcpyAsync(psi, res, p->state_bytes, hipMemcpyDeviceToDevice, st);
    if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync");
  }
  return DL_OK;
}

extern "C" int dl_step_out(dl_plan p, const void* src, void* dst, const double* V,
                           void* stream) {
  dirac::TraceRange trace_range("dl_step_out");
  int rc = check_live(p);
  if (rc) return rc;
  if ((rc = check_state_ptr(src, "src"))) return rc;
  if ((rc = check_state_ptr(dst, "dst"))) return rc;
  if ((rc = check_f64_ptr(V, "V", true))) return rc;
  const char* a = static_cast<const char*>(src);
  const char* b = static_cast<const char*>(dst);
  if (a < b + p->state_bytes && b < a + p->state_bytes)
    return fail(DL_ERR_ARG, "src and dst overlap");
  hipStream_t st = static_cast<hipStream_t>(stream);
  p->ph = make_phase(transports_per_step(p), p->dt, p->c, p->m, phase_mode(p->m, V), p->fp64);
  p->field = nullptr;
  select_tiling(p, p->ph.mode);
  p->ran = PassCount{};
  p->ran.of[PassRun::kMarch] = 1;
  hipError_t e = launch_pass(p, 1, src, dst, V, st);
  return e == hipSuccess ? DL_OK : hip_fail(e, "sweep launch");
}

extern "C" int dl_step_fused_out(dl_plan p, const void* src, void* dst, const double* V,
                                 int64_t nsteps, void* stream) {
  dirac::TraceRange trace_range("dl_step_fused_out");
  int rc = check_live(p);
  if (rc) return rc;
  if ((rc = check_state_ptr(src, "src"))) return rc;
  if ((rc = check_state_ptr(dst, "dst"))) return rc;
  if ((rc = check_f64_ptr(V, "V", true))) return rc;
  if (nsteps < 1) return fail(DL_ERR_ARG, "nsteps = %lld < 1", static_cast<long long>(nsteps));
  const char* a = static_cast<const char*>(src);
  const char* b = static_cast<const char*>(dst);
  if (a < b + p->state_bytes && b < a + p->state_bytes)
    return fail(DL_ERR_ARG, "src and dst overlap");
  hipStream_t st = static_cast<hipStream_t>(stream);
  p->ph = make_phase(transports_per_step(p), p->dt, p->c, p->m, phase_mode(p->m, V), p->fp64);
  p->field = nullptr;
  select_tiling(p, p->ph.mode);
  // passes deepest first; they alternate between dst and the plan's buffer
  // so that the last one writes dst
  int64_t passes = 0;
  {
    int64_t left = nsteps;
    for (int d = p->depth; d >= 1; --d) {
      passes += left / d;
      left %= d;
    }
  }
  p->ran = PassCount{};
  p->ran.of[PassRun::kMarch] = passes;
  const void* in = src;
  int64_t i = 0, left = nsteps;
  for (int d = p->depth; d >= 1; --d) {
    for (; left >= d; left -= d, ++i) {
      void* out = ((passes - 1 - i) % 2 == 0) ? dst : p->tmp;
      hipError_t e = launch_pass(p, d, in, out, V, st);
      if (e != hipSuccess) return hip_fail(e, "sweep launch");
      in = out;
    }
  }
  return DL_OK;
}

// status of an observables result: a non-finite sum means a non-finite cell
// (|psi|^2 of finite FP32 / FP64 values cannot overflow a double sum of fewer
// than 2^40 cells); then the norm watchdog
static int observables_status(dl_plan p, const double* out) {
  for (int i = 0; i < 5; ++i)
    if (!std::isfinite(out[i]))
      return fail(DL_ERR_NONFINITE, "the state holds a NaN or an infinity (observable %d = %g)",
                  i, out[i]);
  if (p->norm_tol > 0.0) {
    const double N = out[0], hi = p->norm_ref * (1.0 + p->norm_tol),
                 lo = p->norm_ref * (1.0 - p->norm_tol);
    if (N > hi)
      return fail(DL_WARN_NORM, "norm %.17g exceeds the reference %.17g by more than %g", N,
                  p->norm_ref, p->norm_tol);
    if (p->bc == DL_BC_PERIODIC && N < lo)
      return fail(DL_WARN_NORM, "norm %.17g fell below the reference %.17g by more than %g "
                  "on a periodic box", N, p->norm_ref, p->norm_tol);
  }
  return DL_OK;
}

static ObsArgs obs_args(dl_plan p, double x_b) {
  ObsArgs a{};
  a.n0 = p->g.n[0];
  a.n1 = p->g.n[1];
  a.n2 = p->g.n[2];
  a.ndim = p->g.ndim;
  a.dx = p->dx;
  a.xmin0 = p->g.xmin[0];
  a.xmin1 = p->g.xmin[1];
  a.xmin2 = p->g.xmin[2];
  a.x_b = x_b;
  a.nc = p->nc;
  return a;
}

// wait for the final reduction, which wrote the five values straight into
// the plan's mapped pinned buffer (no copy back), and check them
static int finish_observables(dl_plan p, hipStream_t st, double out[5]) {
  hipError_t e = hipStreamSynchronize(st);
  if (e != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
  for (int i = 0; i < 5; ++i) out[i] = p->hres[i];
  return observables_status(p, out);
}

extern "C" int dl_observables(dl_plan p, const void* psi, double x_b, double out[5],
                              void* stream) {
  dirac::TraceRange trace_range("dl_observables");
  int rc = check_live(p);
  if (rc) return rc;
  if ((rc = check_state_ptr(psi, "psi"))) return rc;
  if (!out) return fail(DL_ERR_ARG, "out is NULL");
  if (!std::isfinite(x_b) && !std::isinf(x_b)) return fail(DL_ERR_ARG, "x_b is NaN");
  hipStream_t st = static_cast<hipStream_t>(stream);
  hipError_t e = launch_observables(p->fp64, psi, obs_args(p, x_b), p->partials, p->hres_dev, st);
  if (e != hipSuccess) return hip_fail(e, "observables launch");
  return finish_observables(p, st, out);
}

extern "C" int dl_step_observables(dl_plan p, void* psi, const double* V, int64_t nsteps,
                                   double x_b, double out[5], void* stream) {
  dirac::TraceRange trace_range("dl_step_observables");
  int rc = check_live(p);
  if (rc) return rc;
  if ((rc = check_state_ptr(psi, "psi"))) return rc;
  if ((rc = check_f64_ptr(V, "V", true))) return rc;
  if (nsteps < 0) return fail(DL_ERR_ARG, "nsteps = %lld < 0", static_cast<long long>(nsteps));
  if (!out) return fail(DL_ERR_ARG, "out is NULL");
  if (std::isnan(x_b)) return fail(DL_ERR_ARG, "x_b is NaN");
  const int mode = phase_mode(p->m, V);
  // the fused last pass exists for 2-D lowest-order plans of four-component
  // states on grid axes (x, y) and for 3-D lowest-order plans of two-step
  // passes (then at least two steps); every other plan steps, then reduces
  const bool fused2 = nsteps > 0 && p->g.ndim == 2 && !p->strang && p->nc == 4 &&
                      axes_code(p->g) == 10 && mode <= 2;
  const bool fused3 = nsteps > 1 && p->g.ndim == 3 && !p->strang && p->depth == 2 && mode <= 2;
  const bool fused = fused2 || fused3;
  if (!fused) {
    rc = dl_step(p, psi, V, nsteps, stream);
    if (rc) return rc;
    return dl_observables(p, psi, x_b, out, stream);
  }
  hipStream_t st = static_cast<hipStream_t>(stream);
  p->ph = make_phase(transports_per_step(p), p->dt, p->c, p->m, mode, p->fp64);
  p->field = nullptr;
  select_tiling(p, mode);
  if (fused2)
    for (int d = 1; d <= p->depth; ++d)
      if (!sweep2d_obs_available(p->fp64, d, mode))
        return fail(DL_ERR_STATE, "no fused observables pass of depth %d", d);
  int64_t need = 0;
  if (fused3)
    need = p->sw[1].ntiles * 4;
  else
    for (int d = 1; d <= p->depth; ++d) need = std::max<int64_t>(need, p->sw[d - 1].ntiles);
  if (need > p->tile_partials_n) {
    if (p->tile_partials) (void)hipFree(p->tile_partials);
    p->tile_partials = nullptr;
    p->tile_partials_n = 0;
    hipError_t e = hipMalloc(&p->tile_partials, sizeof(double) * kObsDoubles * need);
    if (e != hipSuccess) {
      p->tile_partials = nullptr;
      return hip_fail(e, "hipMalloc (observables partials)");
    }
    p->tile_partials_n = need;
  }
  p->ran = PassCount{};
  // whole graphs for all but the steps of the fused pass (at least one step,
  // two on 3-D grids)
  int64_t done = 0;
  const int64_t keep = fused3 ? 2 : 1;
  if (p->use_graph && nsteps - keep >= 2 * p->graph_pairs) {
    hipGraphExec_t ex = nullptr;
    const int64_t reps = (nsteps - keep) / (2 * p->graph_pairs);
    hipError_t e = graph_for(p, psi, V, p->graph_pairs, reps, &ex);
    if (e != hipSuccess) return hip_fail(e, "graph capture");
    for (int64_t r = 0; r < reps; ++r) {
      e = hipGraphLaunch(ex, st);
      if (e != hipSuccess) return hip_fail(e, "hipGraphLaunch");
    }
    done = reps * 2 * p->graph_pairs;
  }
  const ObsArgs o = obs_args(p, x_b);
  void* res = nullptr;
  int64_t waves = 0;
  hipError_t e = enqueue_steps(p, psi, V, nsteps - done, st, &res, &o, &waves);
  if (e != hipSuccess) return hip_fail(e, "sweep launch");
  if (res != psi) {
    e = hipMemcpyAsync(psi, res, p->state_bytes, hipMemcpyDeviceToDevice, st);
    if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync");
  }
  e = launch_obs_final(p->tile_partials, waves, o, p->hres_dev, st);
  if (e != hipSuccess) return hip_fail(e, "observables launch");
  return finish_observables(p, st, out);
}

extern "C" int dl_plan_set_norm_check(dl_plan p, double N_ref, double tol) {
  if (!p) return fail(DL_ERR_ARG, "plan is NULL");
  if (p->is_batch) return fail(DL_ERR_STATE, "a batch handle has no observables");
  if (!finite_pos(N_ref) || !std::isfinite(tol) || tol < 0.0)
    return fail(DL_ERR_ARG, "need N_ref > 0 and tol >= 0, both finite");
  p->norm_ref = N_ref;
  p->norm_tol = tol;
  return DL_OK;
}

extern "C" const char* dl_last_error(void) { return g_err; }
extern "C" int dl_version(void) { return LIBDIRAC_VERSION; }

// ---- tuning: tiling, fusion depth, plan description ----
extern "C" int dl_plan_set_tiling(dl_plan p, int waves_per_cu, int seg_len, int allow_resident,
                                  int graph_pairs) {
  if (!p) return fail(DL_ERR_ARG, "plan is NULL");
  if (waves_per_cu < 0 || waves_per_cu > 32) return fail(DL_ERR_ARG, "waves_per_cu out of range");
  if (seg_len < 0 || graph_pairs < 1) return fail(DL_ERR_ARG, "bad seg_len / graph_pairs");
  p->waves_per_cu = waves_per_cu;
  p->seg_override = seg_len;
  p->allow_resident = allow_resident != 0;
  p->graph_pairs = graph_pairs;
  if (!p->dry) p->drop_graphs();
  return plan_tiling(p);
}

extern "C" int dl_plan_set_depth(dl_plan p, int depth) {
  if (!p) return fail(DL_ERR_ARG, "plan is NULL");
  if (depth < 1 || depth > kMaxDepth) return fail(DL_ERR_ARG, "depth %d not in 1..%d", depth, kMaxDepth);
  p->depth_limit = depth;
  if (!p->dry) p->drop_graphs();
  return plan_tiling(p);
}

extern "C" int dl_plan_info(dl_plan p, int64_t* info, int n) {
  if (!p || !info) return fail(DL_ERR_ARG, "NULL argument");
  if (p->is_batch) {
    batch_info(p, info, n);
    return DL_OK;
  }
  const SweepArgs& t = p->sw[p->depth - 1];  // tiling of the deepest pass in use
  const int64_t vals[] = {p->bl[p->depth - 1], t.H,          t.nseg,         t.nstrips,
                          t.ntiles,            p->resident,  p->res_threads, p->waves_per_cu,
                          t.xcd_remap,         p->graph_pairs, p->depth,     p->bl[0],
                          reverse_depth(p),    p->depth_field,
                          // obsolete, for callers that read it: the steps of a kind of pass
                          // over short lines that the register passes replaced
                          (p->line_depth > 0 && !p->strang && p->g.n[0] <= 65536) ? 24 : 0,
                          p->tile_depth, p->line_depth,
                          p->tile_depth > 0 ? p->tile_kind + 1 : 0,
                          p->tile_depth_field, reverse_tile_depth(p),
                          p->ran.of[PassRun::kMarch], p->ran.of[PassRun::kTile],
                          p->ran.of[PassRun::kLine], p->ran.whole};
  const int nv = static_cast<int>(sizeof vals / sizeof vals[0]);
  for (int i = 0; i < n && i < nv; ++i) info[i] = vals[i];
  return DL_OK;
}
