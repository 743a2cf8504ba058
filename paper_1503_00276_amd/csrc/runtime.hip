// runtime.hip -- host runtime and C ABI of libpic.so (declared in include/pic.h).
//
// A Sim holds one or more independent periodic instances.  A plain context is
// a Sim of one instance; a batch is a Sim of many.  Each step launches, for
// all instances together: the fused particle kernel (one launch per group of
// dimension, shape order and boundary logic), the current smoothing where
// asked for, the field step (one launch per dimension, which also plans a
// rebin check), and every sort_interval steps the rebin's scatter.  pic_step
// replays captured HIP graphs of whole rebin cycles.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <thread>
#include <chrono>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/pic.h"
#include "pic_dev.h"
#include "pic_kernels.h"

namespace {

// dynamic LDS a fused-kernel workgroup may request: the CU's 160 KiB less
// 4 KiB for the kernel's static LDS (its item prefix, slot counters and
// reduction slots; a build test checks that they fit)
constexpr int kLdsMax = 160 * 1024 - 4096;
constexpr int kNumCU = 256;

struct Species {
  bool used = false;
  double rqm = 0.0;
  int64_t np = 0;
  int64_t cap = 0;
  int max_items = 0;
  std::vector<void*> allocs;
  StoreDesc desc{};
  StoreCtl* ctl = nullptr;
};

struct Instance {
  pic_config cfg{};
  GridDesc g{};
  float* F[2] = {nullptr, nullptr};  // fields, double-buffered by step parity
  float* Jacc[2] = {nullptr, nullptr};
  unsigned long long* J64[2] = {nullptr, nullptr};
  float* Jout = nullptr;
  float* Jsm[2] = {nullptr, nullptr};  // smoothing buffers (only when smoothing is on)
  WinCtl* win = nullptr;               // moving window state (device)
  float* emax = nullptr;               // running bound on |E_c| (device, see InstDesc)
  int* ndst = nullptr;  // neighbour tile table of the rebin
  double wmax[PIC_MAX_SPECIES] = {0, 0, 0, 0, 0, 0, 0, 0};
  double* rho_snap = nullptr;
  bool have_snap = false;
  bool settled = false;  // a step has run with particles: the default tile stays
  int64_t tiled_for = -1;  // particles the default tile was last chosen by
  Species sp[PIC_MAX_SPECIES];
  int64_t steps = 0;
};

struct Group {
  int dim, order, first, count, max_ncell, max_items, max_tiles, max_blocks;
  size_t lds;
  bool fixed64;
  int sm_max[3];  // most smoothing passes of any instance launched pass by pass, per axis
  int sm_tiles_max[3] = {0, 0, 0};  // the same of the instances smoothed in tiles
  int sm_tiles = 0;                 // most tiles of one of those (0: none)
  int inject_max; // moving window: most particles a store injects per shift
  bool window;    // some instance has a moving window
  bool thermal = false;  // stores: some moving window injects thermal momenta
  bool big = false;    // stores: some store has more tiles than the field step's launch plans
  int mode = 0;   // stores: boundary logic of the fused kernel (0 periodic, 1 moving window, 2 r-z)
  int resident = 1;  // stores: fused-kernel workgroups resident per CU (the grid is one full wave of them)
  // stores, per step of a sort cycle: the LDS that step stages (its halo
  // grows with the steps since the check) and the workgroups resident with it
  std::vector<size_t> lds_k;
  std::vector<int> res_k;
  bool cyl = false, cart = false;  // instances: some are r-z / some are Cartesian
  bool march = false, tiles3 = false;  // periodic 3D instances: some march along z / some take tiles
};

// Boundary logic an instance's stores need in the fused particle kernel.
int kernel_mode(const GridDesc& g) {
  // two-phase 3D kernel: int64 current tile for the deterministic int64
  // accumulation, else a 32-bit tile, with compile-time LDS strides when the
  // box's padded strides are the ones of 4x4xN tiles
  if (pic_gpd_split(g)) {
    if (g.acc_mode == PIC_ACC_FIXED64) return 4;
    return (g.fs0 == 12 && g.fs01 == 144 && g.js0 == 12 && g.js01 == 144) ? 5 : 6;
  }
  // two-phase periodic 2D kernel (FP32 accumulation, Esirkepov's deposit)
  if (pic_gpd_two_phase2(g)) return 7;
  return g.window ? (g.cyl ? 3 : 1) : (g.cyl ? 2 : 0);
}

// Particles per work item a store of this box uses: the two-phase kernels
// hold at most pic_gpd_split_chunk() (3D) or pic_gpd_two_phase2_chunk() (2D)
// per item.
int store_chunk(const GridDesc& g, int chunk) {
  if (pic_gpd_split(g)) return std::min(chunk, pic_gpd_split_chunk());
  if (pic_gpd_two_phase2(g)) return std::min(chunk, pic_gpd_two_phase2_chunk());
  return chunk;
}

struct Sim {
  int device = 0;       // HIP device the context was created on
  int num_cu = kNumCU;  // compute units of the device
  hipStream_t stream = nullptr;
  bool own_stream = false;
  std::vector<Instance> inst;
  int sort_interval = 1;
  int64_t total_cells = 0;  // of all instances
  int64_t steps = 0;
  StoreDesc* d_stores = nullptr;
  int d_stores_cap = 0;
  InstDesc* d_inst = nullptr;
  std::vector<Group> sgroups, igroups;
  std::vector<int> store_inst, store_species;  // d_stores index -> (instance, species)
  bool dirty = true;
  // the control words of every (instance, species), in one array, and the
  // host's copy: current unless steps were queued or a store was written since
  StoreCtl* d_ctl = nullptr;
  std::vector<StoreCtl> h_ctl;
  bool ctl_current = false;
  double* d_scratch = nullptr;  // reductions
  double* d_out = nullptr;      // reduction outputs
  void* d_diag = nullptr;       // diagnostics' device buffers, kept between calls
  size_t diag_cap = 0;          // its size in bytes
  std::string err;
  // captured graphs: one rebin cycle (sort_interval steps ending with the
  // check), one per parity of the cycle's first step
  hipGraphExec_t cycle_exec[2] = {nullptr, nullptr};
  bool use_graph = true;
  // profiling: event pairs around each kernel family, summed at read time
  bool profiling = false;
  std::vector<hipEvent_t> ev_free;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> ev_pending[3];
  double prof_ms[3] = {0, 0, 0};
  double prof_n[3] = {0, 0, 0};

  pic_status fail(pic_status code, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    err = buf;
    return code;
  }
};

#define HIPCHK(S, expr)                                                                      \
  do {                                                                                       \
    hipError_t e_ = (expr);                                                                  \
    if (e_ != hipSuccess) return (S).fail(PIC_E_HIP, "%s: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

int bits_for(int n) {
  int b = 0;
  while ((1 << b) < n) b++;
  return b;
}

// Region guards (nodes) of the gather (fa below, fb above) and of the deposit
// window (ja, jb) for a shape order, relative to a particle's cell.
void region_guards(int order, int& fa, int& fb, int& ja, int& jb) {
  if (order == 1) { fa = 1; fb = 2; ja = 1; jb = 3; }
  else if (order == 2) { fa = 1; fb = 3; ja = 2; jb = 4; }
  else { fa = 2; fb = 3; ja = 2; jb = 4; }
}

// Whether tiles of t cells suit an axis of n cells whose particles stray
// need - 2 cells: the remainder, if any, has to hold them too.
bool tile_ok(int n, int t, int need) {
  if (t <= 0 || t > n) return false;
  if (t == n) return true;
  if (t < need) return false;
  int r = n % t;
  return r == 0 || r >= need;
}

// Whether a configuration takes the two-phase periodic 2D kernel: Cartesian
// boxes without a moving window, with Esirkepov's deposit and FP32
// accumulation, whose work items fit in it (the library's chunk, or an
// asked-for chunk of at most what it holds); layouts with larger items keep
// the one-phase kernel.
bool two_phase2(const pic_config& c) {
  return c.ndim == 2 && !c.move_window && c.geometry != PIC_GEOM_RZ && c.deposit == PIC_DEPOSIT_ISIS &&
         c.accumulator != PIC_ACC_FIXED64 && (c.chunk == 0 || c.chunk <= pic_gpd_two_phase2_chunk());
}

// Cells per tile of the default layout.  Every work item stages its tile's
// fields with a halo and folds its current, so tiles are large where there
// are items enough to fill the chip, and small where there are not.
//   3D, two-phase kernel: 512 particles per tile, from 64 to 256 cells (ppc is
//     the mean particles per cell of what is loaded; 0 before, see tile_open).
//     96^3 cells, us a step with 4x4x4 / 8x4x4 / 8x8x4 tiles: quadratic shape at
//     1, 2, 4, 8 per cell 295 / 219 / 175, 313 / 242 / 223, 363 / 319 / 350,
//     522 / 572 / 572; cubic 375 / 267 / 249, 405 / 319 / 330, 483 / 457 / 548,
//     733 / 837 / 958; linear 222 / 157 / 131 ... 375 / 389 / 387.  The cubic shape
//     takes at most 128 cells: there the unit of its current needs no second
//     bound (class_reach in gpd.hip), whose registers cost every cubic box 2.7 %.
//   2D, two-phase kernel: 1,024 tiles (one wave of workgroups), from 64 to 256
//     cells: 64x64 8x8 16.7 us, 16x16 17.9; 512x256 at 4 per cell 16x8 32, 16x16
//     38; 1024x512 at 8 per cell 16x8 155, 16x16 144, 32x16 140; a batch of 24
//     boxes, 7.7 M particles, 16x8 254, 16x16 251, 32x8 249, 32x16 270.
//   2D, one-phase kernel: 512 tiles, from 128 to 256 cells.
//   3D, one-phase kernel: 512 cells.
// total: cells of all instances, which fill the chip together.
double default_tile_cells(const GridDesc& g, int64_t total, double ppc) {
  if (pic_gpd_split(g)) return ppc > 0.0 ? std::min(g.order == 3 ? 128.0 : 256.0, std::max(64.0, 512.0 / ppc)) : 64.0;
  if (g.dim == 3) return 512.0;
  if (pic_gpd_two_phase2(g)) return std::min(256.0, std::max(64.0, (double)total / 1024.0));
  return std::min(256.0, std::max(128.0, (double)total / 512.0));
}

// Default tile: among the extents valid on every axis (the asked-for ones where
// given) whose LDS leaves room for two workgroups per CU, the shape whose mean
// volume (an axis of n cells makes ceil(n / t) tiles of n / ceil(n / t) cells
// on average) is closest to 'cells', x-long in 2D (contiguous field rows), and
// of multiples of four in 3D (the cells of a wavefront then spread over the LDS
// banks; the 4x4xN strides are compile-time constants).  Extents that do not
// divide the axis are taken too: an axis of 37 or 53 cells used to become one
// tile (45x37x53, linear: 120 us in 3x17x25 tiles, 43 us in 9x8x8).
// Where none of those shapes does (a cubic 3D window, an asked-for long tile, a
// long interval: the halo alone fills half the LDS), any extent whose LDS one
// workgroup can have is looked at, so that a box is refused only if no tile
// fits it.  Returns false when no shape does.
// The tiles of the two-phase 3D kernel whose current takes its unit from the sum
// of the moves (the cubic shape, and 4x4xN) have at most the cells whose sum, with
// the shape's peaks, is that of 64 wherever the axes have such tiles.
// That costs no time: quadratic, 120x112x91 at 4 per cell, 4x4x8 474 us a step,
// 5x4x7 413, 8x4x4 410.
bool default_tile(const GridDesc& g0, const pic_config& c, double cells, int out[3]) {
  struct Extent {
    int t;
    double lg, cost;  // log2 of the mean extent; what the extent itself costs
  };
  const double want = std::log2(cells);
  const double aspect = g0.dim == 3 ? 0.0 : (pic_gpd_two_phase2(g0) ? (cells >= 192.0 ? 1.6 : 0.5) : 0.0);
  const double peak = g0.order == 1 ? 1.0 : (g0.order == 2 ? 0.75 : 2.0 / 3.0);
  double best = 1e300;
  for (int pass = 0; pass < 2 && best == 1e300; pass++) {
    const bool any = pass == 1;
    const size_t room = any ? (size_t)kLdsMax : (size_t)kLdsMax / 2;
    GridDesc g = g0;
    // The field tile alone (every kernel stages it; the padded strides of the
    // two-phase 3D kernel, which take a search, only add to it): an extent
    // whose field tile is too large with the smallest extents of the other
    // axes is left out.
    auto fields = [&]() {
      size_t n = 6 * sizeof(float);
      for (int d = 0; d < g.dim; d++) n *= (size_t)(g.tile[d] + 2 * g.slk[d] + g.fa + g.fb);
      return n;
    };
    int least[3] = {1, 1, 1};
    for (int d = 0; d < g.dim; d++) least[d] = c.tile[d] != 0 ? c.tile[d] : std::min(g.nx[d], g.slk[d] + 2);
    std::vector<Extent> cand[3];
    for (int d = 0; d < 3; d++) {
      const int need = g.slk[d] + 2, n = g.nx[d];
      auto add = [&](int t) {
        for (int k = 0; k < 3; k++) g.tile[k] = k == d ? t : least[k];
        if (fields() > room) return;
        double cost = n % t != 0 ? 0.05 : 0.0;
        if (g.dim == 3 && t % 4 != 0) cost += 0.15;
        cand[d].push_back({t, std::log2((double)n / ((n + t - 1) / t)), cost});
      };
      if (d >= g.dim) {
        add(1);
      } else if (c.tile[d] != 0) {
        add(c.tile[d]);
      } else {
        const int most = any ? n : (g.dim == 3 ? 16 : 64);
        for (int t = need; t < n && t <= most; t++)
          if (tile_ok(n, t, need)) add(t);
        if (n <= most || cand[d].empty()) add(n);
      }
    }
    for (const Extent& a : cand[0])
      for (const Extent& b : cand[1])
        for (const Extent& e : cand[2]) {
          double sc = a.cost + b.cost + (g.dim == 3 ? e.cost : 0.0) + std::fabs(a.lg + b.lg + e.lg - want) +
                      0.1 * std::fabs(a.lg - b.lg - aspect);
          if (g.dim == 3) sc += 0.1 * std::fabs(b.lg - e.lg) + 0.01 * (e.lg - a.lg);
          // the tiles whose unit is the sum of the moves alone (see gpd.hip)
          if (pic_gpd_split(g0) && (g0.order == 3 || (a.t == 4 && b.t == 4))) {
            const double over = std::log2(a.t * b.t * e.t * peak * peak / 64.0);
            if (over > 1e-9) sc += 8.0 + 2.0 * over;
          }
          if (sc >= best) continue;
          g.tile[0] = a.t;
          g.tile[1] = b.t;
          g.tile[2] = e.t;
          if (fields() > room || pic_gpd_lds_bytes(g) > room) continue;
          best = sc;
          for (int d = 0; d < 3; d++) out[d] = g.tile[d];
        }
  }
  return best < 1e300;
}

// Fill g from a validated configuration, tile and sort interval.
// ppc: mean particles per cell (0: not known), for the default tile.
pic_status setup_grid(Sim& S, const pic_config& c, int sort_interval, GridDesc& g, double ppc = 0.0) {
  memset(&g, 0, sizeof g);
  g.dim = c.ndim;
  g.order = c.shape_order;
  for (int d = 0; d < 3; d++) {
    g.nx[d] = d < c.ndim ? c.nx[d] : 1;
    g.dxd[d] = d < c.ndim ? c.dx[d] : 1.0;
    g.dx[d] = (float)g.dxd[d];
    g.rdx[d] = (float)(1.0 / g.dxd[d]);
    g.cdt[d] = (float)(g.dxd[d] / c.dt);
    g.e0[d] = (float)c.e0[d];
    g.b0[d] = (float)c.b0[d];
  }
  g.dt = (float)c.dt;
  g.dtd = c.dt;
  g.acc_mode = c.accumulator;
  g.deposit = c.deposit;
  g.window = c.move_window;
  g.cyl = c.geometry == PIC_GEOM_RZ;
  g.wa = c.dt / c.dx[0];
  g.jscale = 1.0f;
  g.jinv = 1.0f;
  g.flag_slack = 1;
  // Stray bound per axis.  After a check a particle sits in its tile (the
  // check re-sorted) or within flag_slack cells of it; each step moves it
  // less than c dt / dx_d cells along axis d.  The staged regions are sized
  // for the last step of a cycle; each launch stages only what its own step
  // needs (see the fused kernel).
  g.slack = 0;
  for (int d = 0; d < 3; d++) {
    const double v = d < c.ndim ? c.dt / c.dx[d] : 0.0;
    g.vstep[d] = std::nextafter((float)v, 2.0f);
    const int extra = d < c.ndim ? (int)std::ceil((sort_interval - 1) * v - 1e-12) : 0;
    g.slk[d] = d < c.ndim ? g.flag_slack + std::max(0, extra) : 0;
    g.slack = std::max(g.slack, g.slk[d]);
  }
  region_guards(g.order, g.fa, g.fb, g.ja, g.jb);
  g.tp2 = two_phase2(c) ? 1 : 0;
  if (pic_gpd_split(g)) {
    // the two-phase kernel stages only what the shapes reach, one node less
    // above than the one-phase kernel: gather taps reach cell offsets
    // [-fa, fb] (orders 1/2/3: [-1,1], [-1,2], [-2,2]) and the deposit
    // window [-ja, jb] ([-1,2], [-2,3], [-2,3]) of the particle's cell
    g.fb -= 1;
    g.jb -= 1;
  }
  g.ntiles = 1;
  int tile[3] = {1, 1, 1};
  bool any_auto = false;
  for (int d = 0; d < c.ndim; d++) {
    const int need = g.slk[d] + 2;
    tile[d] = c.tile[d];
    any_auto = any_auto || tile[d] == 0;
    if (tile[d] != 0 && !tile_ok(g.nx[d], tile[d], need))
      return S.fail(PIC_E_INVALID, "tile[%d]=%d does not suit nx=%d (needs >= %d cells per tile and per remainder)",
                    d, tile[d], g.nx[d], need);
  }
  if (any_auto) {
    const int64_t total = std::max<int64_t>(S.total_cells, (int64_t)g.nx[0] * g.nx[1] * g.nx[2]);
    if (!default_tile(g, c, default_tile_cells(g, total, ppc), tile))
      return S.fail(PIC_E_INVALID, "no tile fits the LDS");
  }
  for (int d = 0; d < 3; d++) {
    g.tile[d] = tile[d];
    g.ntile[d] = (g.nx[d] + tile[d] - 1) / tile[d];
    g.ntiles *= g.ntile[d];
  }
  int b0 = bits_for(g.nx[0]), b1 = bits_for(g.nx[1]), b2 = bits_for(g.nx[2]);
  if (b0 + b1 + b2 > 31) return S.fail(PIC_E_INVALID, "grid too large for a 31-bit packed cell index");
  g.sh1 = b0;
  g.sh2 = b0 + b1;
  g.m0 = (1 << b0) - 1;
  g.m1 = (1 << b1) - 1;
  g.ncell = g.nx[0] * g.nx[1] * g.nx[2];
  if (pic_gpd_split(g)) pic_gpd_split_strides(g);
  if (pic_gpd_lds_bytes(g) > (size_t)kLdsMax) return S.fail(PIC_E_INVALID, "tile needs more LDS than a workgroup has");
  return PIC_OK;
}

pic_status validate(Sim& S, const pic_config& c) {
  if (c.ndim != 2 && c.ndim != 3) return S.fail(PIC_E_INVALID, "ndim must be 2 or 3");
  if (c.shape_order < 1 || c.shape_order > 3) return S.fail(PIC_E_INVALID, "shape_order must be 1, 2 or 3");
  double inv = 0.0;
  for (int d = 0; d < c.ndim; d++) {
    if (c.nx[d] < 1) return S.fail(PIC_E_INVALID, "nx[%d] must be positive", d);
    if (!(c.dx[d] > 0.0) || !std::isfinite(c.dx[d])) return S.fail(PIC_E_INVALID, "dx[%d] must be positive", d);
    if (!std::isfinite(c.xmin[d])) return S.fail(PIC_E_INVALID, "xmin[%d] not finite", d);
    inv += 1.0 / (c.dx[d] * c.dx[d]);
  }
  if (!(c.dt > 0.0) || !std::isfinite(c.dt)) return S.fail(PIC_E_INVALID, "dt must be positive");
  if (c.dt * std::sqrt(inv) >= 1.0)
    return S.fail(PIC_E_INVALID, "dt=%g violates the Courant condition dt*sqrt(sum 1/dx^2) < 1", c.dt);
  if (c.capacity < 0 || c.capacity > (int64_t)0x7fffff00) return S.fail(PIC_E_INVALID, "capacity out of range");
  if (c.accumulator < PIC_ACC_FP32 || c.accumulator > PIC_ACC_FIXED64)
    return S.fail(PIC_E_INVALID, "unknown accumulator %d", c.accumulator);
  if (c.sort_interval < 0 || c.chunk < 0) return S.fail(PIC_E_INVALID, "negative sort_interval or chunk");
  if (c.deposit != PIC_DEPOSIT_ISIS && c.deposit != PIC_DEPOSIT_TRISTAN)
    return S.fail(PIC_E_INVALID, "unknown deposit %d", c.deposit);
  if (c.deposit == PIC_DEPOSIT_TRISTAN && c.shape_order != 1)
    return S.fail(PIC_E_INVALID, "the TRISTAN deposit needs the linear shape (shape_order 1)");
  if (c.move_window != 0 && c.move_window != 1) return S.fail(PIC_E_INVALID, "move_window must be 0 or 1");
  if (c.move_window) {
    for (int a = 0; a < c.ndim; a++)
      if (c.inject_ppc[a] < 1 || c.inject_ppc[a] > 64)
        return S.fail(PIC_E_INVALID, "inject_ppc[%d] must be 1..64 with a moving window", a);
    if (!std::isfinite(c.inject_w)) return S.fail(PIC_E_INVALID, "inject_w not finite");
    if (!(c.inject_uth >= 0.0) || !std::isfinite(c.inject_uth))
      return S.fail(PIC_E_INVALID, "inject_uth must be finite and >= 0");
    if (c.sort_interval > 1) return S.fail(PIC_E_INVALID, "a moving window needs sort_interval 1 (or 0)");
  }
  for (int a = 0; a < c.ndim; a++) {
    if (c.smooth_level[a] < 0 || c.smooth_level[a] > PIC_MAX_SMOOTH)
      return S.fail(PIC_E_INVALID, "smooth_level[%d] must be 0..%d", a, PIC_MAX_SMOOTH);
    for (int p = 0; p < c.smooth_level[a]; p++) {
      const double* wt = c.smooth_weights[a][p];
      double s = wt[0] + wt[1] + wt[2];
      if (!std::isfinite(wt[0]) || !std::isfinite(wt[1]) || !std::isfinite(wt[2]) || !(std::fabs(s) > 0.0))
        return S.fail(PIC_E_INVALID, "smoothing weights of axis %d pass %d must be finite with a nonzero sum", a, p);
    }
  }
  for (int d = 0; d < 3; d++)
    if (!std::isfinite(c.e0[d]) || !std::isfinite(c.b0[d])) return S.fail(PIC_E_INVALID, "external field not finite");
  if (c.geometry != PIC_GEOM_CARTESIAN && c.geometry != PIC_GEOM_RZ)
    return S.fail(PIC_E_INVALID, "unknown geometry %d", c.geometry);
  if (c.geometry == PIC_GEOM_RZ) {
    if (c.ndim != 2) return S.fail(PIC_E_INVALID, "the r-z geometry is two-dimensional");
    if (c.xmin[1] != 0.0) return S.fail(PIC_E_INVALID, "in r-z x2 is the radius: xmin[1] must be 0");
    if (c.nx[1] < 2) return S.fail(PIC_E_INVALID, "the r-z geometry needs at least 2 rows");
    if (c.sort_interval > 1) return S.fail(PIC_E_INVALID, "the r-z geometry needs sort_interval 1 (or 0)");
  }
  return PIC_OK;
}

// asked_tiles: some instance's tiles are given; they have to hold what strays
// in an interval, so the interval then stays short.
int default_interval(const pic_config& c, bool asked_tiles) {
  // 3D tiles are LDS-bound: keep the slack at one cell and check every step;
  // a moving window removes and injects particles at every step's check, and
  // the r-z wall removes the particles that reach it at the step's check
  if (c.ndim == 3 || c.move_window || c.geometry == PIC_GEOM_RZ) return 1;
  double vmax = 0.0;
  for (int d = 0; d < c.ndim; d++) vmax = std::max(vmax, c.dt / c.dx[d]);
  if (two_phase2(c) && !asked_tiles) {
    // field and current tile share the two-phase kernel's LDS, so a wider halo
    // costs it little and the check and the scatter are spread over more
    // steps: 1024x256 laser wakefield (0.92 cells a step) at 2 / 4 / 8 / 12
    // steps 125 / 108 / 104 / 98 us a step, thermal boxes (0.5 cells a step)
    // at 3 / 8 / 12 41-147 / 41-144 / 42-150; the longest interval up to 8
    // whose strayed particles fit tiles of 16 cells or less
    for (int s = 8; s > 1; s--)
      if (3 + (int)std::ceil((s - 1) * vmax - 1e-12) <= 16) return s;
    return 1;
  }
  // largest interval whose slack stays at 2 cells
  int s = 1 + (int)std::floor(1.0 / vmax + 1e-12);
  return std::max(1, std::min(s, 8));
}

// Particles per work item unless asked for (np: the store's particles).  Small
// stores are split so that the chip has work for its workgroups, large ones
// take the items that stage least.
//   2D, two-phase: 512 items, 256 to 1,024 particles.  64x64 at 16 per cell
//     256 / 512 / 1,024: 16.7 / 17.6 / 21 us a step; 256x128 at 8 per cell
//     512 / 1,024 in 16x16 tiles 27 / 30; 1024x512 512 / 1,024: 167 / 144.
//   2D, one-phase: 256 particles in a store of under 2^18, else 2,048 items
//     from 512 to 2,048 particles.  r-z 384x96 256 / 512 / 2,048: 53 / 57 / 71 us
//     a step; moving window 768x192 512 / 1,024 / 2,048: 132 / 135 / 164.
//   3D: 2,048 (the two-phase kernel takes at most 768 of them).
// Tiles that were asked for keep the library's largest items.
int default_chunk(const Sim& S, const pic_config& c, const GridDesc& g, int64_t np) {
  const int64_t all = np * (int64_t)S.inst.size();  // the instances of a batch run together
  auto split = [&](int items, int lo, int hi) {
    const int64_t c = (all / items + 63) / 64 * 64;
    return (int)std::min<int64_t>(hi, std::max<int64_t>(lo, c));
  };
  for (int d = 0; d < g.dim; d++)
    if (c.tile[d] != 0) return 2048;
  if (g.dim == 3) return 2048;
  if (pic_gpd_two_phase2(g)) return split(512, 256, pic_gpd_two_phase2_chunk());
  return all < (1 << 18) ? 256 : split(2048, 512, 2048);
}

// The default chunk of a store that took more particles where they are: larger
// chunks make fewer items, so the item arrays hold them.
void grow_chunk(const Sim& S, const Instance& I, Species& sp, int64_t want) {
  if (I.cfg.chunk > 0) return;
  sp.desc.chunk = std::max(sp.desc.chunk, store_chunk(I.g, default_chunk(S, I.cfg, I.g, want)));
}

// Bytes rounded up to a multiple of 256 (sub-buffers of an allocation).
size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

template <typename T>
pic_status dalloc(Sim& S, std::vector<void*>& list, T** p, size_t n) {
  void* q = nullptr;
  hipError_t e = hipMalloc(&q, std::max<size_t>(n, 1) * sizeof(T));
  if (e != hipSuccess) return S.fail(PIC_E_NOMEM, "hipMalloc of %zu bytes failed: %s", n * sizeof(T), hipGetErrorString(e));
  list.push_back(q);
  *p = (T*)q;
  return PIC_OK;
}

void free_species(Species& sp) {
  for (void* p : sp.allocs) (void)hipFree(p);
  sp.allocs.clear();
  sp.cap = 0;
  sp.np = 0;
  sp.ctl = nullptr;
  memset(&sp.desc, 0, sizeof sp.desc);
}

// Fixed-point unit of the current: a single contribution of particle p is
// at most |w_p| |v_p| < max|w| (the charge fraction that crosses a face in a
// step is at most the displacement in cells, the transverse weight at most
// one), which stays below 2^31 units; the conversion to int32 saturates, so a
// contribution that FP32 rounding lifts a hair above the bound loses a part
// in 10^9 at most.
void set_current_scale(Instance& I) {
  double wmax = 0.0;
  for (int s = 0; s < PIC_MAX_SPECIES; s++) wmax = std::max(wmax, I.wmax[s]);
  double V = wmax;
  int e = 31;
  if (V > 0.0) e = (int)std::floor(31.0 - std::log2(V * 1.0001));
  e = std::max(-60, std::min(60, e));
  I.g.jscale = std::ldexp(1.0f, e);
  I.g.jinv = std::ldexp(1.0f, -e);
  for (int s = 0; s < PIC_MAX_SPECIES; s++) {
    Species& sp = I.sp[s];
    if (!sp.used) continue;
    sp.desc.g = I.g;
    sp.desc.wmax = std::nextafter((float)I.wmax[s], INFINITY);  // the one-phase kernels' per-item unit
  }
}

// Allocate (or grow) a species store for 'cap' particles.
pic_status alloc_species(Sim& S, Instance& I, Species& sp, int64_t cap, int chunk) {
  free_species(sp);
  const GridDesc& g = I.g;
  StoreDesc& d = sp.desc;
  memset(&d, 0, sizeof d);
  d.g = g;
  d.chunk = store_chunk(g, chunk);
  d.max_items = (int)std::min<int64_t>((int64_t)g.ntiles + cap / d.chunk + 1, 0x7fffffff);
  sp.max_items = d.max_items;
  // one allocation for all arrays, each on a 256-byte boundary
  std::vector<std::pair<void**, size_t>> parts;
  auto al = [&](auto** p, size_t n) { parts.push_back({(void**)p, n * sizeof(**p)}); };
  for (int s = 0; s < 2; s++) {
    al(&d.cell[s], cap);
    for (int k = 0; k < g.dim; k++) al(&d.eps[s][k], cap);
    for (int k = 0; k < 3; k++) al(&d.u[s][k], cap);
    al(&d.w[s], cap);
    al(&d.id[s], cap);
    al(&d.toff[s], g.ntiles + 1);
    al(&d.ioff[s], g.ntiles + 1);
    al(&d.items[s], d.max_items);
  }
  al(&d.pre, (size_t)d.max_items * PIC_NSLOT);
  al(&d.dcount, g.ntiles);
  al(&d.bsum, (size_t)2 * ((g.ntiles + PIC_REBIN_TILES - 1) / PIC_REBIN_TILES));
  al(&d.bpre, (size_t)2 * ((g.ntiles + PIC_REBIN_TILES - 1) / PIC_REBIN_TILES));
  size_t bytes = 0;
  for (auto& q : parts) bytes += align256(std::max<size_t>(q.second, 1));
  char* slab = nullptr;
  pic_status st;
  if ((st = dalloc(S, sp.allocs, &slab, bytes)) != PIC_OK) return st;
  for (auto& q : parts) {
    *q.first = slab;
    slab += align256(std::max<size_t>(q.second, 1));
  }
  HIPCHK(S, hipMemset(d.dcount, 0, (size_t)g.ntiles * sizeof(int)));
  sp.ctl = S.d_ctl + ((&I - S.inst.data()) * PIC_MAX_SPECIES + (&sp - I.sp));
  d.ctl = sp.ctl;
  S.ctl_current = false;
  d.F[0] = I.F[0];
  d.F[1] = I.F[1];
  for (int k = 0; k < 2; k++) {
    d.Jacc[k] = I.Jacc[k];
    d.J64[k] = I.J64[k];
  }
  d.ndst = I.ndst;
  d.cap = (int)cap;
  d.win = I.win;
  d.emax = I.emax;
  StoreCtl z{};
  HIPCHK(S, hipMemcpy(sp.ctl, &z, sizeof z, hipMemcpyHostToDevice));
  sp.cap = cap;
  return PIC_OK;
}

// Rebuild the device descriptor arrays (stores grouped by dimension and shape
// order, instances grouped by dimension).
pic_status refresh_descriptors(Sim& S) {
  if (!S.dirty) return PIC_OK;
  std::vector<StoreDesc> stores;
  S.store_inst.clear();
  S.store_species.clear();
  S.sgroups.clear();
  S.igroups.clear();
  for (int dim = 2; dim <= 3; dim++)
    for (int order = 1; order <= 3; order++)
      for (int mode = 0; mode <= 7; mode++) {
      Group gr{dim, order, (int)stores.size(), 0, 0, 0, 0, 0, 0, false, {0, 0, 0}, 0, false};
      gr.mode = mode;
      for (size_t i = 0; i < S.inst.size(); i++) {
        Instance& I = S.inst[i];
        if (I.g.dim != dim || I.g.order != order || kernel_mode(I.g) != mode) continue;
        for (int s = 0; s < PIC_MAX_SPECIES; s++) {
          Species& sp = I.sp[s];
          if (!sp.used || sp.np == 0) continue;
          sp.desc.np = (int)sp.np;
          sp.desc.tile0 = gr.max_tiles;
          sp.desc.blk0 = gr.max_blocks;
          stores.push_back(sp.desc);
          S.store_inst.push_back((int)i);
          S.store_species.push_back(s);
          gr.count++;
          gr.max_items += sp.max_items;
          gr.max_tiles += I.g.ntiles;
          gr.max_blocks += (I.g.ntiles + PIC_REBIN_TILES - 1) / PIC_REBIN_TILES;
          gr.lds = std::max(gr.lds, pic_gpd_lds_bytes(I.g));
          if (I.g.window) gr.window = true;
          if (I.g.ntiles > pic_plan_tiles()) gr.big = true;
          if (sp.desc.inj_uth > 0.0) gr.thermal = true;
          gr.inject_max = std::max(gr.inject_max, sp.desc.inj_ppc[0] * sp.desc.inj_ppc[1] * sp.desc.inj_ppc[2] *
                                                      (I.g.ncell / I.g.nx[0]));
        }
      }
          if (gr.count > 0) {
        if (gr.count > pic_gpd_max_group()) return S.fail(PIC_E_INVALID, "too many stores in one group");
        HIPCHK(S, pic_gpd_prepare(dim, order, gr.mode, gr.lds));
        gr.resident = pic_gpd_resident(dim, order, gr.mode, gr.lds);
        gr.lds_k.assign(std::max(1, S.sort_interval), 0);
        gr.res_k.assign(gr.lds_k.size(), 1);
        for (size_t k = 0; k < gr.lds_k.size(); k++) {
          for (size_t i = 0; i < S.inst.size(); i++) {
            const Instance& I = S.inst[i];
            if (I.g.dim != dim || I.g.order != order || kernel_mode(I.g) != mode) continue;
            gr.lds_k[k] = std::max(gr.lds_k[k], pic_gpd_lds_bytes_step(I.g, (int)k));
          }
          gr.lds_k[k] = std::min(gr.lds_k[k], gr.lds);
          gr.res_k[k] = pic_gpd_resident(dim, order, gr.mode, gr.lds_k[k]);
        }
        S.sgroups.push_back(gr);
      }
    }
  std::vector<InstDesc> insts;
  for (int dim = 2; dim <= 3; dim++) {
    Group gr{dim, 0, (int)insts.size(), 0, 0, 0, 0, 0, 0, false, {0, 0, 0}, 0, false};
    for (size_t i = 0; i < S.inst.size(); i++) {
      Instance& I = S.inst[i];
      if (I.g.dim != dim) continue;
      InstDesc id{};
      id.g = I.g;
      id.F[0] = I.F[0];
      id.F[1] = I.F[1];
      for (int k = 0; k < 2; k++) {
        id.Jacc[k] = I.Jacc[k];
        id.J64[k] = I.J64[k];
      }
      id.Jout = I.Jout;
      int npass = 0;
      for (int a = 0; a < 3; a++) {
        const int lv = a < I.g.dim ? I.cfg.smooth_level[a] : 0;
        id.sm_level[a] = lv;
        id.sm_first[a] = npass;
        npass += lv;
        for (int p = 0; p < lv; p++) {
          const double* wt = I.cfg.smooth_weights[a][p];
          const double s = wt[0] + wt[1] + wt[2];
          for (int k = 0; k < 3; k++) id.sm_w[a][p][k] = (float)(wt[k] / s);
        }
      }
      id.sm_npass = npass;
      if (npass > 0) {
        const bool tiles = !I.g.cyl && pic_smooth_in_tiles(I.g.dim, id.sm_level);
        for (int a = 0; a < 3; a++) {
          int& most = tiles ? gr.sm_tiles_max[a] : gr.sm_max[a];
          most = std::max(most, id.sm_level[a]);
        }
        if (tiles) gr.sm_tiles = std::max(gr.sm_tiles, pic_smooth_tiles(I.g.dim, I.g.nx));
      }
      id.Jsm[0] = I.Jsm[0];
      id.Jsm[1] = I.Jsm[1];
      id.win = I.win;
      id.emax = I.emax;
      if (I.cfg.move_window) {
        int ppc = 1;
        for (int a = 0; a < I.g.dim; a++) ppc *= I.cfg.inject_ppc[a];
        id.win_inject = ppc * (I.g.ncell / I.g.nx[0]);
        gr.window = true;
      }
      insts.push_back(id);
      if (I.g.cyl)
        gr.cyl = true;
      else
        gr.cart = true;
      if (I.g.acc_mode == PIC_ACC_FIXED64) gr.fixed64 = true;
      gr.count++;
      gr.max_ncell = std::max(gr.max_ncell, I.g.ncell);
      if (dim == 3) (pic_yee_marches(I.g.nx) ? gr.march : gr.tiles3) = true;
    }
    // (a group with a moving window takes the tiles for every instance)
    for (size_t i = 0; i < S.inst.size(); i++)
      if (S.inst[i].g.dim == dim) gr.max_tiles = std::max(gr.max_tiles, pic_yee_tiles(dim, S.inst[i].g.nx, gr.window));
    if (gr.count > 0) S.igroups.push_back(gr);
  }
  if ((int)stores.size() > S.d_stores_cap) {
    if (S.d_stores) (void)hipFree(S.d_stores);
    S.d_stores = nullptr;
    int cap = std::max<int>((int)stores.size(), 4);
    HIPCHK(S, hipMalloc(&S.d_stores, cap * sizeof(StoreDesc)));
    S.d_stores_cap = cap;
  }
  if (!stores.empty())
    HIPCHK(S, hipMemcpy(S.d_stores, stores.data(), stores.size() * sizeof(StoreDesc), hipMemcpyHostToDevice));
  if (S.d_inst) (void)hipFree(S.d_inst);
  S.d_inst = nullptr;
  HIPCHK(S, hipMalloc(&S.d_inst, std::max<size_t>(insts.size(), 1) * sizeof(InstDesc)));
  HIPCHK(S, hipMemcpy(S.d_inst, insts.data(), insts.size() * sizeof(InstDesc), hipMemcpyHostToDevice));
  for (int k = 0; k < 2; k++)
    if (S.cycle_exec[k]) {
      (void)hipGraphExecDestroy(S.cycle_exec[k]);
      S.cycle_exec[k] = nullptr;
    }
  S.dirty = false;
  return PIC_OK;
}

int inst_desc_index(const Sim& S, int i) {
  // position of instance i in the dimension-grouped InstDesc array
  int pos = 0;
  for (int dim = 2; dim <= 3; dim++)
    for (size_t k = 0; k < S.inst.size(); k++) {
      if (S.inst[k].g.dim != dim) continue;
      if ((int)k == i) return pos;
      pos++;
    }
  return -1;
}

int store_desc_index(const Sim& S, int i, int s) {
  for (size_t k = 0; k < S.store_inst.size(); k++)
    if (S.store_inst[k] == i && S.store_species[k] == s) return (int)k;
  return -1;
}

hipEvent_t take_event(Sim& S) {
  if (!S.ev_free.empty()) {
    hipEvent_t e = S.ev_free.back();
    S.ev_free.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}

// Record a start event for kernel family f (profiling only); returns it.
hipEvent_t prof_begin(Sim& S) {
  if (!S.profiling) return nullptr;
  hipEvent_t e = take_event(S);
  if (e) (void)hipEventRecord(e, S.stream);
  return e;
}

void prof_end(Sim& S, int f, hipEvent_t start) {
  if (!S.profiling || !start) return;
  hipEvent_t e = take_event(S);
  if (!e) return;
  (void)hipEventRecord(e, S.stream);
  S.ev_pending[f].push_back({start, e});
}

pic_status prof_collect(Sim& S) {
  HIPCHK(S, hipStreamSynchronize(S.stream));
  for (int f = 0; f < 3; f++) {
    for (auto& pr : S.ev_pending[f]) {
      float ms = 0.0f;
      HIPCHK(S, hipEventElapsedTime(&ms, pr.first, pr.second));
      S.prof_ms[f] += ms;
      S.prof_n[f] += 1.0;
      S.ev_free.push_back(pr.first);
      S.ev_free.push_back(pr.second);
    }
    S.ev_pending[f].clear();
  }
  return PIC_OK;
}

// Launch nsteps steps starting at global step 'first' (whose parity picks
// the current accumulator of each step).
// 'first' only sets the parity of each step; phase0 is the number of steps
// done since the last rebin check when the first of them starts.
pic_status launch_steps(Sim& S, int64_t first, int nsteps, bool end_with_check, int phase0) {
  for (int k = 0; k < nsteps; k++) {
    const int par = (int)((first + k) & 1);
    // profiling: the particle family's events are stamped at the start of its
    // first kernel and the end of its last one
    hipEvent_t p0 = nullptr, p1 = nullptr;
    if (S.profiling && !S.sgroups.empty()) {
      p0 = take_event(S);
      p1 = take_event(S);
      if (!p0 || !p1) p0 = p1 = nullptr;
    }
    for (size_t q = 0; q < S.sgroups.size(); q++) {
      const Group& gr = S.sgroups[q];
      // one full wave of resident workgroups: a partial second wave would
      // leave the kernel's tail to a fraction of the chip.  The step's LDS
      // (and with it the workgroups per CU) follows its halo.
      const int kk = std::min<int>(phase0 + k, (int)gr.lds_k.size() - 1);
      const size_t lds = gr.lds_k.empty() ? gr.lds : gr.lds_k[kk];
      const int res = gr.res_k.empty() ? gr.resident : gr.res_k[kk];
      int grid = std::max(1, std::min(gr.max_items, S.num_cu * res));
      HIPCHK(S, pic_launch_gpd(gr.dim, gr.order, gr.mode, S.d_stores + gr.first, gr.count, grid, lds, par,
                               phase0 + k, end_with_check && k == nsteps - 1, S.stream, q == 0 ? p0 : nullptr,
                               q + 1 == S.sgroups.size() ? p1 : nullptr));
    }
    if (p0) S.ev_pending[0].push_back({p0, p1});
    hipEvent_t e0 = prof_begin(S);
    for (const Group& gr : S.igroups)
      if (gr.sm_tiles > 0)
        HIPCHK(S, pic_launch_smooth_tiles(S.d_inst + gr.first, gr.count, gr.dim, gr.sm_tiles, gr.sm_tiles_max, par,
                                          S.stream));
    for (const Group& gr : S.igroups)
      for (int a = 0; a < gr.dim; a++)
        for (int lev = 0; lev < gr.sm_max[a]; lev++)
          HIPCHK(S, pic_launch_smooth_pass(S.d_inst + gr.first, gr.count, gr.max_ncell, a, lev, par, S.stream));
    const bool check = end_with_check && k == nsteps - 1;
    for (const Group& gr : S.igroups) {
      // the group's stores (the store groups are in order of dimension)
      int first = 0, plan = 0;
      for (const Group& sg : S.sgroups) {
        if (sg.dim < gr.dim) first += sg.count;
        if (check && sg.dim == gr.dim) plan += sg.count;
      }
      HIPCHK(S, pic_launch_yee_step(S.d_inst + gr.first, gr.count, gr.max_tiles, gr.dim, gr.cart, gr.cyl,
                                    gr.window, gr.march, gr.tiles3, par, S.d_stores + first, plan, S.stream));
    }
    prof_end(S, 1, e0);
    if (check) {
      e0 = prof_begin(S);
      for (const Group& gr : S.sgroups)
        HIPCHK(S, pic_launch_rebin(S.d_stores + gr.first, gr.count, gr.max_items, gr.max_tiles, gr.max_blocks,
                                   gr.big, gr.inject_max, gr.thermal, par, S.stream));
      prof_end(S, 2, e0);
    }
  }
  return PIC_OK;
}

pic_status capture_cycle(Sim& S, int par) {
  if (S.cycle_exec[par]) return PIC_OK;
  hipGraph_t graph = nullptr;
  HIPCHK(S, hipStreamBeginCapture(S.stream, hipStreamCaptureModeThreadLocal));
  pic_status st = launch_steps(S, par, S.sort_interval, true, 0);  // a cycle starts after a check
  hipError_t e = hipStreamEndCapture(S.stream, &graph);
  if (st != PIC_OK) {
    if (graph) (void)hipGraphDestroy(graph);
    return st;
  }
  if (e != hipSuccess) return S.fail(PIC_E_HIP, "graph capture failed: %s", hipGetErrorString(e));
  e = hipGraphInstantiate(&S.cycle_exec[par], graph, nullptr, nullptr, 0);
  (void)hipGraphDestroy(graph);
  if (e != hipSuccess) {
    S.cycle_exec[par] = nullptr;
    return S.fail(PIC_E_HIP, "graph instantiate failed: %s", hipGetErrorString(e));
  }
  return PIC_OK;
}

pic_status settle_tiles(Sim& S);

pic_status sim_step(Sim& S, int64_t nsteps) {
  if (nsteps < 0) return S.fail(PIC_E_INVALID, "nsteps < 0");
  if (nsteps == 0) return PIC_OK;
  pic_status st = settle_tiles(S);
  if (st == PIC_OK) st = refresh_descriptors(S);
  if (st != PIC_OK) return st;
  if (S.sgroups.empty() && S.igroups.empty()) return PIC_OK;
  const int SI = S.sort_interval;
  S.ctl_current = false;
  int64_t done = 0;
  while (done < nsteps) {
    int64_t phase = S.steps % SI;  // steps already done in the current cycle
    int64_t left = nsteps - done;
    if (phase == 0 && left >= SI && S.use_graph && !S.profiling) {
      const int par = (int)(S.steps & 1);
      st = capture_cycle(S, par);
      if (st != PIC_OK) return st;
      HIPCHK(S, hipGraphLaunch(S.cycle_exec[par], S.stream));
      S.steps += SI;
      done += SI;
      continue;
    }
    int64_t run = std::min<int64_t>(left, SI - phase);
    bool check = (phase + run == SI);
    st = launch_steps(S, S.steps, (int)run, check, (int)phase);
    if (st != PIC_OK) return st;
    S.steps += run;
    done += run;
  }
  for (Instance& I : S.inst) I.steps = S.steps;
  return PIC_OK;
}

// Host copy of an instance's moving-window state (zero without a window).
pic_status read_win(Sim& S, const Instance& I, WinCtl& w) {
  memset(&w, 0, sizeof w);
  if (!I.win) return PIC_OK;
  HIPCHK(S, hipMemcpy(&w, I.win + (S.steps & 1), sizeof w, hipMemcpyDeviceToHost));
  return PIC_OK;
}

// Host copy of a store's control words (after sim_sync).
const StoreCtl& host_ctl(const Sim& S, const Species& sp) { return S.h_ctl[sp.ctl - S.d_ctl]; }

// Raise a store's bound on |u| to at least um, for either parity of the next step.
void raise_umax(StoreCtl& c, float um) {
  c.umax[0] = c.umax[1] = std::max(um, std::max(c.umax[0], c.umax[1]));
}

// Wait for the stream and bring the host's control words up to date: one copy
// and one wait for all stores.  (One blocking copy per store made every
// diagnostic of a 24-instance batch cost 390 us.)
pic_status sim_sync(Sim& S) {
  size_t used = 0;  // up to the last species in use
  if (!S.ctl_current)
    for (size_t i = 0; i < S.inst.size(); i++)
      for (size_t s = 0; s < PIC_MAX_SPECIES; s++)
        if (S.inst[i].sp[s].used && S.inst[i].sp[s].ctl) used = i * PIC_MAX_SPECIES + s + 1;
  if (used > 0)
    HIPCHK(S, hipMemcpyAsync(S.h_ctl.data(), S.d_ctl, used * sizeof(StoreCtl), hipMemcpyDeviceToHost, S.stream));
  HIPCHK(S, hipStreamSynchronize(S.stream));
  S.ctl_current = true;
  for (Instance& I : S.inst)
    for (Species& sp : I.sp) {
      if (!sp.used || !sp.ctl) continue;
      const StoreCtl& c = host_ctl(S, sp);
      if (c.bad) return S.fail(PIC_E_STATE, "a particle left the region staged for its tile");
      if ((I.cfg.move_window || I.g.cyl) && c.nchecks > 0 && c.np != sp.np) {
        // a moving window removed and injected particles, or the r-z wall
        // removed some
        sp.np = c.np;
        sp.desc.np = c.np;
        S.dirty = true;
      }
    }
  return PIC_OK;
}

// ---------------------------------------------------------------------------
// loading
// ---------------------------------------------------------------------------

struct HostParticles {
  std::vector<int> cell, id;
  std::vector<float> eps[3], u[3], w;
  void resize(size_t n) {
    cell.resize(n);
    id.resize(n);
    for (auto& v : eps) v.resize(n);
    for (auto& v : u) v.resize(n);
    w.resize(n);
  }
};

pic_status read_back(Sim& S, Species& sp, int dim, HostParticles& h) {
  h.resize(sp.np);
  if (sp.np == 0) return PIC_OK;
  StoreCtl c{};
  HIPCHK(S, hipMemcpy(&c, sp.ctl, sizeof c, hipMemcpyDeviceToHost));
  const int s = pic_cur(c);
  const StoreDesc& d = sp.desc;
  size_t n = sp.np;
  HIPCHK(S, hipMemcpy(h.cell.data(), d.cell[s], n * 4, hipMemcpyDeviceToHost));
  HIPCHK(S, hipMemcpy(h.id.data(), d.id[s], n * 4, hipMemcpyDeviceToHost));
  for (int k = 0; k < dim; k++) HIPCHK(S, hipMemcpy(h.eps[k].data(), d.eps[s][k], n * 4, hipMemcpyDeviceToHost));
  for (int k = 0; k < 3; k++) HIPCHK(S, hipMemcpy(h.u[k].data(), d.u[s][k], n * 4, hipMemcpyDeviceToHost));
  HIPCHK(S, hipMemcpy(h.w.data(), d.w[s], n * 4, hipMemcpyDeviceToHost));
  return PIC_OK;
}

// Particles binned by tile on the host, ready for upload as buffer set 0.
struct Binned {
  HostParticles o;
  std::vector<int> toff, ioff;
  std::vector<Item> items;
};

// Stable bin by tile; inside a tile the k-th particle of every cell, cell by
// cell, for k = 0, 1, ... (neighbouring lanes of a wavefront then sit in
// different cells and their current deposits hit different LDS addresses).
// Work items of at most 'chunk' particles per tile.  Pure host code.
void bin_particles(const GridDesc& g, int chunk, const HostParticles& h, Binned& B) {
  const size_t n = h.cell.size();
  std::vector<int> tile(n), count(g.ntiles + 1, 0);
  for (size_t p = 0; p < n; p++) {
    int c[3];
    pic_unpack(g, h.cell[p], c);
    int t = pic_tile_index(g, c[0] / g.tile[0], c[1] / g.tile[1], g.dim == 3 ? c[2] / g.tile[2] : 0);
    tile[p] = t;
    count[t + 1]++;
  }
  std::vector<int>& toff = B.toff;
  toff.assign(g.ntiles + 1, 0);
  for (int t = 0; t < g.ntiles; t++) toff[t + 1] = toff[t] + count[t + 1];
  std::vector<int> order(n), slotpos(n);
  {
    std::vector<int> pos(toff.begin(), toff.end() - 1);
    for (size_t p = 0; p < n; p++) order[pos[tile[p]]++] = (int)p;  // stable by tile
    // per tile: rank of each particle within its cell, then a counting sort
    // by rank (stable, so cells keep their order inside a rank)
    const int tvol = g.tile[0] * g.tile[1] * g.tile[2];
    std::vector<int> seen(tvol, 0), lc, rk, bucket;
    for (int t = 0; t < g.ntiles; t++) {
      int a = toff[t], b = toff[t + 1];
      if (b - a < 2) continue;
      int tc[3];
      pic_tile_coords(g, t, tc);
      lc.resize(b - a);
      rk.resize(b - a);
      int maxr = 0;
      for (int k = a; k < b; k++) {
        int c[3];
        pic_unpack(g, h.cell[order[k]], c);
        int l0 = c[0] - tc[0] * g.tile[0], l1 = c[1] - tc[1] * g.tile[1];
        int l2 = g.dim == 3 ? c[2] - tc[2] * g.tile[2] : 0;
        int li = l0 + g.tile[0] * (l1 + g.tile[1] * l2);
        lc[k - a] = li;
        rk[k - a] = seen[li]++;
        maxr = std::max(maxr, rk[k - a]);
      }
      bucket.assign(maxr + 2, 0);
      for (int k = 0; k < b - a; k++) bucket[rk[k] + 1]++;
      for (int r = 0; r <= maxr; r++) bucket[r + 1] += bucket[r];
      for (int k = 0; k < b - a; k++) slotpos[bucket[rk[k]]++] = order[a + k];
      for (int k = 0; k < b - a; k++) order[a + k] = slotpos[k];
      for (int k = 0; k < b - a; k++) seen[lc[k]] = 0;
    }
  }
  HostParticles& o = B.o;
  o.resize(n);
  for (size_t q = 0; q < n; q++) {
    size_t p = (size_t)order[q];
    o.cell[q] = h.cell[p];
    o.id[q] = h.id[p];
    for (int k = 0; k < 3; k++) {
      o.eps[k][q] = h.eps[k][p];
      o.u[k][q] = h.u[k][p];
    }
    o.w[q] = h.w[p];
  }
  B.ioff.assign(g.ntiles + 1, 0);
  B.items.clear();
  for (int t = 0; t < g.ntiles; t++) {
    int c = toff[t + 1] - toff[t];
    B.ioff[t] = (int)B.items.size();
    const int size = pic_item_size(c, chunk);
    for (int b = 0; b < c; b += size) B.items.push_back(Item{t, toff[t] + b, toff[t] + std::min(c, b + size), 0});
  }
  B.ioff[g.ntiles] = (int)B.items.size();
}

// Upload binned particles as buffer set 0 and reset the store's control block.
pic_status upload_bins(Sim& S, Species& sp, const Binned& B) {
  const HostParticles& o = B.o;
  const size_t n = o.cell.size();
  const int dim = sp.desc.g.dim;
  if ((int)B.items.size() > sp.max_items) return S.fail(PIC_E_NOMEM, "work item list overflow");
  const StoreDesc& d = sp.desc;
  if (n > 0) {
    HIPCHK(S, hipMemcpy(d.cell[0], o.cell.data(), n * 4, hipMemcpyHostToDevice));
    HIPCHK(S, hipMemcpy(d.id[0], o.id.data(), n * 4, hipMemcpyHostToDevice));
    for (int k = 0; k < dim; k++) HIPCHK(S, hipMemcpy(d.eps[0][k], o.eps[k].data(), n * 4, hipMemcpyHostToDevice));
    for (int k = 0; k < 3; k++) HIPCHK(S, hipMemcpy(d.u[0][k], o.u[k].data(), n * 4, hipMemcpyHostToDevice));
    HIPCHK(S, hipMemcpy(d.w[0], o.w.data(), n * 4, hipMemcpyHostToDevice));
  }
  HIPCHK(S, hipMemcpy(d.toff[0], B.toff.data(), B.toff.size() * 4, hipMemcpyHostToDevice));
  HIPCHK(S, hipMemcpy(d.ioff[0], B.ioff.data(), B.ioff.size() * 4, hipMemcpyHostToDevice));
  if (!B.items.empty())
    HIPCHK(S, hipMemcpy(d.items[0], B.items.data(), B.items.size() * sizeof(Item), hipMemcpyHostToDevice));
  StoreCtl c{};
  HIPCHK(S, hipMemcpy(&c, sp.ctl, sizeof c, hipMemcpyDeviceToHost));
  c.cur = 0;
  c.pending = 0;
  c.flag = 0;
  c.active = 0;
  c.bad = 0;
  c.n_items[0] = (int)B.items.size();
  c.n_items[1] = 0;
  c.sorted = 1;  // binned exactly: every particle in its own tile
  // the one-phase kernels' bound on |u| covers every particle uploaded
  double um = 0.0;
  for (size_t q = 0; q < n; q++)
    um = std::max(um, std::sqrt((double)o.u[0][q] * o.u[0][q] + (double)o.u[1][q] * o.u[1][q] +
                                (double)o.u[2][q] * o.u[2][q]));
  raise_umax(c, std::nextafter((float)(um * (1.0 + 1e-6)), INFINITY));
  HIPCHK(S, hipMemcpy(sp.ctl, &c, sizeof c, hipMemcpyHostToDevice));
  S.ctl_current = false;
  sp.np = (int64_t)n;
  sp.desc.np = (int)n;
  S.dirty = true;
  return PIC_OK;
}

pic_status upload_binned(Sim& S, Instance& I, Species& sp, const HostParticles& h) {
  Binned B;
  bin_particles(I.g, sp.desc.chunk, h, B);
  return upload_bins(S, sp, B);
}

// Run f(0..n-1) on up to 'most' host threads, the caller's among them (alone if
// no other can be started).
template <class F>
void parallel_for(int n, F f, unsigned most = 16) {
  unsigned hc = std::thread::hardware_concurrency();
  const int nt = std::max(1, std::min(n, (int)std::min(most, hc ? hc : 1u)));
  std::atomic<int> next{0};
  auto work = [&]() {
    for (int i; (i = next.fetch_add(1)) < n;) f(i);
  };
  std::vector<std::thread> th;
  try {
    for (int t = 1; t < nt; t++) th.emplace_back(work);
  } catch (const std::exception&) {
  }
  work();
  for (auto& x : th) x.join();
}

pic_status copy_in(Sim& S, std::vector<double>& dst, const double* src, size_t n, uint32_t flags) {
  dst.resize(n);
  if (n == 0) return PIC_OK;
  if (flags & PIC_DEVICE_PTRS)
    HIPCHK(S, hipMemcpy(dst.data(), src, n * sizeof(double), hipMemcpyDeviceToHost));
  else
    memcpy(dst.data(), src, n * sizeof(double));
  return PIC_OK;
}

pic_status build_tables(Sim& S, Instance& I);

int64_t instance_particles(const Instance& I);

// Whether the library chooses the instance's tile by its particles per cell
// (periodic 3D boxes without asked-for extents), and has not settled it yet.
// Until the first step with particles, each load that finds the instance empty
// chooses the tile, and that step chooses it again by everything loaded: a
// driver bunch loaded before the plasma, or a plasma loaded in slices, looks
// like a box of few particles per cell.
bool tile_open(const Instance& I) {
  bool asked = false;
  for (int d = 0; d < I.g.dim; d++) asked = asked || I.cfg.tile[d] != 0;
  return !I.settled && !asked && pic_gpd_split(I.g);
}

// The grid n more particles would be loaded into; nothing of it is in force
// before take_tiles.
pic_status tiles_for(Sim& S, const Instance& I, int64_t n, GridDesc& g) {
  g = I.g;
  if (n == 0 || !tile_open(I) || instance_particles(I) > 0) return PIC_OK;
  return setup_grid(S, I.cfg, S.sort_interval, g, (double)n / I.g.ncell);
}

bool same_tiles(const GridDesc& a, const GridDesc& b) {
  return a.tile[0] == b.tile[0] && a.tile[1] == b.tile[1] && a.tile[2] == b.tile[2];
}

// Put the tiles of g, chosen by n particles, in force in an instance without
// particles, once a load has passed its checks; its stores, if any, are allocated
// anew.
pic_status take_tiles(Sim& S, Instance& I, const GridDesc& g, int64_t n) {
  if (tile_open(I) && instance_particles(I) == 0) I.tiled_for = n;
  if (same_tiles(g, I.g)) return I.ndst ? PIC_OK : build_tables(S, I);
  for (Species& sp : I.sp)
    if (sp.used) free_species(sp);
  I.g = g;
  S.dirty = true;
  return build_tables(S, I);
}

pic_status diag_scratch(Sim& S, size_t bytes, char** p);

// What a load has to allocate for a store of 'total' particles.
int64_t wanted_capacity(const Instance& I, int species, int64_t total) {
  if (!I.cfg.move_window || species != 0) return total;
  // room for the window's plasma: a full window of injected lattice plus two
  // columns in flight
  int64_t ppc = 1;
  for (int a = 0; a < I.g.dim; a++) ppc *= I.cfg.inject_ppc[a];
  const int64_t col = ppc * (I.g.ncell / I.g.nx[0]);
  return std::max<int64_t>(total, ppc * I.g.ncell) + 2 * col + 1024;
}

// A store's injection settings, its species' largest weight and the units of
// the instance, once the new particles' largest weight is known.
void settle_species(Instance& I, int species, double wm) {
  Species& sp = I.sp[species];
  I.wmax[species] = std::max(I.wmax[species], wm);
  if (I.cfg.move_window && species == 0) {
    for (int a = 0; a < 3; a++) sp.desc.inj_ppc[a] = a < I.g.dim ? I.cfg.inject_ppc[a] : 1;
    sp.desc.inj_w = (float)I.cfg.inject_w;
    sp.desc.inj_uth = I.cfg.inject_uth;
    sp.desc.inj_seed = I.cfg.inject_seed;
    // r-z: injected weights grow with the radius, up to (nr - 1/2) inject_w
    const double wi = std::fabs(I.cfg.inject_w) * (I.g.cyl ? (double)I.g.nx[1] - 0.5 : 1.0);
    I.wmax[0] = std::max(I.wmax[0], wi);
  }
  set_current_scale(I);
}

// Bound on |u| that also covers what a thermal window can inject (a Box-Muller
// deviate from 53-bit uniforms is at most sqrt(2 * 53 ln 2) = 8.5717 per
// component).
float inject_umax(const Instance& I, int species) {
  if (!I.cfg.move_window || species != 0 || !(I.cfg.inject_uth > 0.0)) return 0.0f;
  return (float)(8.5718 * std::sqrt(3.0) * I.cfg.inject_uth * (1.0 + 1e-6));
}

// Device memory of a load: small ones use the diagnostics' scratch, large ones
// memory of their own, freed at the end.
struct LoadMem {
  char* at = nullptr;
  void* own = nullptr;
  LoadMem() = default;
  LoadMem(const LoadMem&) = delete;
  LoadMem& operator=(const LoadMem&) = delete;
  ~LoadMem() { (void)hipFree(own); }
  bool get(Sim& S, size_t bytes) {
    if (bytes <= ((size_t)64 << 20)) {
      if (diag_scratch(S, bytes, &at) != PIC_OK) at = nullptr;
    } else if (hipMalloc(&own, bytes) == hipSuccess) {
      at = (char*)own;
    } else {
      own = nullptr;
    }
    if (!at) (void)hipGetLastError();
    return at != nullptr;
  }
  char* take(size_t b) {
    char* p = at;
    at += align256(b);
    return p;
  }
};

// Keys of a load (pic_load_key).
size_t load_keys(const GridDesc& g) { return (size_t)g.ntiles * g.tile[0] * g.tile[1] * g.tile[2]; }

// What load_args takes for a store of 'total' particles.
size_t load_bytes(const GridDesc& g, int64_t total) {
  return 256 + align256(load_keys(g) * 4) + align256((size_t)g.ntiles * 4) + 2 * align256((size_t)total * 4);
}

// A load of 'old' stored and n new particles into the tiles of g.
LoadArgs load_args(const GridDesc& g, int64_t old, int64_t n, LoadMem& mem) {
  LoadArgs A{};
  A.g = g;
  A.old = old;
  A.n = n;
  A.status = (LoadStatus*)mem.take(sizeof(LoadStatus));
  static_assert(sizeof(LoadStatus) <= 256, "room for the status");
  A.cells = (int*)mem.take(load_keys(g) * 4);
  A.tiles = (int*)mem.take((size_t)g.ntiles * 4);
  A.rank = (int*)mem.take((size_t)(old + n) * 4);
  A.slot = (int*)mem.take((size_t)(old + n) * 4);
  return A;
}

// The stored particles: buffer set 'cur' of d.
void load_from(LoadArgs& A, const StoreDesc& d, int cur) {
  A.ocell = d.cell[cur];
  A.oid = d.id[cur];
  for (int k = 0; k < 3; k++) {
    A.oeps[k] = d.eps[cur][k];
    A.ou[k] = d.u[cur][k];
  }
  A.ow = d.w[cur];
}

pic_status load_count(Sim& S, const LoadArgs& A, LoadStatus& ls) {
  ls = LoadStatus{};
  ls.first = ~0ull;
  ls.idmax = -1;
  HIPCHK(S, hipMemcpy(A.status, &ls, sizeof ls, hipMemcpyHostToDevice));
  HIPCHK(S, hipMemsetAsync(A.cells, 0, load_keys(A.g) * 4, nullptr));
  HIPCHK(S, pic_launch_load_count(A, nullptr));
  HIPCHK(S, hipMemcpy(&ls, A.status, sizeof ls, hipMemcpyDeviceToHost));
  return PIC_OK;
}

pic_status load_place(Sim& S, const LoadArgs& A, const Species& sp, int set, LoadStatus& ls) {
  HIPCHK(S, pic_launch_load_place(A, sp.desc, set, nullptr));
  HIPCHK(S, hipMemcpy(&ls, A.status, sizeof ls, hipMemcpyDeviceToHost));
  if (ls.items > sp.max_items) return S.fail(PIC_E_NOMEM, "work item list overflow");
  return PIC_OK;
}

// Control words of a store whose particles a load has put into buffer set 'set'.
void load_ctl(StoreCtl& c, int set, const LoadStatus& ls) {
  c.cur = set;
  c.pending = c.flag = c.active = c.bad = 0;
  c.n_items[set] = ls.items;
  c.n_items[1 - set] = 0;
  c.sorted = 1;  // binned exactly: every particle in its own tile
  // the one-phase kernels' bound on |u| covers every particle of the store
  double u2;
  memcpy(&u2, &ls.u2, 8);
  raise_umax(c, std::nextafter((float)(std::sqrt(u2) * (1.0 + 1e-6)), INFINITY));
}

// The load on the device.  *done stays false where the host's path has to take
// the call: a state that is reported after the input's own checks, or too
// little device memory for both the old and the new arrays.  The kernels run
// on the null stream, as the copies of the host's path do, so they see what
// was queued there (and on blocking streams) to produce the input.
pic_status load_device(Sim& S, Instance& I, int species, double rqm, int64_t n, const double* x, const double* u,
                       const double* w, uint32_t flags, bool* done) {
  Species& sp = I.sp[species];
  const bool win = I.cfg.move_window != 0, rz = I.g.cyl != 0;
  if (sim_sync(S) != PIC_OK) return PIC_OK;  // fresh particle counts (moving window)
  const int64_t old = sp.np, total = old + n;
  if ((I.cfg.capacity > 0 && total > I.cfg.capacity) || total > 0x7fffff00LL) return PIC_OK;
  if (win && species != 0 && !I.sp[0].used) return PIC_OK;
  GridDesc g;
  if (tiles_for(S, I, n, g) != PIC_OK) return PIC_OK;
  // (the table of tiles that stay needs no checks of the input, and is made
  // before its kernels are queued)
  if (!I.ndst && same_tiles(g, I.g) && build_tables(S, I) != PIC_OK) return PIC_OK;
  WinCtl wc;
  pic_status st = read_win(S, I, wc);
  if (st != PIC_OK) return st;
  // input the kernels can read: memory of this device, aligned; else a copy
  const double* in[3] = {x, u, w};
  size_t in_bytes[3] = {(size_t)n * g.dim * 8, (size_t)n * 24, (size_t)n * 8}, stage = 0;
  bool copy[3];
  for (int k = 0; k < 3; k++) {
    hipPointerAttribute_t pa;
    copy[k] = true;
    if ((flags & PIC_DEVICE_PTRS) && ((uintptr_t)in[k] & 7) == 0) {
      if (hipPointerGetAttributes(&pa, in[k]) == hipSuccess)
        copy[k] = pa.type != hipMemoryTypeDevice || pa.device != S.device;
      else
        (void)hipGetLastError();
    }
    if (copy[k]) stage += align256(in_bytes[k]);
  }
  LoadMem mem;
  if (!mem.get(S, load_bytes(g, total) + stage)) return PIC_OK;
  *done = true;
  LoadArgs A = load_args(g, old, n, mem);
  for (int d = 0; d < 3; d++) A.xmin[d] = I.cfg.xmin[d];
  A.shifts = wc.shifts;
  A.origin = wc.origin;
  for (int k = 0; k < 3; k++)
    if (copy[k]) {
      char* p = mem.take(in_bytes[k]);
      HIPCHK(S, hipMemcpy(p, in[k], in_bytes[k], (flags & PIC_DEVICE_PTRS) ? hipMemcpyDefault : hipMemcpyHostToDevice));
      in[k] = (const double*)p;
    }
  A.x = in[0];
  A.u = in[1];
  A.w = in[2];
  StoreCtl c{};
  int set = 0;
  if (sp.used && sp.ctl) {  // (also an emptied store keeps its counters)
    c = host_ctl(S, sp);
    if (old > 0) load_from(A, sp.desc, pic_cur(c));
    set = 1 - pic_cur(c);  // (the set read from stays as it is)
  }
  LoadStatus ls;
  if ((st = load_count(S, A, ls)) != PIC_OK) return st;
  if (ls.flags & 1) return S.fail(PIC_E_RANGE, "non-finite position");
  if (ls.flags & 2) return S.fail(PIC_E_RANGE, "non-finite momentum");
  if (ls.flags & 4) return S.fail(PIC_E_RANGE, "non-finite weight");
  A.id0 = win ? wc.next_id : (rz ? (int64_t)ls.idmax + 1 : old);
  if (rz && A.id0 + n > 0x7fffff00LL) return S.fail(PIC_E_NOMEM, "particle ids exhausted");
  if (ls.first != ~0ull)
    return (ls.first & 1) ? S.fail(PIC_E_RANGE, "particle radius outside [0, (nr - 1/2) dr)")
                          : S.fail(PIC_E_RANGE, "particle outside the moving window");
  double wm;
  memcpy(&wm, &ls.w, 8);
  if ((st = take_tiles(S, I, g, n)) != PIC_OK) return st;
  const int64_t want = wanted_capacity(I, species, total);
  Species keep;  // the arrays the load reads from, until it is done
  if (!sp.used || want > sp.cap) {
    keep = sp;
    sp.allocs.clear();
    const int64_t cap = I.cfg.capacity > 0 ? std::max<int64_t>(I.cfg.capacity, want) : want;
    const int chunk = I.cfg.chunk > 0 ? I.cfg.chunk : default_chunk(S, I.cfg, I.g, want);
    if (alloc_species(S, I, sp, std::max<int64_t>(cap, 1), chunk) != PIC_OK) {
      (void)hipGetLastError();
      for (void* p : sp.allocs) (void)hipFree(p);
      sp = keep;
      if (sp.ctl) HIPCHK(S, hipMemcpy(sp.ctl, &c, sizeof c, hipMemcpyHostToDevice));
      *done = false;
      return PIC_OK;
    }
    sp.used = true;
    sp.rqm = rqm;
    sp.desc.qm = (float)(1.0 / rqm);
    set = 0;
    c = StoreCtl{};
  } else {
    grow_chunk(S, I, sp, want);
  }
  settle_species(I, species, wm);
  st = load_place(S, A, sp, set, ls);
  for (void* p : keep.allocs) (void)hipFree(p);
  if (st != PIC_OK) return st;
  load_ctl(c, set, ls);
  raise_umax(c, inject_umax(I, species));
  if (win || rz) c.np = (int)total;
  HIPCHK(S, hipMemcpy(sp.ctl, &c, sizeof c, hipMemcpyHostToDevice));
  S.ctl_current = false;
  sp.np = total;
  sp.desc.np = (int)total;
  S.dirty = true;
  if (win) {
    wc.next_id += n;
    HIPCHK(S, hipMemcpy(I.win + (S.steps & 1), &wc, sizeof wc, hipMemcpyHostToDevice));
  }
  return PIC_OK;
}

pic_status sim_load(Sim& S, int inst, int32_t species, double rqm, int64_t n, const double* x,
                    const double* u, const double* w, uint32_t flags) {
  if (inst < 0 || inst >= (int)S.inst.size()) return S.fail(PIC_E_INVALID, "instance %d out of range", inst);
  if (species < 0 || species >= PIC_MAX_SPECIES) return S.fail(PIC_E_INVALID, "species %d out of range", species);
  if (n < 0) return S.fail(PIC_E_INVALID, "n < 0");
  if (n > 0 && (!x || !u || !w)) return S.fail(PIC_E_INVALID, "null particle array");
  if (!std::isfinite(rqm) || rqm == 0.0) return S.fail(PIC_E_INVALID, "rqm must be finite and nonzero");
  Instance& I = S.inst[inst];
  Species& sp = I.sp[species];
  HIPCHK(S, hipStreamSynchronize(S.stream));
  if (sp.used && sp.rqm != rqm) return S.fail(PIC_E_INVALID, "rqm differs from the species' first load");
  const int dim = I.g.dim;
  pic_status st;
  if (n > 0) {
    bool done = false;
    st = load_device(S, I, species, rqm, n, x, u, w, flags, &done);
    if (done || st != PIC_OK) return st;
  }
  std::vector<double> hx, hu, hw;
  if ((st = copy_in(S, hx, x, (size_t)n * dim, flags)) != PIC_OK) return st;
  if ((st = copy_in(S, hu, u, (size_t)n * 3, flags)) != PIC_OK) return st;
  if ((st = copy_in(S, hw, w, (size_t)n, flags)) != PIC_OK) return st;
  for (double v : hx)
    if (!std::isfinite(v)) return S.fail(PIC_E_RANGE, "non-finite position");
  for (double v : hu)
    if (!std::isfinite(v)) return S.fail(PIC_E_RANGE, "non-finite momentum");
  for (double v : hw)
    if (!std::isfinite(v)) return S.fail(PIC_E_RANGE, "non-finite weight");
  const int64_t total = sp.np + n;
  if (I.cfg.capacity > 0 && total > I.cfg.capacity)
    return S.fail(PIC_E_NOMEM, "species %d would hold %lld particles, capacity %lld", species, (long long)total,
                  (long long)I.cfg.capacity);
  if (total > 0x7fffff00LL) return S.fail(PIC_E_NOMEM, "too many particles");
  if ((st = sim_sync(S)) != PIC_OK) return st;  // fresh particle counts (moving window)
  WinCtl wc;
  if ((st = read_win(S, I, wc)) != PIC_OK) return st;
  const bool win = I.cfg.move_window != 0;
  if (win && species != 0 && !I.sp[0].used)
    return S.fail(PIC_E_STATE, "with a moving window species 0 (the injected one) is loaded first");
  const bool rz = I.g.cyl != 0;
  HostParticles h;
  if ((st = read_back(S, sp, dim, h)) != PIC_OK) return st;
  const size_t old = h.cell.size();
  // ids continue after the largest one (the r-z wall may have removed some)
  int64_t id0 = (int64_t)old;
  if (rz) {
    id0 = 0;
    for (size_t q = 0; q < old; q++) id0 = std::max<int64_t>(id0, (int64_t)h.id[q] + 1);
    if (id0 + n > 0x7fffff00LL) return S.fail(PIC_E_NOMEM, "particle ids exhausted");
  }
  h.resize(old + n);
  for (int64_t p = 0; p < n; p++) {
    int c[3] = {0, 0, 0};
    for (int d = 0; d < dim; d++) {
      double L = (double)I.g.nx[d];
      double xi = (hx[p * dim + d] - I.cfg.xmin[d]) / I.cfg.dx[d];
      if (rz && d == 1) {
        // r-z: x2 is the radius; the cell coordinate is r/dr + 1/2
        xi = hx[p * dim + 1] / I.cfg.dx[1] + 0.5;
        if (!(hx[p * dim + 1] >= 0.0 && xi < L))
          return S.fail(PIC_E_RANGE, "particle radius outside [0, (nr - 1/2) dr)");
      }
      if (win && d == 0) {
        // window position, then ring column
        xi -= (double)wc.shifts;
        if (!(xi >= 0.0 && xi < L)) return S.fail(PIC_E_RANGE, "particle outside the moving window");
        xi += (double)wc.origin;
      }
      xi = std::fmod(xi, L);
      if (xi < 0.0) xi += L;
      if (xi >= L) xi -= L;
      double f = std::floor(xi);
      int ci = (int)f;
      float e = (float)(xi - f);
      if (e >= 1.0f) {
        e = 0.0f;
        ci += 1;
      }
      if (ci >= I.g.nx[d]) ci -= I.g.nx[d];
      c[d] = ci;
      h.eps[d][old + p] = e;
    }
    h.cell[old + p] = pic_pack(I.g, c[0], c[1], c[2]);
    h.id[old + p] = win ? (int)(wc.next_id + p) : (int)(id0 + p);
    for (int k = 0; k < 3; k++) h.u[k][old + p] = (float)hu[p * 3 + k];
    h.w[old + p] = (float)hw[p];
  }
  double wm = 0.0;
  for (double v : hw) wm = std::max(wm, std::fabs(v));
  GridDesc g;
  if ((st = tiles_for(S, I, n, g)) != PIC_OK || (st = take_tiles(S, I, g, n)) != PIC_OK) return st;
  const int64_t want = wanted_capacity(I, species, total);
  if (!sp.used || want > sp.cap) {
    int64_t cap = I.cfg.capacity > 0 ? std::max<int64_t>(I.cfg.capacity, want) : want;
    int chunk = I.cfg.chunk > 0 ? I.cfg.chunk : default_chunk(S, I.cfg, I.g, want);
    if ((st = alloc_species(S, I, sp, std::max<int64_t>(cap, 1), chunk)) != PIC_OK) return st;
    sp.used = true;
    sp.rqm = rqm;
    sp.desc.qm = (float)(1.0 / rqm);
  } else {
    grow_chunk(S, I, sp, want);
  }
  settle_species(I, species, wm);
  if (win) {
    wc.next_id += n;
    HIPCHK(S, hipMemcpy(I.win + (S.steps & 1), &wc, sizeof wc, hipMemcpyHostToDevice));
  }
  st = upload_binned(S, I, sp, h);
  if (st == PIC_OK && (win || rz)) {
    StoreCtl c{};
    HIPCHK(S, hipMemcpy(&c, sp.ctl, sizeof c, hipMemcpyDeviceToHost));
    c.np = (int)sp.np;
    raise_umax(c, inject_umax(I, species));
    HIPCHK(S, hipMemcpy(sp.ctl, &c, sizeof c, hipMemcpyHostToDevice));
    S.ctl_current = false;
  }
  return st;
}

// Move the stores of an instance into the tiles of g.  Where the memory does not
// hold the old and the new arrays together, the tiles stay as they are.
pic_status retile(Sim& S, Instance& I, const GridDesc& g) {
  pic_status st = sim_sync(S);
  if (st != PIC_OK) return st;
  const GridDesc g0 = I.g;
  int* const ndst0 = I.ndst;
  Species keep[PIC_MAX_SPECIES];
  StoreCtl ctl[PIC_MAX_SPECIES];
  int64_t most = 0;
  for (int s = 0; s < PIC_MAX_SPECIES; s++) {
    Species& sp = I.sp[s];
    if (!sp.used) continue;
    if (sp.np == 0) free_species(sp);  // (allocated at its next load)
    keep[s] = sp;
    if (sp.np == 0) continue;
    ctl[s] = host_ctl(S, sp);
    most = std::max(most, sp.np);
  }
  LoadMem mem;
  bool room = mem.get(S, load_bytes(g, most));
  I.g = g;
  I.ndst = nullptr;
  room = room && build_tables(S, I) == PIC_OK;
  for (int s = 0; s < PIC_MAX_SPECIES && room; s++) {
    Species& sp = I.sp[s];
    if (keep[s].np == 0) continue;
    sp.allocs.clear();
    room = alloc_species(S, I, sp, keep[s].cap, keep[s].desc.chunk) == PIC_OK;
    sp.np = keep[s].np;
    sp.desc.qm = keep[s].desc.qm;
  }
  if (!room) {
    (void)hipGetLastError();
    for (int s = 0; s < PIC_MAX_SPECIES; s++) {
      if (keep[s].np == 0) continue;
      Species& sp = I.sp[s];
      if (sp.allocs != keep[s].allocs)
        for (void* p : sp.allocs) (void)hipFree(p);
      sp = keep[s];
      HIPCHK(S, hipMemcpy(sp.ctl, &ctl[s], sizeof ctl[s], hipMemcpyHostToDevice));
    }
    if (I.ndst) (void)hipFree(I.ndst);
    I.g = g0;
    I.ndst = ndst0;
    return PIC_OK;
  }
  S.dirty = true;
  set_current_scale(I);
  char* const at = mem.at;
  for (int s = 0; s < PIC_MAX_SPECIES && st == PIC_OK; s++) {
    Species& sp = I.sp[s];
    if (keep[s].np == 0) continue;
    mem.at = at;
    LoadArgs A = load_args(g, sp.np, 0, mem);
    load_from(A, keep[s].desc, pic_cur(ctl[s]));
    LoadStatus ls;
    st = load_count(S, A, ls);
    if (st == PIC_OK) st = load_place(S, A, sp, 0, ls);
    if (st != PIC_OK) break;
    load_ctl(ctl[s], 0, ls);
    HIPCHK(S, hipMemcpy(sp.ctl, &ctl[s], sizeof ctl[s], hipMemcpyHostToDevice));
  }
  S.ctl_current = false;
  for (Species& k : keep)
    for (void* p : k.allocs) (void)hipFree(p);
  (void)hipFree(ndst0);
  return st;
}

// Settle the tiles of every instance that holds particles (see tile_open).
pic_status settle_tiles(Sim& S) {
  for (Instance& I : S.inst) {
    if (I.settled) continue;
    const int64_t n = instance_particles(I);
    if (n == 0) continue;
    if (tile_open(I) && I.tiled_for != n) {
      GridDesc g;
      pic_status st = setup_grid(S, I.cfg, S.sort_interval, g, (double)n / I.g.ncell);
      if (st == PIC_OK && !same_tiles(g, I.g)) st = retile(S, I, g);
      if (st != PIC_OK) return st;
    }
    I.settled = true;
  }
  return PIC_OK;
}

// Moving window: grid arrays are kept in ring order along x1 (ring column r
// holds window column (r - origin) mod nx1).  to_window copies ncomp
// components from ring to window order in place; to_ring the other way.
void ring_rotate(double* a, size_t ncomp, const GridDesc& g, int origin, bool to_window) {
  if (origin == 0) return;
  const size_t nc = (size_t)g.ncell;
  const int n0 = g.nx[0];
  std::vector<double> row(n0);
  for (size_t c = 0; c < ncomp; c++)
    for (size_t r0 = 0; r0 < nc; r0 += n0) {
      double* v = a + c * nc + r0;
      for (int w = 0; w < n0; w++) {
        const int r = (w + origin) % n0;
        if (to_window)
          row[w] = v[r];
        else
          row[r] = v[w];
      }
      memcpy(v, row.data(), n0 * sizeof(double));
    }
}

pic_status sim_load_fields(Sim& S, int inst, const double* e, const double* b, uint32_t flags) {
  if (inst < 0 || inst >= (int)S.inst.size()) return S.fail(PIC_E_INVALID, "instance out of range");
  if (!e || !b) return S.fail(PIC_E_INVALID, "null field array");
  Instance& I = S.inst[inst];
  size_t n = (size_t)3 * I.g.ncell;
  std::vector<double> he, hb;
  pic_status st;
  if ((st = copy_in(S, he, e, n, flags)) != PIC_OK) return st;
  if ((st = copy_in(S, hb, b, n, flags)) != PIC_OK) return st;
  if (I.cfg.move_window) {
    if ((st = sim_sync(S)) != PIC_OK) return st;
    WinCtl wc;
    if ((st = read_win(S, I, wc)) != PIC_OK) return st;
    ring_rotate(he.data(), 3, I.g, wc.origin, false);
    ring_rotate(hb.data(), 3, I.g, wc.origin, false);
  }
  if (I.g.cyl) {
    // r-z row 0: the axis of E_r and B_theta (zero), the mirror row of
    // E_z, E_theta, B_r (not stored); B_z on the axis is kept
    const size_t nz = (size_t)I.g.nx[0], ncl = (size_t)I.g.ncell;
    for (size_t i = 0; i < nz; i++) {
      for (size_t c = 0; c < 3; c++) he[c * ncl + i] = 0.0;
      hb[ncl + i] = 0.0;
      hb[2 * ncl + i] = 0.0;
    }
  }
  std::vector<float> f(2 * n);
  float em = 0.0f;
  for (size_t i = 0; i < n; i++) {
    if (!std::isfinite(he[i]) || !std::isfinite(hb[i])) return S.fail(PIC_E_RANGE, "non-finite field value");
    f[i] = (float)he[i];
    f[n + i] = (float)hb[i];
    em = std::max(em, std::fabs(f[i]));
  }
  HIPCHK(S, hipStreamSynchronize(S.stream));
  HIPCHK(S, hipMemcpy(I.F[S.steps & 1], f.data(), 2 * n * sizeof(float), hipMemcpyHostToDevice));
  // the running field bound covers the loaded E
  float em0 = 0.0f;
  HIPCHK(S, hipMemcpy(&em0, I.emax, sizeof em0, hipMemcpyDeviceToHost));
  if (em > em0) HIPCHK(S, hipMemcpy(I.emax, &em, sizeof em, hipMemcpyHostToDevice));
  return PIC_OK;
}

// ---------------------------------------------------------------------------
// diagnostics
// ---------------------------------------------------------------------------

// The diagnostics' device scratch: kept between calls and reallocated only
// when a call needs more than any call before it, so repeated diagnostics
// do not allocate.  Every diagnostic synchronizes its stream before it
// returns, so no earlier call still uses the buffer when it is replaced.
pic_status diag_scratch(Sim& S, size_t bytes, char** p) {
  if (bytes > S.diag_cap) {
    if (S.d_diag) (void)hipFree(S.d_diag);
    S.d_diag = nullptr;
    S.diag_cap = 0;
    HIPCHK(S, hipMalloc(&S.d_diag, bytes));
    S.diag_cap = bytes;
  }
  *p = (char*)S.d_diag;
  return PIC_OK;
}

pic_status need(Sim& S, size_t want, size_t out_bytes, size_t* written) {
  if (written) *written = want;
  if (out_bytes < want) return S.fail(PIC_E_RANGE, "output buffer of %zu bytes, %zu needed", out_bytes, want);
  return PIC_OK;
}

// Host threads of an export.  A caller's fresh buffer costs a page fault per
// 4 KiB, more than the copy (9.5 GB/s on one thread against 17 GB/s into pages
// in use), so large exports fill it from several.
constexpr unsigned kExportThreads = 8;

// nplane FP32 grid planes to the caller's FP64 array.  The planes cross in
// FP32, by chunks of rows, and are widened on the host: half the bytes of a
// conversion on the device, and a chunk is widened while others cross.
// origin: ring column of window column 0 (moving window; rows are rotated).
// Six planes of 128x64x64 (25 MB): 4.9 ms before, with the binding's copies.
pic_status export_planes(Sim& S, const GridDesc& g, const float* d, size_t nplane, int origin, double* out) {
  const int n0 = g.nx[0];
  const size_t rows = nplane * (size_t)(g.ncell / n0);
  const size_t per = std::max<size_t>(1, (size_t)(1 << 18) / n0);
  const int chunks = (int)((rows + per - 1) / per);
  std::atomic<int> err{(int)hipSuccess};
  const std::thread::id caller = std::this_thread::get_id();
  parallel_for(chunks, [&](int k) {
    const size_t r0 = (size_t)k * per, nr = std::min(per, rows - r0);
    std::unique_ptr<float[]> mem(new (std::nothrow) float[nr * n0]);
    float* buf = mem.get();
    hipError_t e = buf ? hipSuccess : hipErrorOutOfMemory;
    // (a new thread starts on device 0)
    if (e == hipSuccess && std::this_thread::get_id() != caller) e = hipSetDevice(S.device);
    if (e == hipSuccess)
      e = hipMemcpyAsync(buf, d + r0 * n0, nr * n0 * sizeof(float), hipMemcpyDeviceToHost, S.stream);
    if (e == hipSuccess) e = hipStreamSynchronize(S.stream);
    if (e != hipSuccess) {
      err = (int)e;
      return;
    }
    for (size_t r = 0; r < nr; r++) {
      const float* src = buf + r * n0;
      double* dst = out + (r0 + r) * n0;
      for (int w = 0; w < n0 - origin; w++) dst[w] = src[w + origin];
      for (int w = n0 - origin; w < n0; w++) dst[w] = src[w + origin - n0];
    }
  }, kExportThreads);
  HIPCHK(S, (hipError_t)err.load());
  return PIC_OK;
}

// Device memory to the caller's buffer: the pages of a large one are touched
// from several threads first (the bytes are overwritten by the copy).
pic_status export_copy(Sim& S, void* out, const void* d, size_t bytes) {
  constexpr size_t kPart = (size_t)2 << 20;
  if (bytes >= 2 * kPart)
    parallel_for((int)((bytes + kPart - 1) / kPart), [&](int k) {
      volatile char* p = (volatile char*)out;
      const size_t end = std::min(bytes, (size_t)(k + 1) * kPart);
      for (size_t b = (size_t)k * kPart; b < end; b += 4096) p[b] = 0;
    }, kExportThreads);
  HIPCHK(S, hipMemcpyAsync(out, d, bytes, hipMemcpyDeviceToHost, S.stream));
  HIPCHK(S, hipStreamSynchronize(S.stream));
  return PIC_OK;
}

pic_status compute_rho(Sim& S, int i, double* d_rho) {
  Instance& I = S.inst[i];
  // r-z: the folded ring charge first, then the ring volumes and the ions
  HIPCHK(S, pic_launch_fill64(d_rho, I.g.cyl ? 0.0 : I.cfg.ion_density, (size_t)I.g.ncell, S.stream));
  for (int s = 0; s < PIC_MAX_SPECIES; s++) {
    if (!I.sp[s].used || I.sp[s].np == 0) continue;
    int k = store_desc_index(S, i, s);
    if (k < 0) return S.fail(PIC_E_STATE, "species descriptor missing");
    HIPCHK(S, pic_launch_rho64(S.d_stores + k, I.g, I.sp[s].max_items, (int)(S.steps % S.sort_interval),
                               (int)(S.steps & 1), d_rho, S.stream));
  }
  if (I.g.cyl) HIPCHK(S, pic_launch_rz_rho_finish(d_rho, I.g.nx[0], I.g.nx[1], I.cfg.ion_density, S.stream));
  return PIC_OK;
}

pic_status sim_diag(Sim& S, int i, pic_diag_kind kind, void* out, size_t out_bytes, size_t* written) {
  if (i < 0 || i >= (int)S.inst.size()) return S.fail(PIC_E_INVALID, "instance out of range");
  if (written) *written = 0;
  pic_status st = sim_sync(S);  // first: a moving window changes the particle counts
  if (st != PIC_OK) return st;
  if ((st = refresh_descriptors(S)) != PIC_OK) return st;
  Instance& I = S.inst[i];
  const GridDesc& g = I.g;
  const size_t nc = (size_t)g.ncell;
  const int ii = inst_desc_index(S, i);
  const double V = g.dxd[0] * g.dxd[1] * (g.dim == 3 ? g.dxd[2] : 1.0);
  if (kind != PIC_DIAG_RHO_SNAPSHOT && !out) return S.fail(PIC_E_INVALID, "null output buffer");
  char* scr = nullptr;
  switch (kind) {
    case PIC_DIAG_ENERGY:
    case PIC_DIAG_MOMENTUM: {
      size_t want = (kind == PIC_DIAG_ENERGY ? 4 : 3) * sizeof(double);
      if ((st = need(S, want, out_bytes, written)) != PIC_OK) return st;
      // every sum's kernels first, then one copy and one wait
      double sums[2 + 4 * PIC_MAX_SPECIES] = {}, pm[4] = {0, 0, 0, 0};
      const double* fe = sums;
      int nsp = 0;
      if (kind == PIC_DIAG_ENERGY)
        HIPCHK(S, pic_launch_field_sums(S.d_inst + ii, g.ncell, (int)(S.steps & 1), S.d_scratch, S.d_out, S.stream));
      for (int s = 0; s < PIC_MAX_SPECIES; s++) {
        Species& sp = I.sp[s];
        if (!sp.used || sp.np == 0) continue;
        int k = store_desc_index(S, i, s);
        HIPCHK(S, pic_launch_particle_sums(S.d_stores + k, sp.rqm, g.acc_mode == PIC_ACC_FIXED64, S.d_scratch,
                                           S.d_out + 2 + 4 * nsp, S.stream));
        nsp++;
      }
      HIPCHK(S, hipMemcpyAsync(sums, S.d_out, (size_t)(2 + 4 * nsp) * sizeof(double), hipMemcpyDeviceToHost, S.stream));
      HIPCHK(S, hipStreamSynchronize(S.stream));
      for (int k = 0; k < nsp; k++)
        for (int q = 0; q < 4; q++) pm[q] += sums[2 + 4 * k + q];
      double* o = (double*)out;
      // r-z: the field sums carry the ring volumes in units of dz dr^2, and a
      // particle's charge is w 2 pi dr^2 dz
      const double Vf = g.cyl ? g.dxd[0] * g.dxd[1] * g.dxd[1] : V;
      const double Vp = g.cyl ? 6.283185307179586 * g.dxd[0] * g.dxd[1] * g.dxd[1] : V;
      if (kind == PIC_DIAG_ENERGY) {
        o[0] = 0.5 * Vf * fe[0];
        o[1] = 0.5 * Vf * fe[1];
        o[2] = Vp * pm[0];
        o[3] = o[0] + o[1] + o[2];
      } else {
        o[0] = Vp * pm[1];
        o[1] = Vp * pm[2];
        o[2] = Vp * pm[3];
      }
      return PIC_OK;
    }
    case PIC_DIAG_RHO:
    case PIC_DIAG_GAUSS_RESIDUAL:
    case PIC_DIAG_GAUSS_NORM:
    case PIC_DIAG_CHARGE_RESIDUAL: {
      size_t want = (kind == PIC_DIAG_GAUSS_NORM ? 2 : nc) * sizeof(double);
      if ((st = need(S, want, out_bytes, written)) != PIC_OK) return st;
      if (kind == PIC_DIAG_CHARGE_RESIDUAL && !I.have_snap)
        return S.fail(PIC_E_STATE, "CHARGE_RESIDUAL needs an earlier RHO_SNAPSHOT");
      if ((st = diag_scratch(S, 2 * align256(nc * sizeof(double)), &scr)) != PIC_OK) return st;
      double* rho = (double*)scr;
      double* res = (double*)(scr + align256(nc * sizeof(double)));
      if ((st = compute_rho(S, i, rho)) != PIC_OK) return st;
      double* src = rho;
      if (kind != PIC_DIAG_RHO) {
        if (kind == PIC_DIAG_CHARGE_RESIDUAL)
          HIPCHK(S, pic_launch_charge64(S.d_inst + ii, I.rho_snap, rho, res, g.ncell, g.dim, (int)(S.steps & 1), S.stream));
        else
          HIPCHK(S, pic_launch_gauss64(S.d_inst + ii, rho, res, g.ncell, g.dim, (int)(S.steps & 1), S.stream));
        src = res;
      }
      if (kind == PIC_DIAG_GAUSS_NORM) {
        double ss = 0.0;
        HIPCHK(S, pic_launch_sq_sums(res, g.ncell, S.d_scratch, S.d_out, S.stream));
        HIPCHK(S, hipMemcpyAsync(&ss, S.d_out, sizeof(double), hipMemcpyDeviceToHost, S.stream));
        std::vector<double> h(nc);
        HIPCHK(S, hipMemcpyAsync(h.data(), res, nc * sizeof(double), hipMemcpyDeviceToHost, S.stream));
        HIPCHK(S, hipStreamSynchronize(S.stream));
        double mx = 0.0;
        for (double v : h) mx = std::max(mx, std::fabs(v));
        ((double*)out)[0] = mx;
        ((double*)out)[1] = std::sqrt(ss / (double)nc);
        return PIC_OK;
      }
      if ((st = export_copy(S, out, src, nc * sizeof(double))) != PIC_OK) return st;
      if (I.cfg.move_window) {
        WinCtl wc;
        if ((st = read_win(S, I, wc)) != PIC_OK) return st;
        ring_rotate((double*)out, 1, g, wc.origin, true);
      }
      return PIC_OK;
    }
    case PIC_DIAG_RHO_SNAPSHOT: {
      if (!I.rho_snap) HIPCHK(S, hipMalloc(&I.rho_snap, nc * sizeof(double)));
      if ((st = compute_rho(S, i, I.rho_snap)) != PIC_OK) return st;
      HIPCHK(S, hipStreamSynchronize(S.stream));
      I.have_snap = true;
      return PIC_OK;
    }
    case PIC_DIAG_EXPORT_STATE: {
      int64_t ntot = 0;
      for (Species& sp : I.sp)
        if (sp.used) ntot += sp.np;
      const int stride = g.dim + 4;
      if ((st = need(S, (size_t)ntot * stride * sizeof(double), out_bytes, written)) != PIC_OK) return st;
      double* o = (double*)out;
      for (int s = 0; s < PIC_MAX_SPECIES; s++) {
        Species& sp = I.sp[s];
        if (!sp.used || sp.np == 0) continue;
        int k = store_desc_index(S, i, s);
        const size_t rb = align256((size_t)sp.np * stride * sizeof(double));
        if ((st = diag_scratch(S, rb + align256((size_t)sp.np * sizeof(int)), &scr)) != PIC_OK) return st;
        double* dbuf = (double*)scr;
        if (I.cfg.move_window || g.cyl) {
          // rows in storage order with their ids; sorted by id here, x1 from
          // the ring column to the lab position (moving window), x2 from the
          // cell coordinate to the radius (r-z)
          int* dids = (int*)(scr + rb);
          HIPCHK(S, pic_launch_export_state(S.d_stores + k, (int)sp.np, dbuf, dids, nullptr, nullptr, S.stream));
          std::vector<double> rows((size_t)sp.np * stride);
          std::vector<int> ids(sp.np);
          HIPCHK(S, hipMemcpyAsync(rows.data(), dbuf, rows.size() * sizeof(double), hipMemcpyDeviceToHost, S.stream));
          HIPCHK(S, hipMemcpyAsync(ids.data(), dids, ids.size() * sizeof(int), hipMemcpyDeviceToHost, S.stream));
          HIPCHK(S, hipStreamSynchronize(S.stream));
          WinCtl wc;
          if ((st = read_win(S, I, wc)) != PIC_OK) return st;
          std::vector<int64_t> order;
          order.reserve(sp.np);
          for (int64_t p = 0; p < sp.np; p++)
            if (ids[p] >= 0) order.push_back(p);
          std::sort(order.begin(), order.end(), [&](int64_t a, int64_t b) { return ids[a] < ids[b]; });
          if ((int64_t)order.size() != sp.np) return S.fail(PIC_E_STATE, "removed particles left in the store");
          for (size_t q = 0; q < order.size(); q++) {
            const double* r = rows.data() + (size_t)order[q] * stride;
            double* dst = o + q * stride;
            for (int c = 0; c < stride; c++) dst[c] = r[c];
            if (I.cfg.move_window) {
              const double v = r[0];
              const double cr = std::floor(v);
              int wcol = (int)cr - wc.origin;
              if (wcol < 0) wcol += g.nx[0];
              dst[0] = I.cfg.xmin[0] + ((double)wc.shifts + (double)wcol + (v - cr)) * I.cfg.dx[0];
            } else {
              dst[0] = I.cfg.xmin[0] + r[0] * I.cfg.dx[0];
            }
            for (int d = 1; d < g.dim; d++) dst[d] = I.cfg.xmin[d] + r[d] * I.cfg.dx[d];
            if (g.cyl) dst[1] = (r[1] - 0.5) * I.cfg.dx[1];  // r-z: the radius
          }
        } else {
          // scaled on the device to the caller's positions
          HIPCHK(S, pic_launch_export_state(S.d_stores + k, (int)sp.np, dbuf, nullptr, I.cfg.xmin, I.cfg.dx, S.stream));
          if ((st = export_copy(S, o, dbuf, (size_t)sp.np * stride * sizeof(double))) != PIC_OK) return st;
        }
        o += (size_t)sp.np * stride;
      }
      return PIC_OK;
    }
    case PIC_DIAG_EXPORT_FIELDS:
    case PIC_DIAG_EXPORT_CURRENT: {
      size_t ncomp = kind == PIC_DIAG_EXPORT_FIELDS ? 6 : 3;
      if ((st = need(S, ncomp * nc * sizeof(double), out_bytes, written)) != PIC_OK) return st;
      WinCtl wc;
      if ((st = read_win(S, I, wc)) != PIC_OK) return st;
      const float* src = kind == PIC_DIAG_EXPORT_FIELDS ? I.F[S.steps & 1] : I.Jout;
      if ((st = export_planes(S, g, src, ncomp, wc.origin, (double*)out)) != PIC_OK) return st;
      if (g.cyl) {
        // r-z row 0: mirror images of row 1 for the whole-row components
        // (E_z +, E_theta -, B_r -; J_z +, J_theta -); the half-row
        // components keep their axis values
        double* o = (double*)out;
        const size_t nz = (size_t)g.nx[0];
        const double sgn[6] = {1.0, 0.0, -1.0, 0.0, -1.0, 0.0};
        const bool whole[6] = {true, false, true, false, true, false};
        for (size_t c = 0; c < ncomp; c++)
          if (whole[c])
            for (size_t i = 0; i < nz; i++) o[c * nc + i] = sgn[c] * o[c * nc + nz + i];
      }
      return PIC_OK;
    }
    case PIC_DIAG_KERNEL_TIMES: {
      if ((st = need(S, 6 * sizeof(double), out_bytes, written)) != PIC_OK) return st;
      if ((st = prof_collect(S)) != PIC_OK) return st;
      double* o = (double*)out;
      for (int f = 0; f < 3; f++) {
        o[2 * f] = S.prof_ms[f];
        o[2 * f + 1] = S.prof_n[f];
      }
      return PIC_OK;
    }
    case PIC_DIAG_COUNTS: {
      if ((st = need(S, 4 * sizeof(double), out_bytes, written)) != PIC_OK) return st;
      double* o = (double*)out;
      o[0] = (double)I.steps;
      o[1] = 0;
      o[2] = 0;
      o[3] = 0;
      for (Species& sp : I.sp) {
        if (!sp.used || !sp.ctl) continue;
        const StoreCtl& c = host_ctl(S, sp);
        o[1] += (double)sp.np;
        o[2] = std::max(o[2], (double)c.nsorts);
        o[3] = std::max(o[3], (double)c.nchecks);
      }
      return PIC_OK;
    }
  }
  return S.fail(PIC_E_INVALID, "unknown diagnostic kind %d", (int)kind);
}

// ---------------------------------------------------------------------------
// scratch of the diagnostics that allocate nothing (pic_diag_noalloc)
// ---------------------------------------------------------------------------
// The node charge behind the Gauss and charge residuals lives in this
// file-scope device array: every GPU the library runs on holds its own copy
// until the process ends.  In host code the array's name is a host-side
// stand-in, not a device address; the address is taken once per device with
// hipGetSymbolAddress (at the first pic_create on that device) and used
// everywhere instead of the name.
constexpr size_t kNoAllocCells = size_t(1) << 22;  // doubles: 32 MiB, grids up to 4,194,304 cells
__device__ __align__(256) double scratch[kNoAllocCells];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch[kMaxDevices] = {};

// Record the address of this device's copy of the scratch (the context's
// device is current).
pic_status noalloc_scratch_setup(Sim& S) {
  if (S.device < 0 || S.device >= kMaxDevices) return S.fail(PIC_E_UNSUPPORTED, "device index %d", S.device);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (g_scratch[S.device]) return PIC_OK;
  void* p = nullptr;
  hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess || !p) return S.fail(PIC_E_HIP, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
  g_scratch[S.device] = (double*)p;
  return PIC_OK;
}

// RHO, GAUSS_RESIDUAL or CHARGE_RESIDUAL of instance i into a device buffer
// without allocating: the node charge of the residuals is computed in this
// device's copy of the scratch array, the result goes straight to 'out'.
pic_status sim_diag_noalloc(Sim& S, int i, pic_diag_kind kind, void* out, size_t out_bytes, size_t* written) {
  if (i < 0 || i >= (int)S.inst.size()) return S.fail(PIC_E_INVALID, "instance out of range");
  if (written) *written = 0;
  if (kind != PIC_DIAG_RHO && kind != PIC_DIAG_GAUSS_RESIDUAL && kind != PIC_DIAG_CHARGE_RESIDUAL)
    return S.fail(PIC_E_UNSUPPORTED, "pic_diag_noalloc computes RHO, GAUSS_RESIDUAL and CHARGE_RESIDUAL only");
  if (!out) return S.fail(PIC_E_INVALID, "null output buffer");
  Instance& I = S.inst[i];
  if (I.cfg.move_window)
    return S.fail(PIC_E_UNSUPPORTED, "a moving window keeps its grid in ring order: use pic_diag");
  const size_t nc = (size_t)I.g.ncell;
  pic_status st = need(S, nc * sizeof(double), out_bytes, written);
  if (st != PIC_OK) return st;
  if (kind != PIC_DIAG_RHO && nc > kNoAllocCells)
    return S.fail(PIC_E_RANGE, "grid of %zu cells exceeds the %zu-cell scratch of pic_diag_noalloc", nc,
                  kNoAllocCells);
  if (kind == PIC_DIAG_CHARGE_RESIDUAL && !I.have_snap)
    return S.fail(PIC_E_STATE, "CHARGE_RESIDUAL needs an earlier RHO_SNAPSHOT");
  int cur = 0;
  HIPCHK(S, hipGetDevice(&cur));
  if (cur != S.device) return S.fail(PIC_E_STATE, "device %d is current, the context lives on device %d", cur, S.device);
  // the output must be device memory of this device (a kernel writes it)
  hipPointerAttribute_t pa;
  if (hipPointerGetAttributes(&pa, out) != hipSuccess || pa.type != hipMemoryTypeDevice || pa.device != S.device) {
    (void)hipGetLastError();
    return S.fail(PIC_E_INVALID, "out must be device memory of device %d", S.device);
  }
  double* scr = g_scratch[S.device];
  if (!scr) return S.fail(PIC_E_STATE, "no scratch address for device %d", S.device);
  if ((st = sim_sync(S)) != PIC_OK) return st;
  if (S.dirty)
    return S.fail(PIC_E_STATE, "the launch descriptors are out of date (a load since the last step): run "
                               "pic_step or pic_diag first");
  const int ii = inst_desc_index(S, i);
  double* rho = kind == PIC_DIAG_RHO ? (double*)out : scr;
  if ((st = compute_rho(S, i, rho)) != PIC_OK) return st;  // starts with a fill kernel: no stale contents
  if (kind == PIC_DIAG_GAUSS_RESIDUAL)
    HIPCHK(S, pic_launch_gauss64(S.d_inst + ii, rho, (double*)out, I.g.ncell, I.g.dim, (int)(S.steps & 1), S.stream));
  else if (kind == PIC_DIAG_CHARGE_RESIDUAL)
    HIPCHK(S, pic_launch_charge64(S.d_inst + ii, I.rho_snap, rho, (double*)out, I.g.ncell, I.g.dim, (int)(S.steps & 1),
                                  S.stream));
  HIPCHK(S, hipStreamSynchronize(S.stream));
  return PIC_OK;
}

// Neighbour tile table of the rebin: tile t + delta_s for the 27 slots,
// periodic in tiles.
pic_status build_tables(Sim& S, Instance& I) {
  const GridDesc& g = I.g;
  if (I.ndst) (void)hipFree(I.ndst);
  I.ndst = nullptr;
  if (hipMalloc(&I.ndst, (size_t)g.ntiles * PIC_NSLOT * sizeof(int)) != hipSuccess)
    return S.fail(PIC_E_NOMEM, "tile table allocation failed");
  HIPCHK(S, pic_launch_neighbour_table(g, I.ndst, nullptr));
  HIPCHK(S, hipStreamSynchronize(nullptr));
  return PIC_OK;
}

pic_status sim_create(Sim& S, const pic_config* cfgs, int n, void* stream) {
  if (!cfgs || n < 1) return S.fail(PIC_E_INVALID, "no configuration");
  // everything that can be checked on the host is checked before any HIP call
  int SI = 0;
  bool asked_tiles = false;
  for (int i = 0; i < n; i++) {
    pic_status st = validate(S, cfgs[i]);
    if (st != PIC_OK) return st;
    int64_t nc = 1;
    for (int d = 0; d < cfgs[i].ndim; d++) {
      nc *= cfgs[i].nx[d];
      asked_tiles = asked_tiles || cfgs[i].tile[d] != 0;
    }
    S.total_cells += nc;
  }
  for (int i = 0; i < n; i++) {
    int si = cfgs[i].sort_interval > 0 ? cfgs[i].sort_interval : default_interval(cfgs[i], asked_tiles);
    SI = (i == 0) ? si : std::min(SI, si);
  }
  for (int i = 0; i < n; i++) {
    GridDesc g;
    pic_status st = setup_grid(S, cfgs[i], SI, g);
    if (st != PIC_OK) return st;
  }
  S.sort_interval = SI;
  S.stream = (hipStream_t)stream;
  {
    int dev = 0, ncu = 0;
    HIPCHK(S, hipGetDevice(&dev));
    S.device = dev;
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && ncu > 0)
      S.num_cu = ncu;
    pic_status st = noalloc_scratch_setup(S);
    if (st != PIC_OK) return st;
  }
  if (!S.stream) {
    // graph capture needs a stream of our own when the caller gives none
    HIPCHK(S, hipStreamCreateWithFlags(&S.stream, hipStreamNonBlocking));
    S.own_stream = true;
  }
  const char* env = getenv("PIC_NO_GRAPH");
  S.use_graph = !(env && env[0] == '1');
  S.inst.resize(n);
  S.h_ctl.assign((size_t)n * PIC_MAX_SPECIES, StoreCtl{});
  if (hipMalloc(&S.d_ctl, S.h_ctl.size() * sizeof(StoreCtl)) != hipSuccess)
    return S.fail(PIC_E_NOMEM, "control word allocation failed");
  for (int i = 0; i < n; i++) {
    Instance& I = S.inst[i];
    I.cfg = cfgs[i];
    pic_status st = setup_grid(S, cfgs[i], SI, I.g);
    if (st != PIC_OK) return st;
    size_t nc = (size_t)I.g.ncell;
    for (int k = 0; k < 2; k++) {
      if (hipMalloc(&I.F[k], 6 * nc * sizeof(float)) != hipSuccess)
        return S.fail(PIC_E_NOMEM, "field allocation failed");
      HIPCHK(S, hipMemset(I.F[k], 0, 6 * nc * sizeof(float)));
    }
    if (hipMalloc(&I.Jout, 3 * nc * sizeof(float)) != hipSuccess) return S.fail(PIC_E_NOMEM, "current allocation failed");
    if (hipMalloc(&I.emax, sizeof(float)) != hipSuccess) return S.fail(PIC_E_NOMEM, "field bound allocation failed");
    HIPCHK(S, hipMemset(I.emax, 0, sizeof(float)));
    if (I.cfg.move_window) {
      if (hipMalloc(&I.win, 2 * sizeof(WinCtl)) != hipSuccess) return S.fail(PIC_E_NOMEM, "window state allocation failed");
      HIPCHK(S, hipMemset(I.win, 0, 2 * sizeof(WinCtl)));
    }
    int npass = 0;
    for (int a = 0; a < I.cfg.ndim; a++) npass += I.cfg.smooth_level[a];
    if (npass > 0)
      for (int k = 0; k < 2; k++) {
        if (hipMalloc(&I.Jsm[k], 3 * nc * sizeof(float)) != hipSuccess)
          return S.fail(PIC_E_NOMEM, "smoothing buffer allocation failed");
        HIPCHK(S, hipMemset(I.Jsm[k], 0, 3 * nc * sizeof(float)));
      }
    HIPCHK(S, hipMemset(I.Jout, 0, 3 * nc * sizeof(float)));
    for (int k = 0; k < 2; k++) {
      if (cfgs[i].accumulator == PIC_ACC_FIXED64) {
        if (hipMalloc(&I.J64[k], 3 * nc * sizeof(unsigned long long)) != hipSuccess)
          return S.fail(PIC_E_NOMEM, "current allocation failed");
        HIPCHK(S, hipMemset(I.J64[k], 0, 3 * nc * sizeof(unsigned long long)));
      } else {
        if (hipMalloc(&I.Jacc[k], 3 * nc * sizeof(float)) != hipSuccess)
          return S.fail(PIC_E_NOMEM, "current allocation failed");
        HIPCHK(S, hipMemset(I.Jacc[k], 0, 3 * nc * sizeof(float)));
      }
    }
  }
  HIPCHK(S, hipMalloc(&S.d_scratch, (size_t)2 * 4 * pic_reduce_blocks() * sizeof(double)));
  HIPCHK(S, hipMalloc(&S.d_out, (2 + 4 * PIC_MAX_SPECIES) * sizeof(double)));
  S.dirty = true;
  return PIC_OK;
}

pic_status sim_profile(Sim& S, int enable) {
  if (enable < 0 || enable > 2) return S.fail(PIC_E_INVALID, "profile mode must be 0, 1 or 2");
  pic_status st = prof_collect(S);
  if (st != PIC_OK) return st;
  if (enable == 2)
    for (int f = 0; f < 3; f++) S.prof_ms[f] = S.prof_n[f] = 0.0;
  S.profiling = enable != 0;
  return PIC_OK;
}

void sim_destroy(Sim& S) {
  if (S.stream) (void)hipStreamSynchronize(S.stream);
  for (int f = 0; f < 3; f++)
    for (auto& pr : S.ev_pending[f]) {
      (void)hipEventDestroy(pr.first);
      (void)hipEventDestroy(pr.second);
    }
  for (hipEvent_t e : S.ev_free) (void)hipEventDestroy(e);
  for (int k = 0; k < 2; k++)
    if (S.cycle_exec[k]) (void)hipGraphExecDestroy(S.cycle_exec[k]);
  for (Instance& I : S.inst) {
    for (Species& sp : I.sp) free_species(sp);
    for (int k = 0; k < 2; k++)
      if (I.F[k]) (void)hipFree(I.F[k]);
    for (int k = 0; k < 2; k++) {
      if (I.Jacc[k]) (void)hipFree(I.Jacc[k]);
      if (I.J64[k]) (void)hipFree(I.J64[k]);
    }
    if (I.Jout) (void)hipFree(I.Jout);
    for (int k = 0; k < 2; k++)
      if (I.Jsm[k]) (void)hipFree(I.Jsm[k]);
    if (I.win) (void)hipFree(I.win);
    if (I.emax) (void)hipFree(I.emax);
    if (I.ndst) (void)hipFree(I.ndst);
    if (I.rho_snap) (void)hipFree(I.rho_snap);
  }
  if (S.d_stores) (void)hipFree(S.d_stores);
  if (S.d_inst) (void)hipFree(S.d_inst);
  if (S.d_scratch) (void)hipFree(S.d_scratch);
  if (S.d_out) (void)hipFree(S.d_out);
  if (S.d_diag) (void)hipFree(S.d_diag);
  if (S.d_ctl) (void)hipFree(S.d_ctl);
  if (S.own_stream && S.stream) (void)hipStreamDestroy(S.stream);
}

pic_status sim_info(const Sim& S, int i, pic_info* out) {
  if (!out || i < 0 || i >= (int)S.inst.size()) return PIC_E_INVALID;
  memset(out, 0, sizeof *out);
  const Instance& I = S.inst[i];
  for (int d = 0; d < 3; d++) out->tile[d] = I.g.tile[d];
  out->sort_interval = S.sort_interval;
  out->slack = I.g.slack;
  out->accumulator = I.cfg.accumulator;
  out->lds_bytes = (int64_t)pic_gpd_lds_bytes(I.g);
  for (int s = 0; s < PIC_MAX_SPECIES; s++) {
    if (!I.sp[s].used) continue;
    out->nspecies = s + 1;
    out->nparticles[s] = I.sp[s].np;
    out->rqm[s] = I.sp[s].rqm;
    out->chunk = I.sp[s].desc.chunk;
  }
  if (out->chunk == 0) out->chunk = I.cfg.chunk > 0 ? I.cfg.chunk : 2048;
  return PIC_OK;
}


// ---------------------------------------------------------------------------
// autotuner
// ---------------------------------------------------------------------------

// Launch layout of a whole Sim: a particles-per-tile target (0 = keep the
// tiles in use), the sort interval and the chunk (0 = each store keeps its own:
// the default chunks follow the particles loaded).
struct Layout {
  int ppt = 0, aspect = 2, si = 1, chunk = 2048;
};

// The state an autotune restores before every candidate and at the end.
struct Snapshot {
  std::vector<std::vector<HostParticles>> parts;  // [instance][species]
  std::vector<std::vector<int>> chunk;             // of the stores, likewise (0: not in use)
  std::vector<float*> F, Jout;                     // device copies
  int64_t steps = 0;
  ~Snapshot() {
    for (float* p : F) (void)hipFree(p);
    for (float* p : Jout) (void)hipFree(p);
  }
};

int64_t instance_particles(const Instance& I) {
  int64_t n = 0;
  for (const Species& sp : I.sp)
    if (sp.used) n += sp.np;
  return n;
}

// Tile extents worth trying along an axis of n cells.
std::vector<int> tile_ladder(int n, int need) {
  static const int L[] = {2, 3, 4, 5, 6, 8, 10, 12, 16, 20, 24, 32, 40, 48, 64, 96, 128, 192, 256, 384, 512};
  std::vector<int> v;
  for (int t : L)
    if (t < n && tile_ok(n, t, need)) v.push_back(t);
  v.push_back(n);
  return v;
}

// Tile shape whose volume is closest (in log) to 'cells' and whose x extent
// is closest to 'aspect' times the y extent (x-long tiles give contiguous
// field rows), with an LDS footprint that leaves room for two workgroups per
// CU; g carries the slack of the sort interval in question.
void tile_for_cells(const GridDesc& g0, double cells, int aspect, int out[3]) {
  GridDesc g = g0;
  std::vector<int> lad[3];
  for (int d = 0; d < 3; d++) lad[d] = d < g.dim ? tile_ladder(g.nx[d], g.slk[d] + 2) : std::vector<int>{1};
  double best = 1e300;
  out[0] = g0.tile[0];
  out[1] = g0.tile[1];
  out[2] = g0.tile[2];
  for (int pass = 0; pass < 2 && best == 1e300; pass++) {
    const size_t lim = pass == 0 ? (size_t)kLdsMax / 2 : (size_t)kLdsMax;
    for (int a : lad[0])
      for (int b : lad[1])
        for (int c : lad[2]) {
          g.tile[0] = a;
          g.tile[1] = b;
          g.tile[2] = c;
          if (pic_gpd_lds_bytes(g) > lim) continue;
          double vol = (double)a * b * c;
          double sc = std::fabs(std::log2(vol / cells)) + 0.25 * std::fabs(std::log2((double)a / ((double)aspect * b)));
          if (g.dim == 3) sc += 0.25 * std::fabs(std::log2((double)b / c));
          if (sc < best) {
            best = sc;
            out[0] = a;
            out[1] = b;
            out[2] = c;
          }
        }
  }
}

// Per-instance configurations of a layout (tile extents resolved).
pic_status layout_configs(Sim& S, const Layout& L, std::vector<pic_config>& out) {
  out.resize(S.inst.size());
  for (size_t i = 0; i < S.inst.size(); i++) {
    const Instance& I = S.inst[i];
    pic_config c = I.cfg;
    c.sort_interval = L.si;
    if (L.chunk > 0) c.chunk = L.chunk;
    for (int d = 0; d < 3; d++) c.tile[d] = d < c.ndim ? I.g.tile[d] : 0;
    if (L.ppt > 0) {
      pic_config probe = c;
      for (int d = 0; d < 3; d++) probe.tile[d] = 0;
      GridDesc g;
      pic_status st = setup_grid(S, probe, L.si, g);
      if (st != PIC_OK) return st;
      int64_t n = instance_particles(I);
      double ppc = n > 0 ? (double)n / (double)g.ncell : 1.0;
      int t[3];
      tile_for_cells(g, std::max(1.0, L.ppt / ppc), L.aspect, t);
      for (int d = 0; d < 3; d++) c.tile[d] = d < c.ndim ? t[d] : 0;
    }
    GridDesc g;
    pic_status st = setup_grid(S, c, L.si, g);
    if (st != PIC_OK) return st;
    out[i] = c;
  }
  return PIC_OK;
}

// Install a layout and reload the snapshot into it (host binning of all
// instances and species in parallel, then the uploads).
pic_status apply_layout(Sim& S, const std::vector<pic_config>& cfgs, const Layout& L, const Snapshot& snap) {
  const int si = L.si;
  auto chunk = [&](int i, int s) {
    const int own = snap.chunk[i][s];
    return L.chunk > 0 ? L.chunk : (own > 0 ? own : 2048);  // (2048: a store without particles)
  };
  HIPCHK(S, hipStreamSynchronize(S.stream));
  pic_status st;
  const int ni = (int)S.inst.size();
  std::vector<GridDesc> gs(ni);
  for (int i = 0; i < ni; i++)
    if ((st = setup_grid(S, cfgs[i], si, gs[i])) != PIC_OK) return st;
  std::vector<Binned> bins((size_t)ni * PIC_MAX_SPECIES);
  parallel_for(ni * PIC_MAX_SPECIES, [&](int k) {
    const int i = k / PIC_MAX_SPECIES, s = k % PIC_MAX_SPECIES;
    if (S.inst[i].sp[s].used) bin_particles(gs[i], store_chunk(gs[i], chunk(i, s)), snap.parts[i][s], bins[k]);
  });
  for (int i = 0; i < ni; i++) {
    Instance& I = S.inst[i];
    I.cfg.sort_interval = cfgs[i].sort_interval;
    // (what a store that grows later is made with)
    for (int s = PIC_MAX_SPECIES - 1; s >= 0; s--)
      if (snap.chunk[i][s] > 0 || L.chunk > 0) I.cfg.chunk = chunk(i, s);
    for (int d = 0; d < 3; d++) I.cfg.tile[d] = cfgs[i].tile[d];
    I.g = gs[i];
    if ((st = build_tables(S, I)) != PIC_OK) return st;
    for (int s = 0; s < PIC_MAX_SPECIES; s++) {
      Species& sp = I.sp[s];
      if (!sp.used) continue;
      int64_t cap = std::max<int64_t>(sp.cap, 1);
      if ((st = alloc_species(S, I, sp, cap, chunk(i, s))) != PIC_OK) return st;
      sp.desc.qm = (float)(1.0 / sp.rqm);
    }
    set_current_scale(I);
    for (int s = 0; s < PIC_MAX_SPECIES; s++) {
      Species& sp = I.sp[s];
      if (!sp.used) continue;
      Binned& B = bins[(size_t)i * PIC_MAX_SPECIES + s];
      if ((st = upload_bins(S, sp, B)) != PIC_OK) return st;
      B = Binned();
    }
    const size_t nc = (size_t)I.g.ncell;
    HIPCHK(S, hipMemcpy(I.F[snap.steps & 1], snap.F[i], 6 * nc * sizeof(float), hipMemcpyDeviceToDevice));
    HIPCHK(S, hipMemcpy(I.Jout, snap.Jout[i], 3 * nc * sizeof(float), hipMemcpyDeviceToDevice));
    for (int k = 0; k < 2; k++) {
      if (I.J64[k]) HIPCHK(S, hipMemset(I.J64[k], 0, 3 * nc * sizeof(unsigned long long)));
      if (I.Jacc[k]) HIPCHK(S, hipMemset(I.Jacc[k], 0, 3 * nc * sizeof(float)));
    }
  }
  S.sort_interval = si;
  S.steps = snap.steps;
  for (Instance& I : S.inst) I.steps = snap.steps;
  S.dirty = true;
  return refresh_descriptors(S);
}

// Set or clear the host's rebin-at-every-check request on every store.
pic_status set_force(Sim& S, int v) {
  HIPCHK(S, hipStreamSynchronize(S.stream));
  for (Instance& I : S.inst)
    for (Species& sp : I.sp)
      if (sp.used && sp.ctl) HIPCHK(S, hipMemcpy(&sp.ctl->force, &v, sizeof v, hipMemcpyHostToDevice));
  S.ctl_current = false;
  return PIC_OK;
}

// Milliseconds per step of the installed layout, with a rebin forced at
// every 'every'-th check (besides the checks that find strayed particles):
// two warm-up cycles (graph capture of both parities), then 'trial' steps
// rounded up to whole cycles.
pic_status time_layout(Sim& S, int trial, int every, double* ms) {
  const int SI = S.sort_interval;
  pic_status fs = set_force(S, every);
  if (fs != PIC_OK) return fs;
  int64_t phase = S.steps % SI;
  pic_status st = sim_step(S, (SI - phase) % SI + 2 * SI);
  if (st != PIC_OK) return st;
  const int64_t n = ((int64_t)trial + SI - 1) / SI * SI;
  hipEvent_t a = nullptr, b = nullptr;
  HIPCHK(S, hipEventCreate(&a));
  if (hipEventCreate(&b) != hipSuccess) {
    (void)hipEventDestroy(a);
    return S.fail(PIC_E_HIP, "hipEventCreate failed");
  }
  float t = 0.0f;
  hipError_t e = hipEventRecord(a, S.stream);
  if (e == hipSuccess) {
    st = sim_step(S, n);
    if (st == PIC_OK) {
      e = hipEventRecord(b, S.stream);
      if (e == hipSuccess) e = hipEventSynchronize(b);
      if (e == hipSuccess) e = hipEventElapsedTime(&t, a, b);
    }
  }
  (void)hipEventDestroy(a);
  (void)hipEventDestroy(b);
  if (st != PIC_OK) return st;
  if (e != hipSuccess) return S.fail(PIC_E_HIP, "timing a layout: %s", hipGetErrorString(e));
  if ((st = sim_sync(S)) != PIC_OK) return st;
  if ((st = set_force(S, 0)) != PIC_OK) return st;
  *ms = (double)t / (double)n;
  return PIC_OK;
}

pic_status sim_autotune(Sim& S, pic_tune* io) {
  if (!io) return S.fail(PIC_E_INVALID, "null pic_tune");
  if (io->trial_steps < 1) return S.fail(PIC_E_INVALID, "trial_steps must be >= 1");
  if (io->what < 0 || io->what > 7) return S.fail(PIC_E_INVALID, "unknown PIC_TUNE bits");
  const int what = io->what ? io->what : 7;
  for (const Instance& I : S.inst)
    if (I.cfg.move_window || I.g.cyl)
      return S.fail(PIC_E_UNSUPPORTED, "the autotuner does not handle a moving window or the r-z geometry");
  pic_status st = settle_tiles(S);
  if (st == PIC_OK) st = refresh_descriptors(S);
  if (st != PIC_OK) return st;
  if (S.sgroups.empty()) return S.fail(PIC_E_STATE, "autotune needs loaded particles");
  if ((st = sim_sync(S)) != PIC_OK) return st;
  // Trials rebin at the rate the checks have rebinned since the particles
  // were loaded or the layout last changed (a forced rebin every
  // round(checks / rebins)-th check; none if no check has rebinned), so a
  // layout is timed with the rebin cost it will meet.  Without a history
  // (tuned right after loading) every check is forced: the loaded state may
  // be quieter than the plasma it becomes.
  int every = 1;
  {
    int64_t checks = 0, sorts = 0;
    for (Instance& I : S.inst)
      for (Species& sp : I.sp) {
        if (!sp.used || !sp.ctl) continue;
        StoreCtl c{};
        HIPCHK(S, hipMemcpy(&c, sp.ctl, sizeof c, hipMemcpyDeviceToHost));
        checks += c.nchecks;
        sorts += c.nsorts;
      }
    if (checks > 0) every = sorts == 0 ? 0 : std::max<int>(1, (int)std::lround((double)checks / (double)sorts));
  }
  const bool was_profiling = S.profiling;
  if ((st = prof_collect(S)) != PIC_OK) return st;
  S.profiling = false;
  Snapshot snap;
  snap.steps = S.steps;
  snap.parts.resize(S.inst.size());
  snap.chunk.resize(S.inst.size());
  for (size_t i = 0; i < S.inst.size(); i++) {
    Instance& I = S.inst[i];
    snap.parts[i].resize(PIC_MAX_SPECIES);
    snap.chunk[i].assign(PIC_MAX_SPECIES, 0);
    for (int s = 0; s < PIC_MAX_SPECIES; s++)
      if (I.sp[s].used) {
        if ((st = read_back(S, I.sp[s], I.g.dim, snap.parts[i][s])) != PIC_OK) return st;
        snap.chunk[i][s] = I.sp[s].desc.chunk;
      }
    const size_t nc = (size_t)I.g.ncell;
    float *f = nullptr, *j = nullptr;
    HIPCHK(S, hipMalloc(&f, 6 * nc * sizeof(float)));
    snap.F.push_back(f);
    HIPCHK(S, hipMalloc(&j, 3 * nc * sizeof(float)));
    snap.Jout.push_back(j);
    HIPCHK(S, hipMemcpy(f, I.F[S.steps & 1], 6 * nc * sizeof(float), hipMemcpyDeviceToDevice));
    HIPCHK(S, hipMemcpy(j, I.Jout, 3 * nc * sizeof(float), hipMemcpyDeviceToDevice));
  }
  Layout start;
  start.si = S.sort_interval;
  // one chunk if all stores have the same, else each keeps its own
  int own = 0;  // the first store's
  start.chunk = -1;
  for (const auto& v : snap.chunk)
    for (int c : v)
      if (c > 0) {
        if (own == 0) own = c;
        start.chunk = start.chunk < 0 || start.chunk == c ? c : 0;
      }
  start.chunk = std::max(start.chunk, 0);
  std::vector<pic_config> start_cfgs;
  if ((st = layout_configs(S, start, start_cfgs)) != PIC_OK) return st;
  // every layout tried, by its resolved per-instance tiles, interval and chunk
  std::vector<std::vector<int>> seen;
  auto key = [&](const std::vector<pic_config>& c, int si, int chunk) {
    std::vector<int> k{si, chunk};
    for (const pic_config& x : c) k.insert(k.end(), x.tile, x.tile + 3);
    return k;
  };
  Layout best = start;
  std::vector<pic_config> best_cfgs = start_cfgs;
  double best_ms = 0.0;
  int tried = 0;
  auto trial = [&](const Layout& L, const std::vector<pic_config>& c, double* ms) -> pic_status {
    pic_status r = apply_layout(S, c, L, snap);
    if (r == PIC_OK) r = time_layout(S, io->trial_steps, every, ms);
    tried++;
    return r;
  };
  if ((st = trial(start, start_cfgs, &best_ms)) != PIC_OK) {
    (void)apply_layout(S, start_cfgs, start, snap);
    return st;
  }
  seen.push_back(key(start_cfgs, start.si, start.chunk));
  const double ms_before = best_ms;
  // (out_ms, when given, receives the trial's time; 0 when the layout was
  // not tried: invalid for some instance, or tried before)
  auto consider = [&](const Layout& L, double* out_ms = nullptr) -> pic_status {
    if (out_ms) *out_ms = 0.0;
    std::vector<pic_config> c;
    if (layout_configs(S, L, c) != PIC_OK) return PIC_OK;  // not valid for some instance: skip
    std::vector<int> k = key(c, L.si, L.chunk);
    for (auto& q : seen)
      if (q == k) return PIC_OK;
    seen.push_back(k);
    double ms = 0.0;
    pic_status r = trial(L, c, &ms);
    if (r != PIC_OK) return r;
    if (out_ms) *out_ms = ms;
    // a candidate must beat the best so far by 2% (timing noise of a short
    // trial), which keeps the choice stable from run to run
    if (ms < 0.98 * best_ms) {
      best_ms = ms;
      best = L;
      best_cfgs = c;
    }
    return PIC_OK;
  };
  static const int kPpt[] = {256, 512, 1024, 2048, 4096, 8192};
  static const int kAspect[] = {1, 2, 4, 8};
  static const int kSi[] = {1, 2, 3, 4, 6, 8, 12};
  // chunks above 2048 are left out: a tile whose density grows several-fold
  // later in a run (wakes, beams) would become one long item, a tail no trial
  // on the loaded state can see
  static const int kChunk[] = {512, 1024, 2048};
  std::vector<std::pair<double, Layout>> tiles_tried;  // first round's tile trials by time
  for (int round = 0; round < 2 && st == PIC_OK; round++) {
    if (what & PIC_TUNE_TILE)
      for (int p : kPpt) {
        for (int a : kAspect) {
          Layout L = best;
          L.ppt = p;
          L.aspect = a;
          double ms = 0.0;
          if ((st = consider(L, &ms)) != PIC_OK) break;
          if (round == 0 && ms > 0.0) tiles_tried.push_back({ms, L});
        }
        if (st != PIC_OK) break;
      }
    if (st == PIC_OK && (what & PIC_TUNE_SORT) && round == 0) {
      for (int si : kSi) {
        Layout L = best;
        L.si = si;
        if ((st = consider(L)) != PIC_OK) break;
      }
      // Tile and sort interval interact: a longer cycle needs a wider halo,
      // which a longer tile carries at a smaller share of its work, so the
      // next three fastest tiles of the tile search get an interval search
      // of their own.
      std::sort(tiles_tried.begin(), tiles_tried.end(),
                [](const std::pair<double, Layout>& a, const std::pair<double, Layout>& b) { return a.first < b.first; });
      int extra = 0;
      for (size_t q = 0; q < tiles_tried.size() && extra < 3 && st == PIC_OK; q++) {
        const Layout& T = tiles_tried[q].second;
        if (T.ppt == best.ppt && T.aspect == best.aspect) continue;
        extra++;
        for (int si : kSi) {
          Layout L = T;
          L.si = si;
          L.chunk = best.chunk;
          if ((st = consider(L)) != PIC_OK) break;
        }
      }
    }
    if (st == PIC_OK && (what & PIC_TUNE_CHUNK) && round == 0) {
      const int chunk0 = best.chunk;
      for (int ch : kChunk) {
        Layout L = best;
        L.chunk = ch;
        if ((st = consider(L)) != PIC_OK) break;
      }
      // a new chunk can change the kernel (2D items of more than 1024
      // particles take the one-phase kernel) and with it the best interval
      if (st == PIC_OK && (what & PIC_TUNE_SORT) && best.chunk != chunk0)
        for (int si : kSi) {
          Layout L = best;
          L.si = si;
          if ((st = consider(L)) != PIC_OK) break;
        }
    }
    if (!(what & PIC_TUNE_TILE)) break;
  }
  if (st != PIC_OK) {
    std::string why = S.err;
    (void)apply_layout(S, start_cfgs, start, snap);
    S.profiling = was_profiling;
    S.err = why;
    return st;
  }
  if ((st = apply_layout(S, best_cfgs, best, snap)) != PIC_OK) return st;
  S.profiling = was_profiling;
  io->candidates = tried;
  io->particles_per_tile = best.ppt;
  io->sort_interval = best.si;
  io->chunk = best.chunk > 0 ? best.chunk : own;
  io->ms_before = ms_before;
  io->ms_after = best_ms;
  return PIC_OK;
}

}  // namespace

struct pic_ctx {
  Sim s;
};
struct pic_batch {
  Sim s;
};

extern "C" {

pic_status pic_create(const pic_config* cfg, void* hip_stream, pic_ctx** out) {
  if (!out) return PIC_E_INVALID;
  *out = nullptr;
  pic_ctx* c = new (std::nothrow) pic_ctx();
  if (!c) return PIC_E_NOMEM;
  pic_status st = sim_create(c->s, cfg, 1, hip_stream);
  if (st != PIC_OK) {
    fprintf(stderr, "pic_create: %s\n", c->s.err.c_str());
    sim_destroy(c->s);
    delete c;
    return st;
  }
  *out = c;
  return PIC_OK;
}

pic_status pic_destroy(pic_ctx* ctx) {
  if (!ctx) return PIC_OK;
  (void)hipStreamSynchronize(ctx->s.stream);
  sim_destroy(ctx->s);
  delete ctx;
  return PIC_OK;
}

pic_status pic_load_particles(pic_ctx* ctx, int32_t species, double rqm, int64_t n, const double* x,
                              const double* u, const double* w, uint32_t flags) {
  if (!ctx) return PIC_E_INVALID;
  return sim_load(ctx->s, 0, species, rqm, n, x, u, w, flags);
}

pic_status pic_load_fields(pic_ctx* ctx, const double* e, const double* b, uint32_t flags) {
  if (!ctx) return PIC_E_INVALID;
  return sim_load_fields(ctx->s, 0, e, b, flags);
}

pic_status pic_step(pic_ctx* ctx, int64_t nsteps) {
  if (!ctx) return PIC_E_INVALID;
  return sim_step(ctx->s, nsteps);
}

pic_status pic_sync(pic_ctx* ctx) {
  if (!ctx) return PIC_E_INVALID;
  return sim_sync(ctx->s);
}

pic_status pic_diag(pic_ctx* ctx, pic_diag_kind kind, void* out, size_t out_bytes, size_t* written) {
  if (!ctx) return PIC_E_INVALID;
  return sim_diag(ctx->s, 0, kind, out, out_bytes, written);
}

pic_status pic_diag_noalloc(pic_ctx* ctx, pic_diag_kind kind, void* out, size_t out_bytes, size_t* written) {
  if (!ctx) return PIC_E_INVALID;
  return sim_diag_noalloc(ctx->s, 0, kind, out, out_bytes, written);
}

pic_status pic_get_info(const pic_ctx* ctx, pic_info* out) {
  if (!ctx) return PIC_E_INVALID;
  return sim_info(ctx->s, 0, out);
}

pic_status pic_profile(pic_ctx* ctx, int32_t enable) {
  if (!ctx) return PIC_E_INVALID;
  return sim_profile(ctx->s, enable);
}

pic_status pic_autotune(pic_ctx* ctx, pic_tune* io) {
  if (!ctx) return PIC_E_INVALID;
  return sim_autotune(ctx->s, io);
}

const char* pic_last_error(const pic_ctx* ctx) { return ctx ? ctx->s.err.c_str() : "null context"; }

pic_status pic_batch_create(const pic_config* cfgs, int32_t n, void* hip_stream, pic_batch** out) {
  if (!out) return PIC_E_INVALID;
  *out = nullptr;
  pic_batch* b = new (std::nothrow) pic_batch();
  if (!b) return PIC_E_NOMEM;
  pic_status st = sim_create(b->s, cfgs, n, hip_stream);
  if (st != PIC_OK) {
    fprintf(stderr, "pic_batch_create: %s\n", b->s.err.c_str());
    sim_destroy(b->s);
    delete b;
    return st;
  }
  *out = b;
  return PIC_OK;
}

pic_status pic_batch_destroy(pic_batch* b) {
  if (!b) return PIC_OK;
  (void)hipStreamSynchronize(b->s.stream);
  sim_destroy(b->s);
  delete b;
  return PIC_OK;
}

pic_status pic_batch_load_particles(pic_batch* b, int32_t inst, int32_t species, double rqm, int64_t n,
                                    const double* x, const double* u, const double* w, uint32_t flags) {
  if (!b) return PIC_E_INVALID;
  return sim_load(b->s, inst, species, rqm, n, x, u, w, flags);
}

pic_status pic_batch_load_fields(pic_batch* b, int32_t inst, const double* e, const double* bf, uint32_t flags) {
  if (!b) return PIC_E_INVALID;
  return sim_load_fields(b->s, inst, e, bf, flags);
}

pic_status pic_batch_step(pic_batch* b, int64_t nsteps) {
  if (!b) return PIC_E_INVALID;
  return sim_step(b->s, nsteps);
}

pic_status pic_batch_diag(pic_batch* b, int32_t inst, pic_diag_kind kind, void* out, size_t out_bytes,
                          size_t* written) {
  if (!b) return PIC_E_INVALID;
  return sim_diag(b->s, inst, kind, out, out_bytes, written);
}

pic_status pic_batch_sync(pic_batch* b) {
  if (!b) return PIC_E_INVALID;
  return sim_sync(b->s);
}

pic_status pic_batch_profile(pic_batch* b, int32_t enable) {
  if (!b) return PIC_E_INVALID;
  return sim_profile(b->s, enable);
}

pic_status pic_batch_get_info(const pic_batch* b, int32_t inst, pic_info* out) {
  if (!b) return PIC_E_INVALID;
  return sim_info(b->s, inst, out);
}

pic_status pic_batch_autotune(pic_batch* b, pic_tune* io) {
  if (!b) return PIC_E_INVALID;
  return sim_autotune(b->s, io);
}

const char* pic_batch_last_error(const pic_batch* b) { return b ? b->s.err.c_str() : "null batch"; }

}  // extern "C"
