// pic_kernels.h -- host-side launchers of the HIP kernels (one translation
// unit per kernel family; the runtime calls only these).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include "pic_dev.h"

// fused gather + push + deposit (gpd.hip)
size_t pic_gpd_lds_bytes(const GridDesc& g);
// LDS of step kstep of a sort cycle (at most pic_gpd_lds_bytes)
size_t pic_gpd_lds_bytes_step(const GridDesc& g, int kstep);
int pic_gpd_block();
// particles a work item of the two-phase 3D variant can hold (its chunk limit)
int pic_gpd_split_chunk();
// the two-phase periodic 2D kernel (mode 7): whether a grid takes it, and the
// particles one of its work items can hold
bool pic_gpd_two_phase2(const GridDesc& g);
int pic_gpd_two_phase2_chunk();
// padded LDS strides of the two-phase variant for g's tile and stray bound
void pic_gpd_split_strides(GridDesc& g);
int pic_gpd_max_group();
// allow the LDS size a group needs (call before launching or capturing);
// mode: the boundary logic of the group's stores (0 periodic, 1 moving window
// along x1, 2 the 2D r-z geometry, 3 r-z with a moving window, 4 periodic 3D
// in two phases, 5 the same with the compile-time LDS strides of 4x4xN
// tiles), which selects the kernel variant
hipError_t pic_gpd_prepare(int dim, int order, int mode, size_t lds);
// workgroups of the variant that are resident on one CU at once with 'lds'
// bytes of dynamic LDS (after pic_gpd_prepare)
int pic_gpd_resident(int dim, int order, int mode, size_t lds);
// kstep: steps done since the last rebin check (bounds the staged halo);
// count: the step's rebin check follows (the particles are counted by
// destination tile);
// ev0 / ev1 (may be null): events stamped at the kernel's start / end
hipError_t pic_launch_gpd(int dim, int order, int mode, const StoreDesc* d_stores, int nstores, int grid,
                          size_t lds, int parity, int kstep, bool count, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1);

// Yee field solve (field.hip); instances in d_inst[0..ninst)
int pic_yee_tiles(int dim, const int nx[3], bool window);
// whether a periodic 3D box takes the field step that marches along z
bool pic_yee_marches(const int nx[3]);
// current smoothing: Cartesian instances whose passes fit LDS tiles take them
// all in one launch (max_level: most passes of such an instance per axis); the
// others (r-z, many passes in 3D) one launch per pass and axis
bool pic_smooth_in_tiles(int dim, const int level[3]);
int pic_smooth_tiles(int dim, const int nx[3]);
hipError_t pic_launch_smooth_tiles(const InstDesc* d_inst, int ninst, int dim, int max_tiles, const int max_level[3],
                                   int parity, hipStream_t st);
hipError_t pic_launch_smooth_pass(const InstDesc* d_inst, int ninst, int max_ncell, int axis, int lev,
                                  int parity, hipStream_t st);
// cart / cyl: the group holds Cartesian / r-z instances (each kernel skips the
// others); window: some instance has a moving window (selects the variant
// with the window terms); march / tiles: without a window, the group holds 3D
// boxes that march along z / that take the 3D tiles.  The launch also advances
// the moving windows and, with nplan > 0, plans the rebin check of the nplan
// stores at d_plan (those of at most pic_plan_tiles() tiles).
hipError_t pic_launch_yee_step(const InstDesc* d_inst, int ninst, int max_tiles, int dim, bool cart, bool cyl,
                               bool window, bool march, bool tiles, int parity, const StoreDesc* d_plan, int nplan,
                               hipStream_t st);

// tile rebin (sort.hip); stores in d_stores[0..nstores), after the field step
// of the same parity, which planned the stores of at most pic_plan_tiles()
// tiles; big: some store has more; inject_max: most particles a store injects
// per window shift, thermal: some of them with thermal momenta
int pic_plan_tiles();
hipError_t pic_launch_rebin(const StoreDesc* d_stores, int nstores, int max_items, int total_tiles,
                            int total_blocks, bool big, int inject_max, bool thermal, int parity,
                            hipStream_t st);

// loading (load.hip): the new particles (FP64 rows in device memory) and the
// ones already stored, sorted together into a buffer set of the store
struct LoadStatus {
  unsigned flags;            // non-finite: 1 positions, 2 momenta, 4 weights
  unsigned long long first;  // 2 * the first new particle outside the window or (+ 1) beyond the wall
  unsigned long long u2, w;  // bits of max |u|^2 of all and of max |w| of the new particles
  int idmax;                 // largest id stored (-1: none)
  int items;                 // work items planned
};
struct LoadArgs {
  GridDesc g;
  double xmin[3];
  int shifts, origin;        // moving window
  long long old, n, id0;     // particles stored, particles new, id of the first new one
  const double *x, *u, *w;
  const int *ocell, *oid;    // the stored ones
  const float *oeps[3], *ou[3], *ow;
  int* cells;                // [ntiles * tile volume] zeroed
  int* tiles;                // [ntiles]
  int *rank, *slot;          // [old + n]
  LoadStatus* status;        // zeroed but first = ~0 and idmax = -1
};
// Index of a cell in tile order: its tile times the tile's volume plus its place
// in the tile, x fastest.  (Ragged tiles count in full: a box of nearly 2^31
// cells can have more than 2^31 of these.)
__host__ __device__ inline long long pic_load_key(const GridDesc& g, const int c[3]) {
  int t[3] = {0, 0, 0}, l[3] = {0, 0, 0};
  for (int d = 0; d < g.dim; d++) {
    t[d] = c[d] / g.tile[d];
    l[d] = c[d] - t[d] * g.tile[d];
  }
  return (long long)pic_tile_index(g, t[0], t[1], t[2]) * (g.tile[0] * g.tile[1] * g.tile[2]) + l[0] +
         g.tile[0] * (l[1] + g.tile[1] * l[2]);
}
hipError_t pic_launch_load_count(const LoadArgs& a, hipStream_t st);
hipError_t pic_launch_load_place(const LoadArgs& a, const StoreDesc& s, int set, hipStream_t st);
hipError_t pic_launch_neighbour_table(const GridDesc& g, int* ndst, hipStream_t st);

// diagnostics (diag.hip)
// adds a species' charge density; kstep: steps done since the last rebin
// check, par: parity of the steps done
hipError_t pic_launch_rho64(const StoreDesc* d_store, const GridDesc& g, int max_items, int kstep, int par, double* rho,
                            hipStream_t st);
hipError_t pic_launch_fill64(double* p, double v, size_t n, hipStream_t st);
// r-z: rho = ion + folded charge / (r_j/dr) on rows j >= 1, row 0 = row 1
hipError_t pic_launch_rz_rho_finish(double* rho, int nz, int nr, double ion, hipStream_t st);
hipError_t pic_launch_gauss64(const InstDesc* d_inst, const double* rho, double* G, int ncell, int dim,
                              int fpar, hipStream_t st);
hipError_t pic_launch_charge64(const InstDesc* d_inst, const double* rho0, const double* rho1,
                               double* C, int ncell, int dim, int par, hipStream_t st);
// compensated FP64 sums: out[0..nout) with partial scratch (>= 2*nout*pic_reduce_blocks() doubles)
int pic_reduce_blocks();
hipError_t pic_launch_field_sums(const InstDesc* d_inst, int ncell, int fpar, double* scratch, double* out,
                                 hipStream_t st);
// exact: independent of the particles' storage order
hipError_t pic_launch_particle_sums(const StoreDesc* d_store, double rqm, bool exact, double* scratch, double* out,
                                    hipStream_t st);
hipError_t pic_launch_sq_sums(const double* v, int n, double* scratch, double* out, hipStream_t st);
// xmin, dx (3 each): positions scaled to the caller's (null with ids: cell units)
hipError_t pic_launch_export_state(const StoreDesc* d_store, int np, double* out, int* ids, const double* xmin,
                                   const double* dx, hipStream_t st);
