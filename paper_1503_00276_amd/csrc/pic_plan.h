// pic_plan.h -- planning of a rebin check (see sort.hip): whether a store is
// re-sorted, its tile offsets, its work items and its control words, from the
// destination counts the fused particle kernel added up.  Shared by the field
// step, whose launch plans the stores of at most PIC_PLAN_TILES tiles, and by
// the planner kernels of the others.
#pragma once
#include <hip/hip_runtime.h>
#include "pic_dev.h"

// Tiles one workgroup plans.  A workgroup takes 1,024 tiles per round (one
// memory latency and a scan); 16 rounds stay hidden behind the field step of
// a box with that many tiles.
#define PIC_PLAN_TILES 16384

// Whether the host forces this check to rebin (autotuner trials: every
// force-th check).  nchecks only changes at the end of a check's planning, so
// everything before it takes the same decision.
__device__ __forceinline__ bool forced_check(const StoreCtl* c) {
  const int k = c->force;
  return k > 0 && c->nchecks % k == 0;
}

// Moving window: whether the window moves after the step of parity par.
__device__ __forceinline__ bool win_shift_now(const StoreDesc& S, int par) {
  if (!S.g.window) return false;
  const long long n = S.win[par].step;
  return pic_win_shifts(S.g.wa, n + 1) > pic_win_shifts(S.g.wa, n);
}

// Particles a moving window injects into destination tile d at this check
// (the tile's cells in the new front column, which is the ring column of the
// old origin, times the particles per cell); shift: the window moves.
__device__ __forceinline__ int win_inject_count(const StoreDesc& S, int d, int par, bool shift) {
  if (!shift) return 0;
  const GridDesc& g = S.g;
  int tc[3];
  pic_tile_coords(g, d, tc);
  const int o = S.win[par].origin;
  const int org0 = tc[0] * g.tile[0];
  if (o < org0 || o >= org0 + min(g.tile[0], g.nx[0] - org0)) return 0;
  int cells = 1;
  for (int k = 1; k < g.dim; k++) cells *= min(g.tile[k], g.nx[k] - tc[k] * g.tile[k]);
  int n = cells * S.inj_ppc[0] * S.inj_ppc[1] * S.inj_ppc[2];
  // r-z: the lattice points of the axis row below the axis are not injected
  if (g.cyl && tc[1] == 0) n -= S.inj_ppc[0] * (S.inj_ppc[1] / 2);
  return n;
}

// Exclusive scan of two ints over a block of NT threads; returns the totals.
template <int NT>
__device__ __forceinline__ void block_scan2(int a, int b, int& ea, int& eb, int& ta, int& tb) {
  __shared__ int wa[NT / 64], wb[NT / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int ia = a, ib = b;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    int va = __shfl_up(ia, off);
    int vb = __shfl_up(ib, off);
    if (lane >= off) {
      ia += va;
      ib += vb;
    }
  }
  if (lane == 63) {
    wa[wave] = ia;
    wb[wave] = ib;
  }
  __syncthreads();
  int ca = 0, cb = 0;
  ta = 0;
  tb = 0;
#pragma unroll
  for (int w = 0; w < NT / 64; w++) {
    if (w < wave) {
      ca += wa[w];
      cb += wb[w];
    }
    ta += wa[w];
    tb += wb[w];
  }
  ea = ca + ia - a;
  eb = cb + ib - b;
  __syncthreads();
}

// Offsets and work items of tile t, whose c particles start at ra and whose
// items start at rb, into buffer set nxt.  (A moving window whose plasma outgrows
// the store is reported by plan_commit; until the host sees that, the items end
// with the arrays, as what the scatter writes does.)
__device__ __forceinline__ void plan_tile(const StoreDesc& S, int nxt, int t, int c, int ra, int rb) {
  S.toff[nxt][t] = ra;
  S.ioff[nxt][t] = rb;
  const int size = pic_item_size(c, S.chunk);
  int4* items = (int4*)S.items[nxt];
  for (int b = 0, k = rb; b < c && k < S.max_items; b += size, k++)
    items[k] = make_int4(t, min(ra + b, S.cap), min(ra + min(b + size, c), S.cap), 0);
}

// End of a check: totals of the planned set (act) and the control words.  One
// thread, the only writer of the control words during a check, after
// everything that reads them.
__device__ __forceinline__ void plan_commit(const StoreDesc& S, int cur, bool act, int particles, int items) {
  StoreCtl* c = S.ctl;
  if (act) {
    const int nxt = 1 - cur;
    S.toff[nxt][S.g.ntiles] = particles;
    S.ioff[nxt][S.g.ntiles] = items;
    c->n_items[nxt] = min(items, S.max_items);
    c->np = particles;
    // in a periodic box the count is fixed; a moving window (removal,
    // injection) or the r-z wall (removal) change it within the capacity
    if (items > S.max_items || ((S.g.window || S.g.cyl) ? particles > S.cap : particles != S.np)) c->bad |= 4;
  }
  c->cur = cur;
  c->pending = act ? 1 : 0;  // the scatter of this check fills set 1 - cur
  c->active = act ? 1 : 0;
  c->flag = 0;
  c->nchecks += 1;
  c->nsorts += act ? 1 : 0;
  // after this check every particle sits in its own tile (re-sorted), or
  // within flag_slack cells of it (no particle strayed further)
  c->sorted = act ? 1 : 0;
}

// The whole check of one store by one workgroup of NT threads.
template <int NT>
__device__ __forceinline__ void plan_store(const StoreDesc& S, int par) {
  constexpr int PT = 4;  // consecutive tiles per thread and round
  const bool shift = win_shift_now(S, par);
  const bool act = S.ctl->flag || forced_check(S.ctl) || shift;
  const int cur = pic_cur(*S.ctl), nxt = 1 - cur;
  __syncthreads();  // every thread has read the control words
  int na = 0, ni = 0;
  if (act) {
    const int nt = S.g.ntiles;
    int v[PT], vn[PT];
    auto load = [&](int base, int (&o)[PT]) {
#pragma unroll
      for (int k = 0; k < PT; k++) {
        const int t = base + PT * (int)threadIdx.x + k;
        o[k] = t < nt ? S.dcount[t] : 0;
      }
    };
    load(0, v);
    for (int base = 0; base < nt; base += NT * PT) {
      load(base + NT * PT, vn);  // the next round's, in flight meanwhile
      int a = 0, b = 0;
#pragma unroll
      for (int k = 0; k < PT; k++) {
        const int t = base + PT * (int)threadIdx.x + k;
        if (t < nt) v[k] += win_inject_count(S, t, par, shift);  // injected ones follow the incoming
        a += v[k];
        b += pic_item_count(v[k], S.chunk);
      }
      int ea, eb, ta, tb;
      block_scan2<NT>(a, b, ea, eb, ta, tb);
      int ra = na + ea, rb = ni + eb;
#pragma unroll
      for (int k = 0; k < PT; k++) {
        const int t = base + PT * (int)threadIdx.x + k;
        if (t >= nt) break;
        plan_tile(S, nxt, t, v[k], ra, rb);
        ra += v[k];
        rb += pic_item_count(v[k], S.chunk);
      }
#pragma unroll
      for (int k = 0; k < PT; k++) v[k] = vn[k];
      na += ta;
      ni += tb;
    }
  }
  if (threadIdx.x == 0) plan_commit(S, cur, act, na, ni);
}
