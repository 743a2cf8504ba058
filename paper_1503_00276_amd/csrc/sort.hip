// sort.hip -- periodic tile rebin of the particle storage (counting sort by
// tile).  Not part of the dissertation's CPU code, which keeps particles in
// plain arrays; here it keeps every tile's particles contiguous so the fused
// kernel can stage the tile's fields in LDS.
//
// Between rebins a particle strays at most 'slack' cells outside its tile,
// so at a rebin every particle moves to its own tile or to one of the 3^d - 1
// neighbours.  The rebin is a counting sort over those 27 neighbour slots.
// The fused particle kernel of a cycle's last step counts its items' particles
// by slot and adds the counts to the destination tiles' totals; the totals it
// finds there are the items' places in the tiles (moves_add in gpd.hip).
// What is left of a check:
//   plan    (per store)             scan of the totals: tile offsets, work
//                                   items, control words (pic_plan.h)
//   scatter (per source item)       scatter into the other buffer set; the
//                                   plasma of a moving window's new column
// The plan of a store of at most PIC_PLAN_TILES tiles runs in the field
// step's launch, beside it; larger ones take three launches here (block sums,
// their scan, offsets).  Only stores whose fused kernel raised the flag, or
// whose check the host forces (autotuner trials), or whose window moves, do
// any work.  With separate launches for the slot prefixes, the destination
// totals, the scan, the offsets and the injection, a check cost five or six
// launches of 4-5 us, whatever it found to do: 18 us of 420 us a step in a 3D
// box of 4.3 M particles, 30 us of 163 us in a 2D moving window.
#include "pic_dev.h"
#include "pic_kernels.h"
#include "pic_plan.h"

namespace {

constexpr int kBlock = 256;
constexpr int kScanBlock = 1024;
constexpr int kMaxGroup = 256;
constexpr int kTB = PIC_REBIN_TILES;

static_assert(kTB == kBlock, "one destination tile per thread of the planner");

// Store of a flat index over the stores of a group, given per-store starts
// (pref[0..n-1], increasing) in LDS.
__device__ __forceinline__ int store_of(const int* pref, int n, int x) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (pref[mid] <= x) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// Slot of a particle with packed cell 'cell' that is stored in tile t
// (-1 for a particle a moving window removed).
__device__ __forceinline__ int particle_slot(const GridDesc& g, int t, int cell) {
  if (cell < 0) return -1;
  int tc[3], c[3];
  pic_tile_coords(g, t, tc);
  pic_unpack(g, cell, c);
  int dd[3] = {0, 0, 0};
  for (int d = 0; d < g.dim; d++) {
    int o = tc[d] * g.tile[d];
    int e = min(g.tile[d], g.nx[d] - o);
    int l = pic_local(c[d], o, e, g.nx[d]);
    dd[d] = l < 0 ? -1 : (l >= e ? 1 : 0);
  }
  return pic_slot(dd[0], dd[1], dd[2]);
}

// Stores the field step's launch does not plan.
__device__ __forceinline__ bool plan_here(const StoreDesc& S) { return S.g.ntiles > PIC_PLAN_TILES; }

// --- large stores, 1. per block of tiles: particles and items ----------------
__global__ void __launch_bounds__(kBlock) rebin_sums(const StoreDesc* __restrict__ stores, int nstores, int par) {
  __shared__ int b0[kMaxGroup];
  for (int i = threadIdx.x; i < nstores; i += blockDim.x) b0[i] = stores[i].blk0;
  __syncthreads();
  const StoreDesc& S = stores[store_of(b0, nstores, blockIdx.x)];
  const bool shift = win_shift_now(S, par);
  if (!plan_here(S) || !(S.ctl->flag || forced_check(S.ctl) || shift)) return;
  const int blk = blockIdx.x - S.blk0;
  const int d = blk * kTB + threadIdx.x;
  int acc = 0;
  if (d < S.g.ntiles) acc = S.dcount[d] + win_inject_count(S, d, par, shift);
  int ea, eb, ta, tb;
  block_scan2<kBlock>(acc, pic_item_count(acc, S.chunk), ea, eb, ta, tb);
  if (threadIdx.x == 0) {
    S.bsum[2 * blk] = ta;
    S.bsum[2 * blk + 1] = tb;
  }
}

// --- 2. per store: scan of the block sums, totals, control words -------------
__global__ void __launch_bounds__(kScanBlock) rebin_fold(const StoreDesc* __restrict__ stores, int par) {
  const StoreDesc& S = stores[blockIdx.x];
  if (!plan_here(S)) return;
  const bool act = S.ctl->flag || forced_check(S.ctl) || win_shift_now(S, par);
  const int cur = pic_cur(*S.ctl);
  __syncthreads();  // every thread has read the control words
  int na = 0, ni = 0;
  if (act) {
    const int nblk = (S.g.ntiles + kTB - 1) / kTB;
    for (int base = 0; base < nblk; base += kScanBlock) {
      const int k = base + threadIdx.x;
      const int a = k < nblk ? S.bsum[2 * k] : 0;
      const int b = k < nblk ? S.bsum[2 * k + 1] : 0;
      int ea, eb, ta, tb;
      block_scan2<kScanBlock>(a, b, ea, eb, ta, tb);
      if (k < nblk) {
        S.bpre[2 * k] = na + ea;
        S.bpre[2 * k + 1] = ni + eb;
      }
      na += ta;
      ni += tb;
    }
  }
  if (threadIdx.x == 0) plan_commit(S, cur, act, na, ni);
}

// --- 3. per tile: offsets and work items -------------------------------------
__global__ void __launch_bounds__(kBlock) rebin_offsets(const StoreDesc* __restrict__ stores, int nstores, int par) {
  __shared__ int b0[kMaxGroup];
  for (int i = threadIdx.x; i < nstores; i += blockDim.x) b0[i] = stores[i].blk0;
  __syncthreads();
  const StoreDesc& S = stores[store_of(b0, nstores, blockIdx.x)];
  if (!plan_here(S) || !S.ctl->active) return;
  const int nxt = 1 - S.ctl->cur;
  const int blk = blockIdx.x - S.blk0;
  const int t = blk * kTB + threadIdx.x;
  const int c = t < S.g.ntiles ? S.dcount[t] + win_inject_count(S, t, par, win_shift_now(S, par)) : 0;
  int ea, eb, ta, tb;
  block_scan2<kBlock>(c, pic_item_count(c, S.chunk), ea, eb, ta, tb);
  if (t < S.g.ntiles) plan_tile(S, nxt, t, c, S.bpre[2 * blk] + ea, S.bpre[2 * blk + 1] + eb);
}

// Block-shared prefix over stores of a per-store count (0 for idle stores).
template <typename F>
__device__ void group_prefix(const StoreDesc* stores, int nstores, int* pref, F count) {
  // a store per lane: one thread walking the control words would wait for them
  // once per store
  if (threadIdx.x < 64) {
    int acc = 0;
    for (int base = 0; base < nstores; base += 64) {
      const int s = base + (int)threadIdx.x;
      int sum = s < nstores && stores[s].ctl->active ? count(stores[s]) : 0;
      for (int off = 1; off < 64 && off < nstores; off <<= 1) {
        const int v = __shfl_up(sum, off);
        if ((int)threadIdx.x >= off) sum += v;
      }
      if (s < nstores) pref[s + 1] = acc + sum;
      acc += __shfl(sum, 63);
    }
    if (threadIdx.x == 0) pref[0] = 0;
  }
  __syncthreads();
}

// --- per old item: scatter into the other buffer set --------------------------
// (stable within an item and slot; the destination counts are cleared for the
// next check, and a moving window's new column is filled).  INJECT: 0 no store
// has a moving window, 1 the injected plasma is cold, 2 thermal in some store:
// the FP64 deviates of the latter take the kernel from 58 to 99 registers,
// half the wavefronts, so they are compiled in only where they are needed.
template <bool THERMAL>
__device__ void inject_column(const StoreDesc& S, int par);

template <int INJECT>
__global__ void __launch_bounds__(kBlock) rebin_scatter(const StoreDesc* __restrict__ stores, int nstores,
                                                        int total_tiles, int par) {
  __shared__ int pref[kMaxGroup + 1];
  __shared__ int run[PIC_NSLOT];
  __shared__ int wcnt[kBlock / 64][PIC_NSLOT];
  // the source set is cur (the fold set pending for the destination)
  if ((int)(blockIdx.x * blockDim.x) < total_tiles) {
    for (int i = threadIdx.x; i < nstores; i += blockDim.x) pref[i] = stores[i].tile0;
    __syncthreads();
    for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < total_tiles; q += gridDim.x * blockDim.x) {
      const StoreDesc& S = stores[store_of(pref, nstores, q)];
      S.dcount[q - S.tile0] = 0;
    }
    __syncthreads();
  }
  group_prefix(stores, nstores, pref, [](const StoreDesc& S) { return S.ctl->n_items[S.ctl->cur]; });
  if constexpr (INJECT > 0)
    for (int k = 0; k < nstores; k++) inject_column<INJECT == 2>(stores[k], par);
  const int total = pref[nstores];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const unsigned long long lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  int s = (int)blockIdx.x < total ? store_of(pref, nstores, blockIdx.x) : 0;
  for (int gi = blockIdx.x; gi < total; gi += gridDim.x) {
    while (gi >= pref[s + 1]) s++;
    const StoreDesc& S = stores[s];
    const GridDesc& g = S.g;
    const int cur = S.ctl->cur, nxt = 1 - cur;
    const int ii = gi - pref[s];
    const Item it = S.items[cur][ii];
    if (threadIdx.x < PIC_NSLOT) {
      int sl = threadIdx.x;
      int d = S.ndst[it.tile * PIC_NSLOT + sl];
      run[sl] = S.toff[nxt][d] + S.pre[ii * PIC_NSLOT + sl];  // (unused where the item has no particle)
    }
    for (int base = it.begin; base < it.end; base += blockDim.x) {
      __syncthreads();
      if (threadIdx.x < (kBlock / 64) * PIC_NSLOT) (&wcnt[0][0])[threadIdx.x] = 0;
      __syncthreads();
      int p = base + threadIdx.x;
      // every load of the particle is issued here, before the rank
      // computation, so the round waits for one memory latency, not two
      const bool have = p < it.end;
      int cell = 0, pid = 0;
      float ev[3] = {0.0f, 0.0f, 0.0f}, uv[3] = {0.0f, 0.0f, 0.0f}, wv = 0.0f;
      if (have) {
        cell = S.cell[cur][p];
        for (int d = 0; d < g.dim; d++) ev[d] = S.eps[cur][d][p];
        uv[0] = S.u[cur][0][p];
        uv[1] = S.u[cur][1][p];
        uv[2] = S.u[cur][2][p];
        wv = S.w[cur][p];
        pid = S.id[cur][p];
      }
      int sl = have ? particle_slot(g, it.tile, cell) : -1;
      int rank = 0;
      unsigned long long todo = __ballot(sl >= 0);
      while (todo) {
        int leader = __ffsll((long long)todo) - 1;
        int ls = __shfl(sl, leader);
        unsigned long long m = __ballot(sl == ls);
        if (sl == ls) rank = (int)__popcll(m & lt);
        if (lane == leader) wcnt[wave][ls] = (int)__popcll(m);
        todo &= ~m;
      }
      __syncthreads();
      int pos = -1;
      if (sl >= 0) {
        pos = run[sl] + rank;
        for (int w = 0; w < wave; w++) pos += wcnt[w][sl];
        if (pos < 0 || pos >= S.cap) {  // inconsistent counts: never write out of bounds
          atomicOr(&S.ctl->bad, 2);
          pos = -1;
        }
      }
      if (pos >= 0) {
        S.cell[nxt][pos] = cell;
        for (int d = 0; d < g.dim; d++) S.eps[nxt][d][pos] = ev[d];
        S.u[nxt][0][pos] = uv[0];
        S.u[nxt][1][pos] = uv[1];
        S.u[nxt][2][pos] = uv[2];
        S.w[nxt][pos] = wv;
        S.id[nxt][pos] = pid;
      }
      __syncthreads();
      if (threadIdx.x < PIC_NSLOT) {
        int add = 0;
        for (int w = 0; w < kBlock / 64; w++) add += wcnt[w][threadIdx.x];
        run[threadIdx.x] += add;
      }
    }
    __syncthreads();
  }
}

// --- moving window: the plasma of the new front column ------------------------
// Particle k of the column (cells in increasing linear index, lattice points
// of a cell with axis 1 fastest) goes to its tile's range after the incoming
// particles, at its rank among the tile's injected particles; ids continue
// from the window's counter.
// Output n >= 1 of the SplitMix64 generator seeded with s (Steele, Lea and
// Flood, "Fast splittable pseudorandom number generators", 2014): the state
// advances by the golden-ratio increment, the output mixes it.
__device__ unsigned long long splitmix64_output(unsigned long long s, unsigned long long n) {
  unsigned long long z = s + n * 0x9e3779b97f4a7c15ull;
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  return z ^ (z >> 31);
}

// Standard normal deviate of component c of the particle with id 'id':
// Box-Muller (1958) on U1 in (0, 1] and U2 in [0, 1), 53 bits each.
__device__ double thermal_normal(unsigned long long seed, long long id, int c) {
  const unsigned long long n = 8ull * (unsigned long long)id + 2ull * (unsigned long long)c;
  const double u1 = (double)((splitmix64_output(seed, n + 1) >> 11) + 1) * 0x1.0p-53;
  const double u2 = (double)(splitmix64_output(seed, n + 2) >> 11) * 0x1.0p-53;
  return sqrt(-2.0 * log(u1)) * cos(6.283185307179586 * u2);
}

template <bool THERMAL>
__device__ void inject_column(const StoreDesc& S, int par) {
  if (!S.g.window || !S.ctl->active || S.inj_ppc[0] == 0 || !win_shift_now(S, par)) return;
  const GridDesc& g = S.g;
  const int nxt = 1 - S.ctl->cur;
  const int p0 = S.inj_ppc[0], p1 = S.inj_ppc[1], p2 = g.dim == 3 ? S.inj_ppc[2] : 1;
  const int ppc = p0 * p1 * p2;
  const int ny = g.nx[1], nz = g.dim == 3 ? g.nx[2] : 1;
  const int total = ppc * ny * nz;
  const int o = S.win[par].origin;
  const long long id0 = S.win[par].next_id;
  // r-z: lattice points below the axis (axis-row offsets under 1/2) are
  // skipped; the others of the tile holding the axis row move up in rank
  const int nex = g.cyl ? p1 / 2 : 0;
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < total; k += gridDim.x * blockDim.x) {
    const int cidx = k / ppc, li = k - cidx * ppc;
    const int cy = cidx % ny, cz = cidx / ny;
    const int l0 = li % p0, l1 = (li / p0) % p1, l2 = li / (p0 * p1);
    if (cy == 0 && l1 < nex) continue;
    const int ty = cy / g.tile[1], tz = g.dim == 3 ? cz / g.tile[2] : 0;
    const int t = pic_tile_index(g, o / g.tile[0], ty, tz);
    const int oy = ty * g.tile[1], oz = tz * g.tile[2];
    const int ey = min(g.tile[1], ny - oy);
    const int rank = ((cy - oy) + ey * (cz - oz)) * ppc + li - (oy == 0 ? p0 * nex : 0);
    const int pos = S.toff[nxt][t + 1] - win_inject_count(S, t, par, true) + rank;
    if (pos < 0 || pos >= S.cap) {
      atomicOr(&S.ctl->bad, 2);
      continue;
    }
    S.cell[nxt][pos] = pic_pack(g, o, cy, cz);
    S.eps[nxt][0][pos] = ((float)l0 + 0.5f) / (float)p0;
    S.eps[nxt][1][pos] = ((float)l1 + 0.5f) / (float)p1;
    if (g.dim == 3) S.eps[nxt][2][pos] = ((float)l2 + 0.5f) / (float)p2;
    // at rest, or thermal: a Box-Muller normal deviate per component from
    // the SplitMix64 outputs 8 id + 2c + 1 and 8 id + 2c + 2 (FP64)
    const long long id = id0 + k;
#pragma unroll 1
    for (int c = 0; c < 3; c++)
      S.u[nxt][c][pos] = THERMAL && S.inj_uth > 0.0 ? (float)(S.inj_uth * thermal_normal(S.inj_seed, id, c)) : 0.0f;
    // r-z: a uniform density takes a weight proportional to the radius
    S.w[nxt][pos] = g.cyl ? S.inj_w * ((float)cy + ((float)l1 + 0.5f) / (float)p1 - 0.5f) : S.inj_w;
    S.id[nxt][pos] = (int)(id0 + k);
  }
}

// Workgroups of the scatter: the eight per CU that are resident at once (each
// pays the kernel's prologue, a chain of loads, so more would only wait).
constexpr int kScatterGrid = 2048;

}  // namespace

int pic_plan_tiles() { return PIC_PLAN_TILES; }

hipError_t pic_launch_rebin(const StoreDesc* d_stores, int nstores, int max_items, int total_tiles,
                            int total_blocks, bool big, int inject_max, bool thermal, int parity, hipStream_t st) {
  if (nstores > kMaxGroup || nstores < 1) return hipErrorInvalidValue;
  if (big) {
    hipLaunchKernelGGL(rebin_sums, dim3(total_blocks), dim3(kBlock), 0, st, d_stores, nstores, parity);
    hipLaunchKernelGGL(rebin_fold, dim3(nstores), dim3(kScanBlock), 0, st, d_stores, parity);
    hipLaunchKernelGGL(rebin_offsets, dim3(total_blocks), dim3(kBlock), 0, st, d_stores, nstores, parity);
  }
  auto scatter = [&](auto* kernel) {
    hipLaunchKernelGGL(kernel, dim3(max_items < kScatterGrid ? max_items : kScatterGrid), dim3(kBlock), 0, st, d_stores,
                       nstores, total_tiles, parity);
  };
  if (inject_max == 0)
    scatter(rebin_scatter<0>);
  else if (!thermal)
    scatter(rebin_scatter<1>);
  else
    scatter(rebin_scatter<2>);
  return hipGetLastError();
}
