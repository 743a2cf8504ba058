// load.hip -- loading particles: positions to cells and in-cell offsets, the
// counting sort by tile and, inside a tile, the order the fused kernel wants:
// the first particle of every cell, cell by cell, then the second of every
// cell, and so on (the lanes of a wavefront then sit in different cells and
// their current deposits hit different LDS addresses).
//
// The particles already in the store and the new ones are sorted together into
// the store's other buffer set (or new arrays):
//   count   (per particle)  checks, cell counts, the particle's rank in its cell
//   sums    (per tile)      particles of the tile
//   plan    (one workgroup) tile offsets, work items
//   slots   (per tile)      place of every (cell, rank) of the tile
//   place   (per particle)  converted and written to its place
// Bound by memory: 48 or 56 B of FP64 input (2D, 3D) read twice and 32 or 36 B
// of state written once per particle, besides its rank and its place (4 B each,
// written and read).  On one host thread (copies to the host included) a load took
// 2.0 ms for 65,536 particles and about 70 ns for each of 16.8 M.
#include <climits>

#include "pic_dev.h"
#include "pic_kernels.h"
#include "pic_plan.h"

namespace {

constexpr int kBlock = 256;
constexpr int kPlanBlock = 1024;

// Cell coordinates and offsets of new particle q; false outside the window
// (*why = 0) or beyond the wall (*why = 1).
__device__ __forceinline__ bool load_convert(const LoadArgs& A, long long q, int c[3], float e[3], int* why) {
  const GridDesc& g = A.g;
  for (int d = 0; d < g.dim; d++) {
    const double L = (double)g.nx[d];
    const double x = A.x[q * g.dim + d];
    double xi = (x - A.xmin[d]) / g.dxd[d];
    if (g.cyl && d == 1) {
      // r-z: x2 is the radius; the cell coordinate is r/dr + 1/2
      xi = x / g.dxd[1] + 0.5;
      if (!(x >= 0.0 && xi < L)) {
        *why = 1;
        return false;
      }
    }
    if (g.window && d == 0) {
      // window position, then ring column
      xi -= (double)A.shifts;
      if (!(xi >= 0.0 && xi < L)) {
        *why = 0;
        return false;
      }
      xi += (double)A.origin;
    }
    if (!(xi >= 0.0 && xi < L)) {
      xi = fmod(xi, L);
      if (xi < 0.0) xi += L;
      if (xi >= L) xi -= L;
    }
    const double f = floor(xi);
    int ci = (int)f;
    float ei = (float)(xi - f);
    if (ei >= 1.0f) {
      ei = 0.0f;
      ci += 1;
    }
    if (ci >= g.nx[d]) ci -= g.nx[d];
    c[d] = ci;
    e[d] = ei;
  }
  return true;
}

__device__ __forceinline__ bool finite64(double v) { return fabs(v) <= 1.7976931348623157e308; }

__global__ void __launch_bounds__(kBlock) load_count(const LoadArgs A) {
  const GridDesc& g = A.g;
  unsigned flags = 0;
  unsigned long long first = ~0ull;
  double um = 0.0, wm = 0.0;
  int idm = -1;
  for (long long p = blockIdx.x * (long long)kBlock + threadIdx.x; p < A.old + A.n; p += (long long)gridDim.x * kBlock) {
    int c[3] = {0, 0, 0};
    float u[3];
    if (p < A.old) {
      pic_unpack(g, A.ocell[p], c);
      for (int k = 0; k < 3; k++) u[k] = A.ou[k][p];
      idm = max(idm, A.oid[p]);
    } else {
      const long long q = p - A.old;
      unsigned bad = 0;
      for (int d = 0; d < g.dim; d++)
        if (!finite64(A.x[q * g.dim + d])) bad |= 1;
      for (int k = 0; k < 3; k++) {
        const double v = A.u[q * 3 + k];
        if (!finite64(v)) bad |= 2;
        u[k] = (float)v;
      }
      const double w = A.w[q];
      if (!finite64(w)) bad |= 4;
      flags |= bad;
      if (bad) continue;
      wm = fmax(wm, fabs(w));
      float e[3];
      int why = 0;
      if (!load_convert(A, q, c, e, &why)) {
        const unsigned long long at = (unsigned long long)q * 2 + why;
        if (at < first) first = at;
        continue;
      }
    }
    um = fmax(um, (double)u[0] * u[0] + (double)u[1] * u[1] + (double)u[2] * u[2]);
    A.rank[p] = atomicAdd(&A.cells[pic_load_key(g, c)], 1);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    flags |= __shfl_xor(flags, off);
    um = fmax(um, __shfl_xor(um, off));
    wm = fmax(wm, __shfl_xor(wm, off));
    idm = max(idm, __shfl_xor(idm, off));
    const unsigned long long o = __shfl_xor(first, off);
    if (o < first) first = o;
  }
  // One thread per workgroup reports, and only what the status does not hold
  // yet: it grows (first: falls) only, so a value read late costs an atomic
  // and never a result.  Three atomics of every wavefront on one cache line
  // bounded the kernel: 65,536 particles 43 -> 14 us, 2.1 M 625 -> 198,
  // 45x37x53 cells at 6 297 -> 55, 16.8 M (bound by the cells' counts) 1,560
  // -> 1,430.
  constexpr int W = kBlock / 64;
  __shared__ double s_u[W], s_w[W];
  __shared__ unsigned long long s_first[W];
  __shared__ unsigned s_flags[W];
  __shared__ int s_id[W];
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    s_u[wave] = um;
    s_w[wave] = wm;
    s_first[wave] = first;
    s_flags[wave] = flags;
    s_id[wave] = idm;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
#pragma unroll
  for (int k = 1; k < W; k++) {
    um = fmax(um, s_u[k]);
    wm = fmax(wm, s_w[k]);
    first = s_first[k] < first ? s_first[k] : first;
    flags |= s_flags[k];
    idm = max(idm, s_id[k]);
  }
  auto now = [](auto* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  // (nonnegative doubles are ordered like their bits)
  const unsigned long long ub = (unsigned long long)__double_as_longlong(um);
  const unsigned long long wb = (unsigned long long)__double_as_longlong(wm);
  LoadStatus* st = A.status;
  if (flags) atomicOr(&st->flags, flags);
  if (first != ~0ull) atomicMin(&st->first, first);
  if (ub > now(&st->u2)) atomicMax(&st->u2, ub);
  if (wb > now(&st->w)) atomicMax(&st->w, wb);
  if (idm > now(&st->idmax)) atomicMax(&st->idmax, idm);
}

// Particles of each tile, a wavefront per tile.
__global__ void __launch_bounds__(kBlock) load_sums(const LoadArgs A) {
  const int vol = A.g.tile[0] * A.g.tile[1] * A.g.tile[2];
  const int lane = threadIdx.x & 63;
  for (int t = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6); t < A.g.ntiles; t += gridDim.x * (kBlock / 64)) {
    int n = 0;
    for (int k = lane; k < vol; k += 64) n += A.cells[(size_t)t * vol + k];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) n += __shfl_xor(n, off);
    if (lane == 0) A.tiles[t] = n;
  }
}

__global__ void __launch_bounds__(kPlanBlock) load_plan(const LoadArgs A, const StoreDesc S, int set) {
  const int nt = A.g.ntiles;
  int na = 0, ni = 0;
  for (int base = 0; base < nt; base += kPlanBlock) {
    const int t = base + threadIdx.x;
    const int c = t < nt ? A.tiles[t] : 0;
    int ea, eb, ta, tb;
    block_scan2<kPlanBlock>(c, pic_item_count(c, S.chunk), ea, eb, ta, tb);
    if (t < nt) plan_tile(S, set, t, c, na + ea, ni + eb);
    na += ta;
    ni += tb;
  }
  if (threadIdx.x == 0) {
    S.toff[set][nt] = na;
    S.ioff[set][nt] = ni;
    A.status->items = ni;
  }
}

// Places of a tile's particles: rank r of the cells that have one, in cell
// order, after all lower ranks.  The ranks from one count that occurs in the
// tile up to the next go to the same cells, so they are placed together: a round
// for each different count, however many particles a cell has.  (A round per
// rank, and no interleaving past the 512th, left a 64x64 box at 2,000 per cell
// with wavefronts in one cell: 197 us a step, linear, 280 quadratic.)
// A round is a chain of a few LDS reads, shuffles and one barrier; the cells that
// have its ranks write them themselves where there are few, and are listed for
// the whole workgroup where there are many.
constexpr int kSlotBytes = 2 * sizeof(int) + sizeof(unsigned short);  // LDS per cell of a tile

__global__ void __launch_bounds__(kBlock) load_slots(const LoadArgs A, const int* __restrict__ toff) {
  extern __shared__ int lds[];
  constexpr int W = kBlock / 64;
  __shared__ int s_n[2][W], s_top[2][W];
  const int vol = A.g.tile[0] * A.g.tile[1] * A.g.tile[2];
  int* cnt = lds;                                          // particles of each cell
  int* first = lds + vol;                                  // its first place in the (cell, rank) list
  unsigned short* act = (unsigned short*)(lds + 2 * vol);  // the cells that have the round's ranks
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const unsigned long long lt = (1ull << lane) - 1ull;
  // each wavefront looks at a run of the cells
  const int per = (vol + kBlock - 1) / kBlock * 64, k0 = wave * per, k1 = min(vol, k0 + per);
  for (int t = blockIdx.x; t < A.g.ntiles; t += gridDim.x) {
    int* cells = A.cells + (size_t)t * vol;
    int run = toff[t], at = run;  // at: places given out
    for (int base = 0; base < vol; base += kBlock) {
      const int k = base + tid;
      const int c = k < vol ? cells[k] : 0;
      int ea, eb, ta, tb;
      block_scan2<kBlock>(c, 0, ea, eb, ta, tb);
      if (k < vol) {
        cnt[k] = c;
        first[k] = cells[k] = run + ea;
      }
      run += ta;
    }
    __syncthreads();
    for (int r = 0, par = 0;; par ^= 1) {
      int n = 0, top = INT_MAX;  // the cells of more than r, and the smallest count of them
      for (int k = k0; k < k1; k += 64) {
        const int c = k + lane < k1 ? cnt[k + lane] : 0;
        n += (int)__popcll(__ballot(c > r));
        if (c > r) top = min(top, c);
      }
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) top = min(top, __shfl_xor(top, off));
      if (lane == 0) {
        s_n[par][wave] = n;
        s_top[par][wave] = top;
      }
      __syncthreads();  // (the other parity's entries may still be read)
      int na = 0, j0 = 0;
#pragma unroll
      for (int w = 0; w < W; w++) {
        if (w < wave) j0 += s_n[par][w];
        na += s_n[par][w];
        top = min(top, s_top[par][w]);
      }
      if (na == 0) break;  // (the same in every thread)
      const int ranks = top - r;
      const bool list = ranks > 4;
      for (int k = k0; k < k1; k += 64) {
        const bool has = k + lane < k1 && cnt[k + lane] > r;
        const unsigned long long m = __ballot(has);
        const int j = j0 + (int)__popcll(m & lt);
        if (has && list) act[j] = (unsigned short)(k + lane);
        if (has && !list)
          for (int q = 0; q < ranks; q++) A.slot[first[k + lane] + r + q] = at + q * na + j;
        j0 += (int)__popcll(m);
      }
      if (list) {
        __syncthreads();
        // consecutive threads take consecutive ranks of a cell, which lie together
        for (int p = tid; p < na * ranks; p += kBlock) {
          const int j = p / ranks, q = p - j * ranks;
          A.slot[first[act[j]] + r + q] = at + q * na + j;
        }
        __syncthreads();  // the list is read before another round writes it
      }
      at += na * ranks;
      r = top;
    }
    __syncthreads();  // the counts are read before the next tile's are written
  }
}

__global__ void __launch_bounds__(kBlock) load_place(const LoadArgs A, const StoreDesc S, int set) {
  const GridDesc& g = A.g;
  for (long long p = blockIdx.x * (long long)kBlock + threadIdx.x; p < A.old + A.n; p += (long long)gridDim.x * kBlock) {
    int c[3] = {0, 0, 0}, cell, id;
    float e[3] = {0.0f, 0.0f, 0.0f}, u[3], w;
    if (p < A.old) {
      cell = A.ocell[p];
      pic_unpack(g, cell, c);
      for (int d = 0; d < g.dim; d++) e[d] = A.oeps[d][p];
      for (int k = 0; k < 3; k++) u[k] = A.ou[k][p];
      w = A.ow[p];
      id = A.oid[p];
    } else {
      const long long q = p - A.old;
      int why;
      (void)load_convert(A, q, c, e, &why);
      cell = pic_pack(g, c[0], c[1], c[2]);
      for (int k = 0; k < 3; k++) u[k] = (float)A.u[q * 3 + k];
      w = (float)A.w[q];
      id = (int)(A.id0 + q);
    }
    const int pos = A.slot[A.cells[pic_load_key(g, c)] + A.rank[p]];
    S.cell[set][pos] = cell;
    for (int d = 0; d < g.dim; d++) S.eps[set][d][pos] = e[d];
    for (int k = 0; k < 3; k++) S.u[set][k][pos] = u[k];
    S.w[set][pos] = w;
    S.id[set][pos] = id;
  }
}

__global__ void __launch_bounds__(kBlock) neighbour_table(const GridDesc g, int* ndst) {
  for (int q = blockIdx.x * kBlock + threadIdx.x; q < g.ntiles * PIC_NSLOT; q += gridDim.x * kBlock) {
    const int t = q / PIC_NSLOT, sl = q - t * PIC_NSLOT;
    const int dd[3] = {sl % 3 - 1, (sl / 3) % 3 - 1, sl / 9 - 1};
    int tc[3];
    pic_tile_coords(g, t, tc);
    for (int d = 0; d < 3; d++) tc[d] = pic_wrap(tc[d] + dd[d], g.ntile[d]);
    ndst[q] = pic_tile_index(g, tc[0], tc[1], tc[2]);
  }
}

int grid_of(long long n, int per) {
  const long long b = (n + per - 1) / per;
  return b < 1 ? 1 : (b > 4096 ? 4096 : (int)b);
}

}  // namespace

hipError_t pic_launch_load_count(const LoadArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(load_count, dim3(grid_of(a.old + a.n, kBlock)), dim3(kBlock), 0, st, a);
  return hipGetLastError();
}

hipError_t pic_launch_load_place(const LoadArgs& a, const StoreDesc& s, int set, hipStream_t st) {
  const int vol = a.g.tile[0] * a.g.tile[1] * a.g.tile[2];
  hipLaunchKernelGGL(load_sums, dim3(grid_of(a.g.ntiles, kBlock / 64)), dim3(kBlock), 0, st, a);
  hipLaunchKernelGGL(load_plan, dim3(1), dim3(kPlanBlock), 0, st, a, s, set);
  hipLaunchKernelGGL(load_slots, dim3(grid_of(a.g.ntiles, 1)), dim3(kBlock), vol * kSlotBytes, st, a,
                     s.toff[set]);
  hipLaunchKernelGGL(load_place, dim3(grid_of(a.old + a.n, kBlock)), dim3(kBlock), 0, st, a, s, set);
  return hipGetLastError();
}

hipError_t pic_launch_neighbour_table(const GridDesc& g, int* ndst, hipStream_t st) {
  hipLaunchKernelGGL(neighbour_table, dim3(grid_of((long long)g.ntiles * PIC_NSLOT, kBlock)), dim3(kBlock), 0, st, g,
                     ndst);
  return hipGetLastError();
}
