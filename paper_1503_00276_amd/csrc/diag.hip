// diag.hip -- FP64 diagnostics on the GPU: charge density from the stored
// particle positions, Gauss-law residual div E - rho (Hemker 2000, Ch. 3,
// Sec. 3.1, Eq. maxwell-1 in normalised units), charge-conservation residual
// (rho1 - rho0)/dt + div J (Sec. 3.2, Eq. continuity), and compensated
// (Neumaier) FP64 sums of the field and particle energies and momentum (exact
// ones of the particles with the int64 current); plus the state export.
#include "pic_dev.h"
#include "pic_kernels.h"

namespace {

constexpr int kBlock = 256;
constexpr int kRedBlocks = 512;

// Node-centred B-spline weights of order ORDER for an offset eps in [0,1):
// nodes base..base+ORDER relative to the particle's cell (FP64).
template <int ORDER>
__device__ __forceinline__ int rho_weights(double eps, double w[ORDER + 1]) {
  if constexpr (ORDER == 1) {
    w[0] = 1.0 - eps;
    w[1] = eps;
    return 0;
  } else if constexpr (ORDER == 2) {
    int n = eps >= 0.5 ? 1 : 0;
    double t = eps - n, a = 0.5 - t, b = 0.5 + t;
    w[0] = 0.5 * a * a;
    w[1] = 0.75 - t * t;
    w[2] = 0.5 * b * b;
    return n - 1;
  } else {
    double f = eps, g = 1.0 - f, f2 = f * f, f3 = f2 * f;
    w[0] = g * g * g / 6.0;
    w[1] = (4.0 - 6.0 * f2 + 3.0 * f3) / 6.0;
    w[2] = (1.0 + 3.0 * f + 3.0 * f2 - 3.0 * f3) / 6.0;
    w[3] = f3 / 6.0;
    return -1;
  }
}

// Nodes the shape reaches below and above the particle's cell.
__host__ __device__ inline int rho_below(int order) { return order >= 2 ? 1 : 0; }
__host__ __device__ inline int rho_above(int order) { return order >= 2 ? 2 : 1; }

// How far a particle can sit outside its tile kstep steps after a rebin check
// (as in the fused particle kernel), at most the last step's bound.
__host__ __device__ inline int rho_stray(const GridDesc& g, int d, int s0, int kstep) {
  const int s = s0 + (int)ceilf((float)kstep * g.vstep[d]);
  return s < g.slk[d] ? s : g.slk[d];
}

constexpr int kRhoPer = 4;  // particles per thread and pass over a tile

// Charge density of one species at the nodes, a workgroup per work item: the
// particles of the item (they belong to one tile) are summed on the tile's
// nodes in LDS and the sums are added to the global array once.  Adding every
// particle's (ORDER+1)^DIM contributions to the global array with FP64 atomics
// cost 26.5 ms for 16.8 M particles of a cubic shape (64 each, 40 G adds/s);
// this kernel adds about three sums per particle there and takes 0.72 ms.
// The LDS sums are FP64 too, so a node reached by light particles only keeps its
// relative precision beside heavy ones.  (64-bit integer sums in units of the
// heaviest particle took 0.56 ms there, 143 against 178 us for 7.1 M of a
// quadratic shape, 74 against 71 for a linear one.)
template <int DIM, int ORDER>
__global__ void __launch_bounds__(kBlock) rho64(const StoreDesc* __restrict__ sp, double* rho, int kstep, int par) {
  extern __shared__ double sR[];
  constexpr int NO = ORDER + 1;
  const StoreDesc& S = *sp;
  const GridDesc& g = S.g;
  const int cur = pic_cur(*S.ctl);
  const int total = S.ctl->n_items[cur];
  const int s0 = S.ctl->sorted ? 0 : g.flag_slack;
  const int tid = threadIdx.x;
  const int wo = g.window ? S.win[par].origin : 0;
  const int lo = rho_below(ORDER), hi = rho_above(ORDER);
  for (int ii = blockIdx.x; ii < total; ii += gridDim.x) {
    const Item it = S.items[cur][ii];
    int tc[3], org[3] = {0, 0, 0}, ext[3] = {1, 1, 1}, sl[3] = {0, 0, 0}, R[3] = {1, 1, 1};
    pic_tile_coords(g, it.tile, tc);
#pragma unroll
    for (int d = 0; d < DIM; d++) {
      org[d] = tc[d] * g.tile[d];
      ext[d] = min(g.tile[d], g.nx[d] - org[d]);
      sl[d] = rho_stray(g, d, s0, kstep);
      R[d] = ext[d] + 2 * sl[d] + lo + hi;
    }
    const int rn = R[0] * R[1] * R[2];
    for (int begin = it.begin; begin < it.end; begin += kRhoPer * kBlock) {
      int cell[kRhoPer];
      float w[kRhoPer], e[kRhoPer][DIM];
#pragma unroll
      for (int r = 0; r < kRhoPer; r++) {
        const int p = begin + r * kBlock + tid;
        cell[r] = -1;  // none, or removed (moving window, r-z wall)
        w[r] = 0.0f;
        if (p < it.end) {
          cell[r] = S.cell[cur][p];
          w[r] = S.w[cur][p];
#pragma unroll
          for (int d = 0; d < DIM; d++) e[r][d] = S.eps[cur][d][p];
        }
      }
      for (int q = tid; q < rn; q += kBlock) sR[q] = 0.0;
      __syncthreads();
#pragma unroll
      for (int r = 0; r < kRhoPer; r++) {
        if (cell[r] < 0) continue;
        int c[3];
        pic_unpack(g, cell[r], c);
        double wt[3][NO];
        int at[3] = {0, 0, 0};
#pragma unroll
        for (int d = 0; d < DIM; d++) {
          int l = pic_local(c[d], org[d], ext[d], g.nx[d]);
          l = min(max(l, -sl[d]), ext[d] + sl[d] - 1);
          at[d] = sl[d] + lo + l + rho_weights<ORDER>((double)e[r][d], wt[d]);
        }
        if (g.window) {
          // nodes beyond the window's ends get nothing
          int wc = c[0] - wo;
          if (wc < 0) wc += g.nx[0];
          const int b = at[0] - sl[0] - lo - pic_local(c[0], org[0], ext[0], g.nx[0]);
#pragma unroll
          for (int i = 0; i < NO; i++)
            if ((unsigned)(wc + b + i) >= (unsigned)g.nx[0]) wt[0][i] = 0.0;
        }
        const double q = (double)w[r];
        double* base = sR + at[0] + R[0] * (at[1] + R[1] * at[2]);
#pragma unroll
        for (int k = 0; k < (DIM == 3 ? NO : 1); k++) {
          const double qz = DIM == 3 ? q * wt[2][k] : q;
#pragma unroll
          for (int j = 0; j < NO; j++) {
            const double qy = qz * wt[1][j];
            double* row = base + R[0] * (j + R[1] * k);
#pragma unroll
            for (int i = 0; i < NO; i++)
              __hip_atomic_fetch_add(row + i, qy * wt[0][i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          }
        }
      }
      __syncthreads();
      for (int n = tid; n < rn; n += kBlock) {
        const double v = sR[n];
        if (v == 0.0) continue;
        const int x = n % R[0], y = (n / R[0]) % R[1], z = DIM == 3 ? n / (R[0] * R[1]) : 0;
        const int gx = pic_wrap(org[0] - sl[0] - lo + x, g.nx[0]);
        int gy = org[1] - sl[1] - lo + y;
        if (g.cyl) {
          // r-z: charge below the axis belongs to the mirror row, beyond the
          // wall it is dropped (rows are divided by their ring volume later)
          gy = gy <= 0 ? 1 - gy : gy;
          if (gy >= g.nx[1]) continue;
        } else {
          gy = pic_wrap(gy, g.nx[1]);
        }
        const int gz = DIM == 3 ? pic_wrap(org[2] - sl[2] - lo + z, g.nx[2]) : 0;
        unsafeAtomicAdd(rho + gx + (size_t)g.nx[0] * (gy + (size_t)g.nx[1] * gz), v);
      }
      __syncthreads();
    }
  }
}

// r-z: rho = ion density + (folded ring charge) / (r_j / dr) on the rows
// j >= 1; row 0 holds the image of row 1.
__global__ void rz_rho_finish(double* rho, int nz, int nr, double ion) {
  for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < nz * nr; c += gridDim.x * blockDim.x) {
    const int j = c / nz;
    if (j >= 1) rho[c] = ion + rho[c] / ((double)j - 0.5);
  }
}

__global__ void rz_rho_mirror(double* rho, int nz) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nz; i += gridDim.x * blockDim.x) rho[i] = rho[nz + i];
}

__global__ void fill64(double* p, double v, size_t n) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}

// Backward-difference divergence of a 3-component staggered field at node c.
template <typename T>
// wo: ring origin of a moving window (-1 without one); the x1 neighbour
// behind the window's back column is zero.  r-z: the cylindrical divergence
// dV_z/dz + (1/r) d(r V_r)/dr on the rows j >= 1 (V_r on the half rows j and
// j - 1, radii j dr and (j - 1) dr; the row radius (j - 1/2) dr); row 0
// takes the value of row 1.
__device__ __forceinline__ double div_at(const GridDesc& g, const T* V, int nc, int c, int dim, int wo = -1) {
  if (g.cyl) {
    if (c < g.nx[0]) c += g.nx[0];
    const int i = c % g.nx[0];
    const int j = c / g.nx[0];
    const int cxm = (i > 0) ? c - 1 : c + g.nx[0] - 1;
    const double vxm = (wo >= 0 && i == wo) ? 0.0 : (double)V[cxm];
    return ((double)V[c] - vxm) / g.dxd[0] +
           ((double)j * (double)V[nc + c] - (double)(j - 1) * (double)V[nc + c - g.nx[0]]) /
               (((double)j - 0.5) * g.dxd[1]);
  }
  int i = c % g.nx[0];
  int r = c / g.nx[0];
  int j = r % g.nx[1];
  int k = r / g.nx[1];
  int cxm = (i > 0) ? c - 1 : c + g.nx[0] - 1;
  int cym = (j > 0) ? c - g.nx[0] : c + (g.nx[1] - 1) * g.nx[0];
  const double vxm = (wo >= 0 && i == wo) ? 0.0 : (double)V[cxm];
  double d = ((double)V[c] - vxm) / g.dxd[0] +
             ((double)V[nc + c] - (double)V[nc + cym]) / g.dxd[1];
  if (dim == 3) {
    int sz = g.nx[0] * g.nx[1];
    int czm = (k > 0) ? c - sz : c + (g.nx[2] - 1) * sz;
    d += ((double)V[2 * nc + c] - (double)V[2 * nc + czm]) / g.dxd[2];
  }
  return d;
}

__global__ void __launch_bounds__(kBlock) gauss64(const InstDesc* __restrict__ ip, const double* rho, double* G,
                                                  int dim, int fpar) {
  const InstDesc& I = *ip;
  const int nc = I.g.ncell;
  for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < nc; c += gridDim.x * blockDim.x)
    G[c] = div_at(I.g, I.F[fpar], nc, c, dim, I.g.window ? I.win[fpar].origin : -1) - rho[c];
}

__global__ void __launch_bounds__(kBlock) charge64(const InstDesc* __restrict__ ip, const double* rho0,
                                                   const double* rho1, double* C, int dim, int par) {
  const InstDesc& I = *ip;
  const int nc = I.g.ncell;
  for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < nc; c += gridDim.x * blockDim.x)
    C[c] = (rho1[c] - rho0[c]) / I.g.dtd + div_at(I.g, I.Jout, nc, c, dim, I.g.window ? I.win[par].origin : -1);
}

// ---------------------------------------------------------------------------
// compensated sums: each thread keeps Neumaier (sum, compensation) pairs;
// pairs are merged with an error-free two-sum; per-block pairs are combined by
// a second single-block pass.  Deterministic for a fixed launch shape and order
// of the values (cells; particles have no fixed order).
// ---------------------------------------------------------------------------

struct Pair {
  double s, c;
};

__device__ __forceinline__ void neumaier(Pair& a, double x) {
  double t = a.s + x;
  if (fabs(a.s) >= fabs(x))
    a.c += (a.s - t) + x;
  else
    a.c += (x - t) + a.s;
  a.s = t;
}

__device__ __forceinline__ Pair merge(Pair a, Pair b) {
  Pair r{a.s, a.c + b.c};
  neumaier(r, b.s);
  return r;
}

template <int N>
__device__ void block_reduce_store(Pair (&v)[N], double* partial) {
  __shared__ double ss[N][kBlock], sc[N][kBlock];
  for (int k = 0; k < N; k++) {
    ss[k][threadIdx.x] = v[k].s;
    sc[k][threadIdx.x] = v[k].c;
  }
  __syncthreads();
  for (int off = kBlock / 2; off > 0; off >>= 1) {
    if (threadIdx.x < off)
      for (int k = 0; k < N; k++) {
        Pair a{ss[k][threadIdx.x], sc[k][threadIdx.x]};
        Pair b{ss[k][threadIdx.x + off], sc[k][threadIdx.x + off]};
        Pair r = merge(a, b);
        ss[k][threadIdx.x] = r.s;
        sc[k][threadIdx.x] = r.c;
      }
    __syncthreads();
  }
  if (threadIdx.x == 0)
    for (int k = 0; k < N; k++) {
      partial[(size_t)k * 2 * gridDim.x + 2 * blockIdx.x] = ss[k][0];
      partial[(size_t)k * 2 * gridDim.x + 2 * blockIdx.x + 1] = sc[k][0];
    }
}

// final pass: one block folds nb partial pairs of each of nout sums
__global__ void __launch_bounds__(kBlock) reduce_final(const double* partial, int nb, int nout, double* out) {
  __shared__ double ss[kBlock], sc[kBlock];
  for (int k = 0; k < nout; k++) {
    Pair a{0.0, 0.0};
    for (int b = threadIdx.x; b < nb; b += blockDim.x) {
      Pair x{partial[(size_t)k * 2 * nb + 2 * b], partial[(size_t)k * 2 * nb + 2 * b + 1]};
      a = merge(a, x);
    }
    ss[threadIdx.x] = a.s;
    sc[threadIdx.x] = a.c;
    __syncthreads();
    for (int off = kBlock / 2; off > 0; off >>= 1) {
      if (threadIdx.x < off) {
        Pair r = merge(Pair{ss[threadIdx.x], sc[threadIdx.x]}, Pair{ss[threadIdx.x + off], sc[threadIdx.x + off]});
        ss[threadIdx.x] = r.s;
        sc[threadIdx.x] = r.c;
      }
      __syncthreads();
    }
    if (threadIdx.x == 0) out[k] = ss[0] + sc[0];
    __syncthreads();
  }
}

// sum E^2 and B^2 over all cells (times V/2 applied on the host)
__global__ void __launch_bounds__(kBlock) field_sums(const InstDesc* __restrict__ ip, double* partial, int fpar) {
  const InstDesc& I = *ip;
  const int nc = I.g.ncell;
  Pair v[2] = {{0.0, 0.0}, {0.0, 0.0}};
  for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < nc; c += gridDim.x * blockDim.x) {
    // r-z: each value weighted by its ring volume in units of dz dr^2:
    // 2 pi r / dr off the axis, pi / 4 for the disc of the half rows on the
    // axis, 0 for the image row 0 of the whole-row components
    double vw = 1.0, vh = 1.0;
    if (I.g.cyl) {
      const int j = c / I.g.nx[0];
      const double two_pi = 6.283185307179586;
      vw = j == 0 ? 0.0 : two_pi * ((double)j - 0.5);
      vh = j == 0 ? 0.25 * 3.141592653589793 : two_pi * (double)j;
    }
    for (int k = 0; k < 3; k++) {
      const float* F = I.F[fpar];
      double e = F[(size_t)k * nc + c], b = F[(size_t)(3 + k) * nc + c];
      // whole rows: E_z, E_theta (k = 0, 2), B_r (k = 1); half rows the others
      neumaier(v[0], (k == 1 ? vh : vw) * e * e);
      neumaier(v[1], (k == 1 ? vw : vh) * b * b);
    }
  }
  block_reduce_store<2>(v, partial);
}

// What particle p adds to the sums of w*rqm*(gamma-1) and w*rqm*u (times V on
// the host); false for one that was removed (moving window, r-z wall).
__device__ __forceinline__ bool particle_terms(const StoreDesc& S, int cur, int p, double rqm, double v[4]) {
  if (S.cell[cur][p] < 0) return false;
  double ux = S.u[cur][0][p], uy = S.u[cur][1][p], uz = S.u[cur][2][p];
  double usq = ux * ux + uy * uy + uz * uz;
  double m = (double)S.w[cur][p] * rqm;
  v[0] = m * (usq / (sqrt(1.0 + usq) + 1.0));
  v[1] = m * ux;
  v[2] = m * uy;
  if (S.g.cyl) {
    // r-z: angular momentum about the axis, r u_theta
    const int row = (S.cell[cur][p] >> S.g.sh1) & S.g.m1;
    const double r = ((double)row + (double)S.eps[cur][1][p] - 0.5) * S.g.dxd[1];
    v[3] = m * r * uz;
  } else {
    v[3] = m * uz;
  }
  return true;
}

__global__ void __launch_bounds__(kBlock) particle_sums(const StoreDesc* __restrict__ sp, double rqm,
                                                        double* partial) {
  const StoreDesc& S = *sp;
  const int cur = pic_cur(*S.ctl);
  Pair v[4] = {{0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}};
  for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < S.np; p += gridDim.x * blockDim.x) {
    double t[4];
    if (!particle_terms(S, cur, p, rqm, t)) continue;
#pragma unroll
    for (int k = 0; k < 4; k++) neumaier(v[k], t[k]);
  }
  block_reduce_store<4>(v, partial);
}

// The same sums, exact: the storage order of the particles is not the same from
// run to run (the loader and the rebin place them by atomics), and with the
// int64 current everything else is.  A value's 53-bit mantissa is cut at the
// multiples of 32 bits of its exponent and the pieces are added to 64-bit
// integers, one per 32 bits of the FP64 range: integer sums, so the order does not
// matter; 2^31 particles fit.
// Bound by the LDS adds, most of which meet in a few bins, so the lanes spread
// over eight copies: 4.2 M particles 63 us (one copy 136, the compensated sums 43).
constexpr int kBins = 67;  // 2^-1074 to 2^1024, and the carries
constexpr int kBinCopies = 8;

__global__ void __launch_bounds__(kBlock) particle_sums_exact(const StoreDesc* __restrict__ sp, double rqm,
                                                              unsigned long long* bins) {
  __shared__ unsigned long long sb[kBinCopies][4 * kBins];
  __shared__ unsigned s_odd[4];
  const StoreDesc& S = *sp;
  const int cur = pic_cur(*S.ctl);
  for (int q = threadIdx.x; q < kBinCopies * 4 * kBins; q += kBlock) (&sb[0][0])[q] = 0ull;
  if (threadIdx.x < 4) s_odd[threadIdx.x] = 0u;
  __syncthreads();
  for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < S.np; p += gridDim.x * blockDim.x) {
    double t[4];
    if (!particle_terms(S, cur, p, rqm, t)) continue;
#pragma unroll
    for (int k = 0; k < 4; k++) {
      const unsigned long long b = (unsigned long long)__double_as_longlong(t[k]);
      const bool neg = b >> 63;
      int e = (int)(b >> 52) & 2047;
      unsigned long long m = b & 0xfffffffffffffull;
      if (e == 2047) {  // infinite or not a number
        atomicOr(&s_odd[k], m ? 4u : (neg ? 2u : 1u));
        continue;
      }
      if (e > 0)
        m |= 1ull << 52;
      else
        e = 1;  // (denormal)
      // the value is m 2^(e - 1075): bit e - 1 of the bins is worth 2^(e - 1075)
      const int at = (e - 1) >> 5, sh = (e - 1) & 31;
      const unsigned long long lo = m << sh;                            // bits 0 to 63 of m << sh
      const unsigned long long hi = sh ? m >> (64 - sh) : 0ull;         // the rest (at most 20 bits)
      const unsigned long long piece[3] = {lo & 0xffffffffull, lo >> 32, hi};
      unsigned long long* base = &sb[threadIdx.x % kBinCopies][k * kBins + at];
#pragma unroll
      for (int j = 0; j < 3; j++)
        if (piece[j])
          __hip_atomic_fetch_add(base + j, neg ? 0ull - piece[j] : piece[j], __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  }
  __syncthreads();
  for (int q = threadIdx.x; q < 4 * kBins; q += kBlock) {
    unsigned long long n = 0ull;
#pragma unroll
    for (int c = 0; c < kBinCopies; c++) n += sb[c][q];
    if (n) atomicAdd(bins + q, n);
  }
  if (threadIdx.x < 4 && s_odd[threadIdx.x]) atomicOr((unsigned*)(bins + 4 * kBins + threadIdx.x), s_odd[threadIdx.x]);
}

// The bins of a sum as one FP64 number (a thread per sum).
__global__ void __launch_bounds__(kBlock) particle_sums_round(const unsigned long long* __restrict__ bins, double* out) {
  __shared__ long long sv[4 * kBins];
  for (int q = threadIdx.x; q < 4 * kBins; q += kBlock) sv[q] = (long long)bins[q];
  __syncthreads();
  const int k = threadIdx.x;
  if (k >= 4) return;
  long long* v = sv + k * kBins;
  const unsigned odd = *(const unsigned*)(bins + 4 * kBins + k);
  if (odd) {
    const double inf = __longlong_as_double(0x7ff0000000000000ll);
    out[k] = odd == 1u ? inf : (odd == 2u ? -inf : __longlong_as_double(0x7ff8000000000000ll));
    return;
  }
  // carries: every bin in [0, 2^32), the sign in the last
  auto carry = [&]() {
    for (int b = 0; b + 1 < kBins; b++) {
      v[b + 1] += v[b] >> 32;
      v[b] &= 0xffffffffll;
    }
  };
  carry();
  const bool neg = v[kBins - 1] < 0;
  if (neg) {
    for (int b = 0; b < kBins; b++) v[b] = -v[b];
    carry();
  }
  int top = kBins - 1;
  while (top > 0 && v[top] == 0) top--;
  // the two highest bins hold 33 to 64 bits; a third makes 65 or more, and the
  // last bit stands for everything below
  unsigned long long hi = (unsigned long long)v[top] << 32, lo = 0ull;
  if (top > 0) hi |= (unsigned long long)v[top - 1];
  if (top > 1) lo = (unsigned long long)v[top - 2];
  for (int b = top - 3; b >= 0; b--)
    if (v[b]) lo |= 1ull;
  // to 64 bits with the highest set, then one rounding
  const int z = hi ? __clzll((long long)hi) : 0;  // (below 32: v[top] is not zero unless all are)
  if (z) {
    hi = (hi << z) | (lo >> (32 - z));
    lo = (lo << z) & 0xffffffffull;
  }
  if (lo) hi |= 1ull;
  const double r = ldexp((double)hi, 32 * (top - 1) - z - 1074);
  out[k] = neg ? -r : r;
}

__global__ void __launch_bounds__(kBlock) sq_sums(const double* x, int n, double* partial) {
  Pair v[1] = {{0.0, 0.0}};
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) neumaier(v[0], x[i] * x[i]);
  block_reduce_store<1>(v, partial);
}

// Export position, u and w of every particle into row id (load order).
// With ids != null (moving window, r-z: ids have gaps) rows go to their storage
// index with the id in ids[] (-1 for a removed particle) for the host to sort,
// and positions stay in cell units (cell + offset); else they are scaled,
// xmin + (cell + offset) dx in separate FP64 roundings.
struct Scale {
  double xmin[3], dx[3];
};

__global__ void __launch_bounds__(kBlock) export_state(const StoreDesc* __restrict__ sp, double* out, int* ids,
                                                       Scale sc) {
  const StoreDesc& S = *sp;
  const GridDesc& g = S.g;
  const int cur = pic_cur(*S.ctl);
  const int stride = g.dim + 4;
  for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < S.np; p += gridDim.x * blockDim.x) {
    const int cell = S.cell[cur][p];
    if (ids) ids[p] = cell < 0 ? -1 : S.id[cur][p];
    if (cell < 0) continue;
    int c[3];
    pic_unpack(g, cell, c);
    double* row = out + (size_t)(ids ? p : S.id[cur][p]) * stride;
    for (int d = 0; d < g.dim; d++) {
#pragma clang fp contract(off)
      const double x = (double)c[d] + (double)S.eps[cur][d][p];
      const double s = x * sc.dx[d];
      row[d] = ids ? x : sc.xmin[d] + s;
    }
    row[g.dim + 0] = S.u[cur][0][p];
    row[g.dim + 1] = S.u[cur][1][p];
    row[g.dim + 2] = S.u[cur][2][p];
    row[g.dim + 3] = S.w[cur][p];
  }
}

int grid_for(size_t n) {
  size_t b = (n + kBlock - 1) / kBlock;
  if (b > 4096) b = 4096;
  return b < 1 ? 1 : (int)b;
}

}  // namespace

int pic_reduce_blocks() { return kRedBlocks; }

hipError_t pic_launch_rho64(const StoreDesc* d_store, const GridDesc& g, int max_items, int kstep, int par, double* rho,
                            hipStream_t st) {
  // the largest region: flag_slack is the base after a check that did not re-sort
  size_t lds = sizeof(unsigned long long);
  for (int d = 0; d < g.dim; d++)
    lds *= (size_t)(g.tile[d] + 2 * rho_stray(g, d, g.flag_slack, kstep) + rho_below(g.order) + rho_above(g.order));
  const dim3 grid(max_items < 1 ? 1 : (max_items > 4096 ? 4096 : max_items));
  if (g.dim == 2) {
    if (g.order == 1) rho64<2, 1><<<grid, dim3(kBlock), lds, st>>>(d_store, rho, kstep, par);
    if (g.order == 2) rho64<2, 2><<<grid, dim3(kBlock), lds, st>>>(d_store, rho, kstep, par);
    if (g.order == 3) rho64<2, 3><<<grid, dim3(kBlock), lds, st>>>(d_store, rho, kstep, par);
  } else {
    if (g.order == 1) rho64<3, 1><<<grid, dim3(kBlock), lds, st>>>(d_store, rho, kstep, par);
    if (g.order == 2) rho64<3, 2><<<grid, dim3(kBlock), lds, st>>>(d_store, rho, kstep, par);
    if (g.order == 3) rho64<3, 3><<<grid, dim3(kBlock), lds, st>>>(d_store, rho, kstep, par);
  }
  return hipGetLastError();
}

hipError_t pic_launch_rz_rho_finish(double* rho, int nz, int nr, double ion, hipStream_t st) {
  hipLaunchKernelGGL(rz_rho_finish, dim3(grid_for((size_t)nz * nr)), dim3(kBlock), 0, st, rho, nz, nr, ion);
  hipLaunchKernelGGL(rz_rho_mirror, dim3(grid_for((size_t)nz)), dim3(kBlock), 0, st, rho, nz);
  return hipGetLastError();
}

hipError_t pic_launch_fill64(double* p, double v, size_t n, hipStream_t st) {
  hipLaunchKernelGGL(fill64, dim3(grid_for(n)), dim3(kBlock), 0, st, p, v, n);
  return hipGetLastError();
}

hipError_t pic_launch_gauss64(const InstDesc* d_inst, const double* rho, double* G, int ncell, int dim, int fpar,
                              hipStream_t st) {
  hipLaunchKernelGGL(gauss64, dim3(grid_for(ncell)), dim3(kBlock), 0, st, d_inst, rho, G, dim, fpar);
  return hipGetLastError();
}

hipError_t pic_launch_charge64(const InstDesc* d_inst, const double* rho0, const double* rho1, double* C,
                               int ncell, int dim, int par, hipStream_t st) {
  hipLaunchKernelGGL(charge64, dim3(grid_for(ncell)), dim3(kBlock), 0, st, d_inst, rho0, rho1, C, dim, par);
  return hipGetLastError();
}

hipError_t pic_launch_field_sums(const InstDesc* d_inst, int ncell, int fpar, double* scratch, double* out,
                                 hipStream_t st) {
  (void)ncell;
  hipLaunchKernelGGL(field_sums, dim3(kRedBlocks), dim3(kBlock), 0, st, d_inst, scratch, fpar);
  hipLaunchKernelGGL(reduce_final, dim3(1), dim3(kBlock), 0, st, scratch, kRedBlocks, 2, out);
  return hipGetLastError();
}

hipError_t pic_launch_particle_sums(const StoreDesc* d_store, double rqm, bool exact, double* scratch, double* out,
                                    hipStream_t st) {
  if (exact) {
    static_assert(4 * kBins + 4 <= 2 * 4 * kRedBlocks, "the bins fit the scratch");
    unsigned long long* bins = (unsigned long long*)scratch;
    hipLaunchKernelGGL(fill64, dim3(1), dim3(kBlock), 0, st, scratch, 0.0, (size_t)(4 * kBins + 4));
    hipLaunchKernelGGL(particle_sums_exact, dim3(kRedBlocks), dim3(kBlock), 0, st, d_store, rqm, bins);
    hipLaunchKernelGGL(particle_sums_round, dim3(1), dim3(kBlock), 0, st, bins, out);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(particle_sums, dim3(kRedBlocks), dim3(kBlock), 0, st, d_store, rqm, scratch);
  hipLaunchKernelGGL(reduce_final, dim3(1), dim3(kBlock), 0, st, scratch, kRedBlocks, 4, out);
  return hipGetLastError();
}

hipError_t pic_launch_sq_sums(const double* v, int n, double* scratch, double* out, hipStream_t st) {
  hipLaunchKernelGGL(sq_sums, dim3(kRedBlocks), dim3(kBlock), 0, st, v, n, scratch);
  hipLaunchKernelGGL(reduce_final, dim3(1), dim3(kBlock), 0, st, scratch, kRedBlocks, 1, out);
  return hipGetLastError();
}

hipError_t pic_launch_export_state(const StoreDesc* d_store, int np, double* out, int* ids, const double* xmin,
                                   const double* dx, hipStream_t st) {
  Scale sc{};
  for (int d = 0; d < 3 && xmin; d++) {
    sc.xmin[d] = xmin[d];
    sc.dx[d] = dx[d];
  }
  hipLaunchKernelGGL(export_state, dim3(grid_for(np)), dim3(kBlock), 0, st, d_store, out, ids, sc);
  return hipGetLastError();
}
