// d2q9_vortex.hpp -- the stream function Psi and vortex extraction from it
// (the stream-function values and vortex centres of Tables 1-2): arg-extrema
// of Psi over three regions and the list of all vortex centres.
//
// Psi is a dense FP64 [ny][nx] field (k_psi).  Sites are addressed by their
// linear index k = y nx + x.
#pragma once
#include <hip/hip_runtime.h>

#include "d2q9_monitor.hpp"

namespace lbm {

constexpr int kVortexThreads = 256;
constexpr int kVortexRegions = 3;

// Region r of site (x, y): 0 = whole lattice (maximum of Psi: the primary
// vortex); 1 = x < nx/2, y < hy and 2 = x >= nx/2, y < hy (minimum of Psi:
// the lower-left and lower-right vortices), hy = min(ny, nx/2).
__device__ __forceinline__ bool in_region(int r, int x, int y, int nx, int hy) {
  if (r == 0) return true;
  if (y >= hy) return false;
  return r == 1 ? x < nx / 2 : x >= nx / 2;
}

// a better than b: strictly larger (region 0) or smaller (1, 2) value, ties
// to the smaller site index; index -1 marks "no candidate".
__device__ __forceinline__ bool better(int r, double av, int ak, double bv, int bk) {
  if (ak < 0) return false;
  if (bk < 0) return true;
  if (av != bv) return r == 0 ? av > bv : av < bv;
  return ak < bk;
}

// Reduce the per-thread candidates of one NT-thread block, all regions in the
// same passes, in LDS; thread 0 ends with the block's best.  The result does
// not depend on the order of reduction (the comparison is a total order), so
// it is deterministic.
template <int NT>
__device__ __forceinline__ void block_best(double (&v)[kVortexRegions], int (&k)[kVortexRegions]) {
  __shared__ double sv[kVortexRegions][NT / 64];
  __shared__ int sk[kVortexRegions][NT / 64];
  const int t = threadIdx.x;
#pragma unroll
  for (int r = 0; r < kVortexRegions; ++r) {
    // the wavefront first, by lane exchange
    for (int off = 32; off > 0; off >>= 1) {
      const double ov = __shfl_xor(v[r], off, 64);
      const int ok = __shfl_xor(k[r], off, 64);
      if (better(r, ov, ok, v[r], k[r])) {
        v[r] = ov;
        k[r] = ok;
      }
    }
    if ((t & 63) == 0) {
      sv[r][t >> 6] = v[r];
      sk[r][t >> 6] = k[r];
    }
  }
  __syncthreads();
  if (t == 0)
#pragma unroll
    for (int r = 0; r < kVortexRegions; ++r)
      for (int w = 1; w < NT / 64; ++w)
        if (better(r, sv[r][w], sk[r][w], v[r], k[r])) {
          v[r] = sv[r][w];
          k[r] = sk[r][w];
        }
}

// Stream function up each column, a running sum from the bottom wall:
//   half-way walls: Psi(y) = -(sum_{y' < y} u_x(y') + u_x(y) / 2), the
//   midpoint rule on site centres;
//   on-node walls (g.on_node): Psi(0) = 0, Psi(y) = Psi(y - 1) - (u_x(y - 1)
//   + u_x(y)) / 2, the trapezoid rule.
// A block owns kPsiCols columns and takes them 64 J rows at a time: all
// its threads compute the terms of the sum (u_x; on nodes the half sum of
// neighbours, exact scalings of what the formula adds) into LDS, one lane
// per column replaces them by the running sums in row order (an addition
// per row, so the order does not depend on the tiling), and all threads
// form Psi and store it.  The next tile is loaded while the sums run.
// EXT: also each block's best site of every region, partials
// [region][block].  *zero (if not null) is cleared for the kernel after it.
// Bound by latency: the loads of a tile, then its chain of additions (about
// 12 cycles a row).  500 x 600 FP64: 20 us, 28 with the extrema; one thread
// per column, nine loads and the addition row by row, took 290 us.  J = 8 rows
// per thread; 1 on lattices of up to 64 rows, where the other seven would
// be beyond the lattice (16 x 16 FP64, whole call: 27.0 -> 24.0 us).
constexpr int kPsiThreads = 512, kPsiCols = 8;
template <typename T, bool SHIFT, bool EXT, bool NODE, int J>
__global__ __launch_bounds__(kPsiThreads) void k_psi(const T *__restrict__ s, Geometry g,
                                                     double *__restrict__ psi,
                                                     double *__restrict__ pv,
                                                     int *__restrict__ pk,
                                                     unsigned int *__restrict__ zero) {
  constexpr int C = kPsiCols, R = J * kPsiThreads / C;   // rows of a tile, J per thread
  constexpr int E = NODE ? 1 : 0;                        // and the row below them
  __shared__ double col[R * C];
  const int c = threadIdx.x % C, r0 = threadIdx.x / C * J;
  const int b = xcd_tile(blockIdx.x, gridDim.x);
  const int x = b * C + c, nx = g.nx, ny = g.ny, hy = min(ny, nx / 2);
  const bool in = x < nx;
  if (zero && blockIdx.x == 0 && threadIdx.x == 0) *zero = 0u;
  double bv[kVortexRegions];
  int bk[kVortexRegions];
#pragma unroll
  for (int r = 0; r < kVortexRegions; ++r) {
    bv[r] = 0.0;
    bk[r] = -1;
  }
  double ux[J + E], acc = 0.0;
  // (rows and columns beyond the lattice read its last ones: no branch, so
  // all of a thread's loads are in flight together)
  auto load = [&](int yb) {
    T v[J + E][9];
#pragma unroll
    for (int j = 0; j < J + E; ++j) {
      const int o = min(max(yb + r0 + j - E, 0), ny - 1) * g.pitch + min(x, nx - 1);
#pragma unroll
      for (int i = 0; i < 9; ++i) v[j][i] = s[i * g.plane + o];
    }
#pragma unroll
    for (int j = 0; j < J + E; ++j) {
      double drho, jx, jy;
      moments_of<T, SHIFT>(v[j], drho, jx, jy);
      ux[j] = jx / (1.0 + drho);
    }
  };
  load(0);
  for (int yb = 0; yb < ny; yb += R) {
    const int rows = min(R, ny - yb);
    double half[J];                 // half-way walls: u_x / 2 of the site itself
#pragma unroll
    for (int j = 0; j < J; ++j) {
      half[j] = 0.5 * ux[j];
      double t = ux[j];
      if constexpr (NODE) t = yb + r0 + j == 0 ? 0.0 : 0.5 * (ux[j] + ux[j + 1]);
      col[(r0 + j) * C + c] = t;
    }
    __syncthreads();
    if (yb + R < ny) load(yb + R);
    if (threadIdx.x < C) {   // the next U terms are read while U are summed
      constexpr int U = 16;
      static_assert(R % U == 0, "whole groups");
      double u[U], nu[U];
#pragma unroll
      for (int j = 0; j < U; ++j) u[j] = col[j * C + c];
      for (int r = 0; r < rows; r += U) {
        double *at = col + r * C + c, *next = r + U < R ? at + U * C : at;
#pragma unroll
        for (int j = 0; j < U; ++j) nu[j] = next[j * C];
#pragma unroll
        for (int j = 0; j < U; ++j) {
          if constexpr (NODE) {
            acc -= u[j];
            at[j * C] = acc;
          } else {
            at[j * C] = acc;
            acc += u[j];
          }
        }
#pragma unroll
        for (int j = 0; j < U; ++j) u[j] = nu[j];
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int r = r0 + j, y = yb + r;
      if (in && r < rows) {
        const double p = NODE ? col[r * C + c] : -(col[r * C + c] + half[j]);
        const int q = y * nx + x;
        psi[q] = p;
        if (EXT)
#pragma unroll
          for (int e = 0; e < kVortexRegions; ++e)
            if (in_region(e, x, y, nx, hy) && better(e, p, q, bv[e], bk[e])) {
              bv[e] = p;
              bk[e] = q;
            }
      }
    }
    __syncthreads();
  }
  if (EXT) {
    block_best<kPsiThreads>(bv, bk);
    if (threadIdx.x == 0)
#pragma unroll
      for (int e = 0; e < kVortexRegions; ++e) {
        pv[e * gridDim.x + blockIdx.x] = bv[e];
        pk[e * gridDim.x + blockIdx.x] = bk[e];
      }
  }
}

// What the host reads of a vortex call, copied in one piece: the extrema,
// the number of centres, and the first kVortexFirst of them (the rest
// are fetched by a second copy; see find_vortices in lbm.hip).
constexpr int kVortexFirst = 64;
struct VortexOut {
  double v[kVortexRegions];
  int k[kVortexRegions];
  unsigned int count;
};
struct VortexCentre {
  double psi;
  int k, kind;
};

// One block: best of the nb partials of each region into out.
static __global__ __launch_bounds__(kVortexThreads) void k_vortex_final(
    const double *__restrict__ pv, const int *__restrict__ pk, int nb,
    VortexOut *__restrict__ out) {
  double v[kVortexRegions];
  int k[kVortexRegions];
#pragma unroll
  for (int r = 0; r < kVortexRegions; ++r) {
    v[r] = 0.0;
    k[r] = -1;
    for (int b = threadIdx.x; b < nb; b += kVortexThreads)
      if (better(r, pv[r * nb + b], pk[r * nb + b], v[r], k[r])) {
        v[r] = pv[r * nb + b];
        k[r] = pk[r * nb + b];
      }
  }
  block_best<kVortexThreads>(v, k);
  if (threadIdx.x == 0)
#pragma unroll
    for (int r = 0; r < kVortexRegions; ++r) {
      out->v[r] = v[r];
      out->k[r] = k[r];
    }
}

// Vortex centres: interior sites (1 <= x <= nx-2, 1 <= y <= ny-2) where Psi
// is strictly above (kind +1) or strictly below (kind -1) all eight
// neighbours and |Psi| >= min_abs.  Each centre takes a slot from *count
// (a global atomic) and, if the slot is below cap, stores (Psi, k, kind);
// the slots come in no particular order.
static __global__ __launch_bounds__(kVortexThreads) void k_vortex_centres(
    const double *__restrict__ psi, int nx, int ny, double min_abs, int cap,
    unsigned int *__restrict__ count, VortexCentre *__restrict__ list) {
  const int q = blockIdx.x * kVortexThreads + threadIdx.x;
  if (q >= nx * ny) return;
  const int y = q / nx, x = q - y * nx;
  if (x < 1 || x > nx - 2 || y < 1 || y > ny - 2) return;
  const double c = psi[q];
  if (!(fabs(c) >= min_abs)) return;
  bool mx = true, mn = true;
#pragma unroll
  for (int dy = -1; dy <= 1; ++dy)
#pragma unroll
    for (int dx = -1; dx <= 1; ++dx) {
      if (dx == 0 && dy == 0) continue;
      const double b = psi[q + dy * nx + dx];
      mx = mx && c > b;
      mn = mn && c < b;
    }
  if (!mx && !mn) return;
  const unsigned int slot = atomicAdd(count, 1u);
  if (slot < (unsigned int)cap) list[slot] = VortexCentre{c, q, mx ? 1 : -1};
}

}  // namespace lbm
