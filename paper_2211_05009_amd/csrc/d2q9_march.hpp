// d2q9_march.hpp -- K steps of Eq. 1 per launch in registers: a wavefront
// marches up a strip of columns.
#pragma once
#include <hip/hip_runtime.h>

#include "d2q9_monitor.hpp"
#include "d2q9_step.hpp"
#include "d2q9_temporal.hpp"

namespace lbm {

// Strip geometry: a wavefront holds S adjacent columns per lane, 64 S in
// all, and stores all but M on each side that is not a wall.
template <int K, int S>
struct MarchGeom {
  static constexpr int WW = 64 * S;
  static constexpr int M = S == 1 ? K : (K + 1) / 2 * 2;
  static constexpr int TX = WW - 2 * M;
  static __host__ __device__ int strips(int nx) {
    return nx <= WW ? 1 : (nx - 2 * M + TX - 1) / TX;
  }
};

// The value of the lane below (UP) or above; the window's first (last) lane
// keeps `old`.
template <bool UP>
__device__ __forceinline__ int lane_shift(int old, int v) {
  // wave_shr:1 = 0x138, wave_shl:1 = 0x130
  return __builtin_amdgcn_update_dpp(old, v, UP ? 0x138 : 0x130, 0xf, 0xf, false);
}
template <bool UP>
__device__ __forceinline__ float lane_shift(float old, float v) {
  return __builtin_bit_cast(
      float, lane_shift<UP>(__builtin_bit_cast(int, old), __builtin_bit_cast(int, v)));
}
template <bool UP>
__device__ __forceinline__ double lane_shift(double old, double v) {
  typedef int i2 __attribute__((ext_vector_type(2)));
  const i2 o = __builtin_bit_cast(i2, old), a = __builtin_bit_cast(i2, v);
  i2 r;
  r.x = lane_shift<UP>(o.x, a.x);
  r.y = lane_shift<UP>(o.y, a.y);
  return __builtin_bit_cast(double, r);
}

template <typename T, bool SHIFT, int K, int S, int MON, bool WALL, bool NARROW>
__device__ __forceinline__ void march_tile(const T *__restrict__ src, T *__restrict__ dst, int nx,
                                           int ny, int pitch, int P, T omega, T u6, int X0, int c0,
                                           int c1, int y0, int y1, const TbMonBlock &mon) {
  const int lane = threadIdx.x & 63;
  const int gx = X0 + lane * S;                       // the lane's first column
  const int lx = NARROW ? min(gx, pitch - S) : gx;    // columns loaded
  // value arriving from x - 1 / x + 1; `old` at the wall
  auto from_left = [&](const T(&v)[S], const T(&old)[S], T(&r)[S]) {
    r[0] = lane_shift<true>(WALL ? old[0] : v[S - 1], v[S - 1]);
    if constexpr (S == 2) r[1] = v[0];
  };
  auto from_right = [&](const T(&v)[S], const T(&old)[S], T(&r)[S]) {
    r[S - 1] = lane_shift<false>(WALL ? old[S - 1] : v[0], v[0]);
    if constexpr (S == 2) r[0] = v[1];
    if constexpr (NARROW) {
#pragma unroll
      for (int k = 0; k < S; ++k)
        if (gx + k == nx - 1) r[k] = old[k];
    }
  };
  T cur[K][9][S];    // row below the incoming one: 0, 1, 3, 2, 5, 6 are used
  T prev[K][3][S];   // links 2, 5, 6 arriving at that row from the row below it
#pragma unroll
  for (int s = 0; s < K; ++s)
#pragma unroll
    for (int k = 0; k < S; ++k) {
#pragma unroll
      for (int i = 0; i < 9; ++i) cur[s][i][k] = T(0);
#pragma unroll
      for (int i = 0; i < 3; ++i) prev[s][i][k] = T(0);
    }
  T nxt[9][S];
  auto load = [&](int row) {
    const unsigned o = (unsigned)(min(row, ny - 1) * pitch + lx) * (unsigned)sizeof(T);
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      const char *pl = reinterpret_cast<const char *>(src + (size_t)i * P);
      VecT<T, S> t;
      __builtin_memcpy(&t, pl + o, sizeof t);
#pragma unroll
      for (int k = 0; k < S; ++k) nxt[i][k] = t.v[k];
    }
  };
  const int qs = max(0, y0 - K), qe = y1 + K;
  load(qs);
  const bool st = gx + S - 1 >= c0 && gx < c1;
#pragma unroll 2
  for (int q = qs; q < qe; ++q) {
    T in[9][S];
#pragma unroll
    for (int i = 0; i < 9; ++i)
#pragma unroll
      for (int k = 0; k < S; ++k) in[i][k] = nxt[i][k];
    load(q + 1);
#pragma unroll
    for (int s = 1; s <= K; ++s) {
      T(&c)[9][S] = cur[s - 1];
      T(&pv)[3][S] = prev[s - 1];
      const int row = q - s;           // the row this level updates
      const int lo = max(0, y0 - (K - s)), hi = min(ny, y1 + (K - s));
      const bool act = row >= lo && row < hi;
      T f[9][S];
      if (act) {
#pragma unroll
        for (int k = 0; k < S; ++k) {
          f[0][k] = c[0][k];
          f[2][k] = pv[0][k];
          f[5][k] = pv[1][k];
          f[6][k] = pv[2][k];
        }
        from_left(c[1], c[3], f[1]);
        from_right(c[3], c[1], f[3]);
        if (WALL && row == ny - 1) {
#pragma unroll
          for (int k = 0; k < S; ++k) {
            f[4][k] = c[2][k];
            f[7][k] = c[5][k] - u6;
            f[8][k] = c[6][k] + u6;
          }
        } else {
#pragma unroll
          for (int k = 0; k < S; ++k) f[4][k] = in[4][k];
          from_right(in[7], c[5], f[7]);
          from_left(in[8], c[6], f[8]);
        }
      }
      // the incoming row becomes the current one
      if (WALL && q - (s - 1) == 0) {
#pragma unroll
        for (int k = 0; k < S; ++k) {
          pv[0][k] = in[4][k];
          pv[1][k] = in[7][k];
          pv[2][k] = in[8][k];
        }
      } else {
#pragma unroll
        for (int k = 0; k < S; ++k) pv[0][k] = c[2][k];
        from_left(c[5], in[7], pv[1]);
        from_right(c[6], in[8], pv[2]);
      }
      constexpr int keep[6] = {0, 1, 3, 2, 5, 6};
#pragma unroll
      for (int j = 0; j < 6; ++j)
#pragma unroll
        for (int k = 0; k < S; ++k) c[keep[j]][k] = in[keep[j]][k];
      if (act) {
#pragma unroll
        for (int k = 0; k < S; ++k) {
          T g[9];
#pragma unroll
          for (int i = 0; i < 9; ++i) g[i] = f[i][k];
          bgk_collide<T, SHIFT>(g, omega);
#pragma unroll
          for (int i = 0; i < 9; ++i) in[i][k] = g[i];
        }
        if (s == K && st) {
          const unsigned o = (unsigned)(row * pitch + gx) * (unsigned)sizeof(T);
#pragma unroll
          for (int i = 0; i < 9; ++i) {
            char *pl = reinterpret_cast<char *>(dst + (size_t)i * P);
            if constexpr (S == 1) {
              __builtin_nontemporal_store(in[i][0], reinterpret_cast<T *>(pl + o));
            } else {
              VecT<T, S> t;
#pragma unroll
              for (int k = 0; k < S; ++k) t.v[k] = in[i][k];
              __builtin_memcpy(pl + o, &t, sizeof t);
            }
          }
        }
      }
    }
  }
}

template <typename T, bool SHIFT, int K, int S, int MON>
__global__ __launch_bounds__(64) void k_step_march(StepParams<T> p, int strips, int rows,
                                                   TbMonitor mon) {
  using G = MarchGeom<K, S>;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int strip = tile % strips, chunk = tile / strips;
  const int c0 = strip == 0 ? 0 : G::M + strip * G::TX;
  const int c1 = strip == strips - 1 ? p.nx : G::M + (strip + 1) * G::TX;
  const int X0 = max(0, min(strip * G::TX, p.nx - G::WW));
  const int y0 = chunk * rows, y1 = min(p.ny, y0 + rows);
  TbMonBlock mb{mon.uref, nullptr, nullptr, 0, nullptr};
  const bool wall = strip == 0 || strip == strips - 1 || y0 < K || y1 + K > p.ny;
  if (p.nx < G::WW)
    march_tile<T, SHIFT, K, S, MON, true, true>(p.src, p.dst, p.nx, p.ny, p.pitch, p.plane,
                                                p.omega, p.u6, X0, c0, c1, y0, y1, mb);
  else if (wall)
    march_tile<T, SHIFT, K, S, MON, true, false>(p.src, p.dst, p.nx, p.ny, p.pitch, p.plane,
                                                 p.omega, p.u6, X0, c0, c1, y0, y1, mb);
  else
    march_tile<T, SHIFT, K, S, MON, false, false>(p.src, p.dst, p.nx, p.ny, p.pitch, p.plane,
                                                  p.omega, p.u6, X0, c0, c1, y0, y1, mb);
}

}  // namespace lbm
