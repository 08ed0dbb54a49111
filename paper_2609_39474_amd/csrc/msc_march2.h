// Several lattice steps of the 2D explicit march (the source-free map of
// Sec. 4.1) in one launch.
//
// One explicit step moves 18 values per site for about 90 FP64 operations, so
// a march of single-step launches is bound by the launches and their load
// latency on small grids (3.2 us per step at N = 256 FP64) and by memory on
// large ones.  Here a block loads its tile with a halo of S sites, runs S
// steps on it in LDS, the part of the halo that is still exact shrinking by
// one ring per step, and stores the tile.  Neighbouring blocks repeat each
// other's halo collisions instead of exchanging them.
//
// In LDS the steps alternate by the AA pattern (see msc_aa.h): the even step
// works on a site's own slots, the odd step gathers from and scatters to
// slots that no other site touches, so each step needs one barrier and the
// tile one copy of the populations.  The first even step collides straight
// from global memory and the last odd step stores straight to it.  The
// collision is the sweep's own code: the result is bit-identical to S steps
// of the in-place march.
//
// Measured per step against the single-step launches: N = 256 FP64 3.19 ->
// 1.26 us (8 steps per launch), N = 2048 FP64 100 -> 45 us and FP32 44 -> 28 us
// (4 steps).  On large grids bound by the FP64 instructions of the collisions,
// 1.5-2.5 times the useful ones with the halo's; at N = 256 (one block per
// compute unit) by a step's chain of barrier, LDS reads (0.3 us of LDS traffic)
// and dependent sums.  At the operating point the kernel is an instantiation
// of its own without the population terms (POINT, 97 -> 62 instructions per
// site): 1.26 -> 1.17 us.
#pragma once

#include "msc_aa.h"

namespace msc {

template <class T>
struct March2Args {
  const T* in;   // 9 x NS populations
  T* out;        // the state S steps later (another buffer: neighbouring tiles read in)
  int Nx, Ny, lgy;
  int lgty;      // log2 of the tiles along y
  double wp, wm;
};

template <class T, bool POINT>
__device__ __forceinline__ void march2_collide(const March2Args<T>& A,
                                               const RawSite<D2Q9, T, typename CompT<T>::type, SW_EXPLICIT>& r,
                                               typename CompT<T>::type* C) {
  using CT = typename CompT<T>::type;
  SweepArgs<T, CT> S{};
  S.wp = A.wp;
  S.wm = A.wm;
  CT f[9];
  double hs[4];
  collide_raw<D2Q9, T, CT, SW_EXPLICIT, POINT>(S, r, f, C, hs);
}

// odd step number E (counted from 0, so S - 1 is the last) and, unless it is
// the last, the even step after it
template <class T, bool POINT, int BX, int BY, int S, int NT, int E>
__device__ __forceinline__ void march2_pair(const March2Args<T>& A, T (*f)[(BX + 2 * S) * (BY + 2 * S)], int x0,
                                            int y0) {
  using L = D2Q9;
  using CT = typename CompT<T>::type;
  constexpr int RX = BX + 2 * S, RY = BY + 2 * S;
  {
    constexpr int WX = RX - 2 * E, WY = RY - 2 * E;
    __syncthreads();
    for (int i = threadIdx.x; i < WX * WY; i += NT) {
      const int ix = E + i / WY, iy = E + i % WY;
      const int c = ix * RY + iy;
      RawSite<L, T, CT, SW_EXPLICIT> r;
#pragma unroll
      for (int k = 0; k < 9; ++k) r.f0[k] = f[L::opp(k)][c - L::cx(k) * RY - L::cy(k)];
      CT C[9];
      march2_collide<T, POINT>(A, r, C);
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        if constexpr (E < S - 1) {
          f[k][c + L::cx(k) * RY + L::cy(k)] = (T)C[k];
        } else {
          // tile coordinates of the destination
          const int jx = ix + L::cx(k) - S, jy = iy + L::cy(k) - S;
          if ((unsigned)jx < (unsigned)BX && (unsigned)jy < (unsigned)BY)
            A.out[(int64_t)k * A.Nx * A.Ny + (((x0 + jx) << A.lgy) | (y0 + jy))] = (T)C[k];
        }
      }
    }
  }
  if constexpr (E < S - 1) {
    constexpr int WX = RX - 2 * (E + 1), WY = RY - 2 * (E + 1);
    __syncthreads();
    for (int i = threadIdx.x; i < WX * WY; i += NT) {
      const int c = (E + 1 + i / WY) * RY + E + 1 + i % WY;
      RawSite<L, T, CT, SW_EXPLICIT> r;
#pragma unroll
      for (int k = 0; k < 9; ++k) r.f0[k] = f[k][c];
      CT C[9];
      march2_collide<T, POINT>(A, r, C);
#pragma unroll
      for (int k = 0; k < 9; ++k) f[L::opp(k)][c] = (T)C[k];
    }
    march2_pair<T, POINT, BX, BY, S, NT, E + 2>(A, f, x0, y0);
  }
}

template <class T, bool POINT, int BX, int BY, int S, int NT>
__global__ __launch_bounds__(NT) void k_march2(March2Args<T> A) {
  static_assert(S % 2 == 0, "pairs of steps");
  using L = D2Q9;
  using CT = typename CompT<T>::type;
  constexpr int RX = BX + 2 * S, RY = BY + 2 * S;
  __shared__ T f[9][RX * RY];
  const int item = xcd_item(blockIdx.x, gridDim.x);
  const int x0 = (item >> A.lgty) * BX, y0 = (item & ((1 << A.lgty) - 1)) * BY;
  const int64_t NS = (int64_t)A.Nx * A.Ny;
  for (int i = threadIdx.x; i < RX * RY; i += NT) {
    const int gx = (x0 - S + i / RY) & (A.Nx - 1), gy = (y0 - S + i % RY) & (A.Ny - 1);
    const int s = (gx << A.lgy) | gy;
    RawSite<L, T, CT, SW_EXPLICIT> r;
#pragma unroll
    for (int k = 0; k < 9; ++k) r.f0[k] = A.in[k * NS + s];
    CT C[9];
    march2_collide<T, POINT>(A, r, C);
#pragma unroll
    for (int k = 0; k < 9; ++k) f[L::opp(k)][i] = (T)C[k];
  }
  march2_pair<T, POINT, BX, BY, S, NT, 1>(A, f, x0, y0);
}

}  // namespace msc
