// Stockham transforms of lines whose length is fixed at compile time, held in
// registers between stages.
//
// A line of N = 2^LG complex elements belongs to TPL = N / 2^LE consecutive
// threads; thread t holds the 2^LE elements t + i TPL.  Every stage of radix
// R <= 2^LE takes its butterflies' inputs and leaves its outputs in that
// distribution: the first stage needs no load from LDS, the last no store to
// it, and the stages between exchange once.  The transforms here are short
// chains that one or a few wavefronts run alone, so their time is instruction
// and LDS latency: with the length known, indices, strides and twiddle
// positions fold into constants, the first stage has no twiddles, and the
// twiddles of the others can be loaded before the data arrives.  One line of
// 256 alone takes 0.44 us in FP64 and 0.35 us in FP32, against 2.05 and 1.92
// us with a run-time length and every stage through LDS.
//
// Lines that fit one wavefront (TPL <= 64, TPL threads aligned inside a
// wavefront) need no barrier: LDS operations of a wavefront complete in order.
// Longer lines exchange through two buffers with one barrier per exchange, in
// which the whole block takes part.
#pragma once

#include <cmath>
#include <string>
#include <type_traits>
#include <vector>

#include "msc_cpx.h"
#include "msc_solver.h"

namespace msc {

template <class CT, int R, int ST, int SIGN>
__device__ __forceinline__ void reg_dft(cpx<CT>* a) {
#pragma clang fp contract(on)
  if constexpr (R == 2) {
    const cpx<CT> s = cadd(a[0], a[ST]), d = csub(a[0], a[ST]);
    a[0] = s;
    a[ST] = d;
  } else if constexpr (R == 4) {
    const cpx<CT> s02 = cadd(a[0], a[2 * ST]), d02 = csub(a[0], a[2 * ST]);
    const cpx<CT> s13 = cadd(a[ST], a[3 * ST]), d13 = cmuli(csub(a[ST], a[3 * ST]), SIGN);
    a[0] = cadd(s02, s13);
    a[ST] = cadd(d02, d13);
    a[2 * ST] = csub(s02, s13);
    a[3 * ST] = csub(d02, d13);
  } else {
    static_assert(R == 8, "radix 2, 4 or 8");
    // even outputs: the 4-point DFT of v_m + v_{m+4}; odd ones: that of
    // (v_m - v_{m+4}) e^(SIGN 2 pi i m / 8)
    cpx<CT> e[4], o[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      e[m] = cadd(a[m * ST], a[(m + 4) * ST]);
      o[m] = csub(a[m * ST], a[(m + 4) * ST]);
    }
    const CT r = (CT)0.70710678118654752440, sg = (CT)SIGN;
    o[1] = cpx<CT>{r * (o[1].x - sg * o[1].y), r * (o[1].y + sg * o[1].x)};
    o[2] = cmuli(o[2], SIGN);
    o[3] = cpx<CT>{r * (-o[3].x - sg * o[3].y), r * (-o[3].y + sg * o[3].x)};
    reg_dft<CT, 4, 1, SIGN>(e);
    reg_dft<CT, 4, 1, SIGN>(o);
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      a[2 * m * ST] = e[m];
      a[(2 * m + 1) * ST] = o[m];
    }
  }
}

// orders a wavefront's own LDS accesses (the hardware keeps them in order;
// this keeps the compiler from moving them)
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <class CT, int LG, int LE>
struct LineFft {
  static_assert(LG >= LE && LE >= 2 && LE <= 3, "radices up to 8, a line holds a thread's elements");
  static constexpr int N = 1 << LG, E = 1 << LE, TPL = N / E;
  static constexpr bool WAVE = TPL <= 64;
  static constexpr int NST = (LG + LE - 1) / LE;  // stages: radix E while it divides, then the rest
  static constexpr int NX = NST - 1;              // exchanges
  static constexpr int lr(int p) { return p < LG / LE ? LE : LG - (LG / LE) * LE; }
  static constexpr int tw_before(int p) {  // twiddles of the stages before p
    int n = 0;
    for (int q = 1; q < p; ++q) n += (E >> lr(q)) * ((1 << lr(q)) - 1);
    return n;
  }
  static constexpr int NTW = tw_before(NST) > 0 ? tw_before(NST) : 1;

  // Twiddles exp(-2 pi i m k / (R Ns)) of every stage, entry by entry with t
  // fastest, so that a wavefront's loads are contiguous: as gathers from the
  // table of the N roots they were 64 cache lines each and cost more than the
  // transform (no-op launches of the N = 1024 column pass 11.8 us).  This part
  // of an axis's table (twiddle_tables) starts at TW_AT.
  static constexpr int TW_AT = N + (LE == 3 ? LineFft<CT, LG, 2>::NTW * LineFft<CT, LG, 2>::TPL : 0);
  static void fill_tw(cpx<CT>* table) {
    for (int p = 1; p < NST; ++p) {
      const int R = 1 << lr(p), lns = p * LE, nb = E / R;
      for (int b = 0; b < nb; ++b)
        for (int m = 1; m < R; ++m)
          for (int t = 0; t < TPL; ++t) {
            const int k = (t + b * TPL) & ((1 << lns) - 1);
            table[TW_AT + (tw_before(p) + b * (R - 1) + m - 1) * TPL + t] = table[m * k * ((N / R) >> lns)];
          }
    }
  }
  // this thread's, from an axis's table
  static __device__ __forceinline__ void load_tw(const cpx<CT>* __restrict__ table, int t, cpx<CT>* w) {
    if constexpr (NST > 1) {
#pragma unroll
      for (int e = 0; e < NTW; ++e) w[e] = table[TW_AT + e * TPL + t];
    }
  }

  static __device__ __forceinline__ int slot(int i) {
    constexpr int G = 128 / (int)sizeof(cpx<CT>);
    return N >= G ? lds_swz<CT>(i) : i;
  }

  // in place: v[i] = x[t + i TPL] -> X[t + i TPL], SIGN = -1 forward, +1
  // inverse (no scaling).  a, b: the line's N elements of LDS for the even
  // and the odd exchanges (may be one and the same where WAVE).
  template <int SIGN, int P = 0>
  static __device__ __forceinline__ void run(cpx<CT>* v, int t, cpx<CT>* a, cpx<CT>* b, const cpx<CT>* w) {
#pragma clang fp contract(on)
    constexpr int R = 1 << lr(P), LNS = P * LE, NB = E / R;
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      if constexpr (P > 0) {
#pragma unroll
        for (int m = 1; m < R; ++m) {
          cpx<CT> x = w[tw_before(P) + q * (R - 1) + m - 1];
          if (SIGN > 0) x.y = -x.y;
          v[q + m * NB] = cmul(v[q + m * NB], x);
        }
      }
      reg_dft<CT, R, NB, SIGN>(v + q);
    }
    if constexpr (P + 1 < NST) {
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        const int j = t + q * TPL, k = j & ((1 << LNS) - 1);
        const int base = ((j - k) << lr(P)) + k;
#pragma unroll
        for (int m = 0; m < R; ++m) a[slot(base + (m << LNS))] = v[q + m * NB];
      }
      if constexpr (WAVE)
        wave_fence();
      else
        __syncthreads();
#pragma unroll
      for (int i = 0; i < E; ++i) v[i] = a[slot(t + i * TPL)];
      if constexpr (WAVE) wave_fence();
      run<SIGN, P + 1>(v, t, b, a, w);
    }
  }
};

// Element (x, j) of one field of the 2D band spectrum: groups of G columns (one
// 128-byte line), x inside a group, so the column pass, one column per block,
// reads consecutive lines that G neighbouring columns share.  (With j fastest
// over the whole band the column's elements lay N_y/4 + 1 apart, 8 x 256 + 8
// bytes at N = 1024 FP32, so that most of them met in two of an L2's 16
// channels.)
template <class CT>
struct Spec2 {
  static constexpr int G = 128 / (int)sizeof(cpx<CT>);
  static __host__ __device__ int64_t field(int Nx, int NB) { return (int64_t)((NB + G - 1) / G) * G * Nx; }
  static __device__ __forceinline__ int64_t at(int x, int j, int Nx) {
    return ((int64_t)(j / G) * Nx + x) * G + (j & (G - 1));
  }
};

constexpr int ilog2c(int n) { return n <= 1 ? 0 : 1 + ilog2c(n / 2); }

// log2 of the elements per thread where a few lines run alone (the 2D passes):
// radix 4 for short instruction chains while the threads last; N = 512 fits
// one wavefront with radix 8 (FP64 0.72 us against 0.86 with radix 4), N =
// 1024 does not (radix 4 on four wavefronts 1.27, radix 8 on two 1.83 us).
constexpr int line_le(int lg) { return (lg <= 8 || lg == 10) ? 2 : 3; }

// log2 of the longest lines that each family of passes is instantiated for, CT
// the transforms' real type.  The corrector's support tests and the launches
// both go by these, so that an extent that is accepted has its passes.
template <class CT>
struct LineMax {
  static constexpr int W = sizeof(CT) == 8 ? 1 : 0;
  static constexpr int rows2 = 12 - W, cols2 = 11 - W;     // 2D shadow passes (along y, along x)
  static constexpr int line3 = 11 - W;                     // 3D shadow passes (every axis)
  static constexpr int fs_rows = 10 - W, fs_cols = 9 - W;  // full symbol
  static constexpr int wall_rows = 9, wall_cols = 8;       // wall corrector (FP64)
};

// f(integral_constant<int, lg>) for LO <= lg <= HI; a length outside that range
// has no pass, which is an error of the caller's and no launch left out
template <int LO, int HI, class F>
void with_lg(int lg, F&& f) {
  if (lg == LO)
    f(std::integral_constant<int, LO>{});
  else if constexpr (LO < HI)
    with_lg<LO + 1, HI>(lg, f);
  else
    throw DeviceError{hipErrorInvalidValue, "no transform pass for lines of 2^" + std::to_string(lg) + " elements"};
}

// An axis's table on the host: the N roots exp(-2 pi i j / N), then the
// transforms' own order of them for four and for eight elements per thread.
template <class CT>
std::vector<cpx<CT>> twiddle_tables(int lg) {
  std::vector<cpx<CT>> table;
  with_lg<2, 12>(lg, [&](auto c) {
    constexpr int LG = c.value, N = 1 << LG;
    using F2 = LineFft<CT, LG, 2>;
    int size = F2::TW_AT + F2::NTW * F2::TPL;
    if constexpr (LG >= 3) size = LineFft<CT, LG, 3>::TW_AT + LineFft<CT, LG, 3>::NTW * LineFft<CT, LG, 3>::TPL;
    table.assign(size, cpx<CT>{0, 0});
    const double two_pi = 6.283185307179586476925286766559;
    for (int i = 0; i < N; ++i) {
      const double ang = -two_pi * (double)i / (double)N;
      table[i] = {(CT)std::cos(ang), (CT)std::sin(ang)};
    }
    F2::fill_tw(table.data());
    if constexpr (LG >= 3) LineFft<CT, LG, 3>::fill_tw(table.data());
  });
  return table;
}

}  // namespace msc
