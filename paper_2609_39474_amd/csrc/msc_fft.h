// Periodic macroscopic shadow correction (paper Sec. 3.2, Eq. shadow-update):
// dm = F^{-1}[ chi(k) H^{-1}(k) F[P r](k) ] with the transform convention of
// Eq. (fft-convention) (forward unnormalised, inverse 1/N_Omega), the signed
// wavenumbers of Eq. (wavenumbers) and the rectangular mask of Eq.
// (shadow-mask).  Only the masked band |j_alpha| <= N_alpha/4 is ever
// materialised: the residual moments are real, so the contiguous axis keeps
// j = 0..N/4 (the negative half follows by conjugate symmetry) and the other
// axes keep |j| <= N/4.
//
// Transforms are Stockham passes on complex lines (msc_linefft.h); the twiddle
// tables are precomputed per axis.  The per-wavevector
// 3x3 (2D) / 4x4 (3D) solve of Eq. (schur) runs in FP64 inside the kernel that
// holds the full spectrum line of the last axis.
#pragma once

#include "msc_kernels.h"
#include "msc_linefft.h"

namespace msc {


// Eq. (schur) at one wavevector, FP64.  r[0] = F[r_p], r[1..D] = F[r_m];
// out[0] = dp, out[1..D] = du, each scaled by `scale` (the 1/N_Omega of the
// inverse transform).
template <int D>
__device__ __forceinline__ void schur_solve(const double* kv, const double (*r)[2], double a, double nu,
                                            double scale, double (*out)[2]) {
  const double cs2 = 1.0 / 3.0;
  double kk = 0.0;
  for (int b = 0; b < D; ++b) kk += kv[b] * kv[b];
  const double bc = a + nu * kk;
  // k . r_m
  double kr_re = 0.0, kr_im = 0.0;
  for (int b = 0; b < D; ++b) {
    kr_re += kv[b] * r[1 + b][0];
    kr_im += kv[b] * r[1 + b][1];
  }
  // numerator r_p - i (k.r_m)/b ; -i*(x + iy) = y - ix.  Two divisions, the
  // other quotients by their reciprocals (one FP64 division is a chain of
  // about ten dependent operations)
  const double ib = 1.0 / bc, iden = 1.0 / (a + cs2 * kk * ib);
  const double num_re = r[0][0] + kr_im * ib;
  const double num_im = r[0][1] - kr_re * ib;
  const double dp_re = num_re * iden, dp_im = num_im * iden;
  out[0][0] = dp_re * scale;
  out[0][1] = dp_im * scale;
  for (int b = 0; b < D; ++b) {
    // (r_b - cs2 i k_b dp)/b ; i*dp = (-dp_im, dp_re)
    const double re = (r[1 + b][0] + cs2 * kv[b] * dp_im) * ib;
    const double im = (r[1 + b][1] - cs2 * kv[b] * dp_re) * ib;
    out[1 + b][0] = re * scale;
    out[1 + b][1] = im * scale;
  }
}

// Eq. (schur) conjugate-transposed, for the adjoint of the correction:
// solve H^H y = r, H^H = [[a, -i cs2 k^T], [-i k, b I]], b = a + nu |k|^2:
//   y_p = (r_p + i cs2 (k.r_u)/b) / (a + cs2 |k|^2 / b),  y_u = (r_u + i k y_p)/b.
template <int D>
__device__ __forceinline__ void schur_solve_adjoint(const double* kv, const double (*r)[2], double a, double nu,
                                                    double scale, double (*out)[2]) {
  const double cs2 = 1.0 / 3.0;
  double kk = 0.0;
  for (int b = 0; b < D; ++b) kk += kv[b] * kv[b];
  const double bc = a + nu * kk;
  double kr_re = 0.0, kr_im = 0.0;
  for (int b = 0; b < D; ++b) {
    kr_re += kv[b] * r[1 + b][0];
    kr_im += kv[b] * r[1 + b][1];
  }
  const double ib = 1.0 / bc, iden = 1.0 / (a + cs2 * kk * ib);
  const double yp_re = (r[0][0] - cs2 * kr_im * ib) * iden;
  const double yp_im = (r[0][1] + cs2 * kr_re * ib) * iden;
  out[0][0] = yp_re * scale;
  out[0][1] = yp_im * scale;
  for (int b = 0; b < D; ++b) {
    out[1 + b][0] = (r[1 + b][0] - kv[b] * yp_im) * ib * scale;
    out[1 + b][1] = (r[1 + b][1] + kv[b] * yp_re) * ib * scale;
  }
}

// Guard shared by the correction kernels: run only right after sweep ell of
// step n without acceptance (Algorithm 1 mode), or always (diagnostic mode).
struct CorrGuard {
  const DevCtl* ctl;
  int n, ell;
  __device__ bool skip() const { return ctl && !phase_correct(ctl->phase, n, ell); }
};

// ---------------------------------------------------------------- 2D ----
// Pass 1: forward transform along y (contiguous) of the three residual-moment
// rows of each x, keeping j_y = 0..N_y/4.  Rows (r_p, r_x) share one complex
// transform (real/imaginary packing); r_y takes a second one.
template <class CT, class TM>
struct Fft2Args {
  CorrGuard g;
  int do_accept;  // Algorithm 1 mode: the first pass decides acceptance (and reconstructs m^{n+1})
  int decide;     // the row pass ran inside the sweep: the column pass decides instead
  int adjoint;    // apply chi H^{-H} (transpose of the correction) instead of chi H^{-1}
  int Nx, Ny;
  int NBy;      // N_y/4 + 1
  const TM* Pr;            // 3 x Nx x Ny
  cpx<CT>* spec;           // 3 fields of the band (Spec2)
  TM* dm;                  // 3 x Nx x Ny
  const cpx<CT>* twx;      // Nx
  const cpx<CT>* twy;      // Ny
  double a, nu, inv_ns;
};

// Block shape of the row passes: 2 R lines of one block's R rows, R > 1 only
// where one row's two lines would not fill two wavefronts.
template <class CT, int LG>
struct RowsShape {
  using F = LineFft<CT, LG, line_le(LG)>;
  static constexpr int R = 2 * F::TPL >= 128 ? 1 : 128 / (2 * F::TPL);
  static constexpr int NT = 2 * R * F::TPL;
  static constexpr int LDS = 2 * R * F::N * (F::WAVE ? 1 : 2);
};

template <class L, class T, class CT, class TM, int LG>
__global__ __launch_bounds__((RowsShape<CT, LG>::NT)) void k_fft2_rows_fwd(Fft2Args<CT, TM> A, AcceptArgs<L, T> Ac,
                                                                         FinishArgs Fin) {
  fetch_kernargs<sizeof(A) + sizeof(Ac) + sizeof(Fin)>();
  using S = RowsShape<CT, LG>;
  using F = typename S::F;
  constexpr int N = F::N, E = F::E, TPL = F::TPL;
  __shared__ cpx<CT> lds[S::LDS];
  const int line = threadIdx.x / TPL, t = threadIdx.x & (TPL - 1);
  const int x = blockIdx.x * S::R + (line >> 1);
  cpx<CT> w[F::NTW];
  F::load_tw(A.twy, t, w);
  if (A.do_accept) {
    // Algorithm 1: decide on sweep ell of step n here; if accepted,
    // reconstruct m^{n+1} on this block's rows instead of transforming
    __shared__ double red[S::NT / 64];
    const int dec = finish_block(Fin, red);
    if (dec != DEC_RUNNING) {
      if (dec == DEC_ACCEPTED) {
        const int64_t s0 = (int64_t)blockIdx.x * S::R * N, s1 = s0 + (int64_t)S::R * N;
        accept_sites<L, T>(Ac, s0 + threadIdx.x, s1 < Ac.NS ? s1 : Ac.NS, blockDim.x);
      }
      return;
    }
  } else if (A.g.skip()) {
    return;
  }
  if (F::WAVE && x >= A.Nx) return;  // fewer rows than one block's
  const int64_t NS = (int64_t)A.Nx * N, s0 = (int64_t)x * N;
  cpx<CT> v[E];
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const int64_t s = s0 + t + i * TPL;
    v[i] = (line & 1) ? cpx<CT>{(CT)A.Pr[2 * NS + s], (CT)0} : cpx<CT>{(CT)A.Pr[s], (CT)A.Pr[NS + s]};
  }
  cpx<CT>* a = lds + line * N;
  cpx<CT>* b = F::WAVE ? a : a + S::LDS / 2;
  F::template run<-1>(v, t, a, b, w);
  cpx<CT>* nat = (F::NX & 1) ? b : a;
#pragma unroll
  for (int i = 0; i < E; ++i) nat[t + i * TPL] = v[i];
  if constexpr (F::WAVE)
    wave_fence();
  else
    __syncthreads();
  const int NB = A.NBy;
  const int64_t FS = Spec2<CT>::field(A.Nx, NB);
  auto store = [&](int j, cpx<CT> z) {
    if (line & 1) {
      A.spec[2 * FS + Spec2<CT>::at(x, j, A.Nx)] = z;
      return;
    }
    // unpack: F0 = (Z(j) + conj Z(-j))/2, F1 = (Z(j) - conj Z(-j))/(2i)
    const cpx<CT> zc = nat[(N - j) & (N - 1)];
    const int64_t o = Spec2<CT>::at(x, j, A.Nx);
    A.spec[o] = {(CT)0.5 * (z.x + zc.x), (CT)0.5 * (z.y - zc.y)};
    A.spec[FS + o] = {(CT)0.5 * (z.y + zc.y), (CT)0.5 * (zc.x - z.x)};
  };
#pragma unroll
  for (int i = 0; i < E / 4; ++i) store(t + i * TPL, v[i]);
  if (t == 0) store(N / 4, v[E / 4]);
}

// Pass 2: one retained j_y column per block, its three fields on TPL threads
// each: forward transform along x, the FP64 Schur solve on the band |j_x| <=
// N_x/4 (zero elsewhere), and the inverse transform along x, in place in the
// band spectrum array.  A few dozen to a few hundred blocks: the pass is one
// block's chain of load, transform, solve, transform, store, so a column is
// spread over as many threads as its stages can use.
template <class CT, int LG>
struct ColsShape {
  using F = LineFft<CT, LG, line_le(LG)>;
  static constexpr int NT = 3 * F::TPL > 256 ? 3 * F::TPL : 256;
  static constexpr int LDS = 3 * F::N * (F::WAVE ? 1 : 2);
};

template <class L, class T, class CT, class TM, int LG>
__global__ __launch_bounds__((ColsShape<CT, LG>::NT)) void k_fft2_cols_solve(Fft2Args<CT, TM> A, AcceptArgs<L, T> Ac,
                                                                           FinishArgs Fin) {
  fetch_kernargs<sizeof(A) + sizeof(Ac) + sizeof(Fin)>();
  using S = ColsShape<CT, LG>;
  using F = typename S::F;
  constexpr int N = F::N, E = F::E, TPL = F::TPL;
  static_assert(F::WAVE || S::NT == 3 * TPL, "every thread takes part in the barriers of long lines");
  __shared__ cpx<CT> lds[S::LDS];
  const int f = threadIdx.x / TPL, t = threadIdx.x & (TPL - 1);
  // XCD-aware column order (the grid is padded to a multiple of 8)
  const int NB = A.NBy, jy = xcd_item(blockIdx.x, gridDim.x);
  const int64_t FS = Spec2<CT>::field(N, NB);
  const bool mine = f < 3 && jy < NB;
  cpx<CT> w[F::NTW], v[E];
  F::load_tw(A.twx, t, w);
#pragma unroll
  for (int i = 0; i < E; ++i) v[i] = mine ? A.spec[f * FS + Spec2<CT>::at(t + i * TPL, jy, N)] : cpx<CT>{0, 0};
  // Algorithm 1 with the row pass fused into the sweep: the decision is taken
  // here, behind the forward transform that its loads then overlap
  FinishPre pre;
  if (A.decide)
    pre = finish_begin(Fin);
  else if (A.g.skip())
    return;
  cpx<CT>* a = lds + (f < 3 ? f : 0) * N;
  cpx<CT>* b = F::WAVE ? a : a + S::LDS / 2;
  if (f < 3) F::template run<-1>(v, t, a, b, w);
  // the band of the three spectra meets in LDS; wavevector q of the band is
  // j_x = q or q - (N/2 + 1) mod N
  cpx<CT>* s = (F::NX & 1) ? b : a;
  const cpx<CT>* base = (F::NX & 1) ? lds + S::LDS / 2 : lds;
  if (F::WAVE) base = lds;
  if (f < 3) {
#pragma unroll
    for (int i = 0; i < E; ++i)
      if (in_band(signed_index(t + i * TPL, N), N)) s[t + i * TPL] = v[i];
  }
  if (A.decide) {  // (its barrier serves the band too)
    __shared__ double red[S::NT / 64];
    const int dec = finish_end(Fin, pre, red);
    if (dec != DEC_RUNNING) {
      // if accepted, reconstruct m^{n+1} over the whole field instead
      if (dec == DEC_ACCEPTED)
        accept_sites<L, T>(Ac, (int64_t)blockIdx.x * blockDim.x + threadIdx.x, Ac.NS,
                           (int64_t)gridDim.x * blockDim.x);
      return;
    }
  } else {
    __syncthreads();
  }
  if (jy >= NB) return;  // grid padding
  const double two_pi = 6.283185307179586476925286766559;
  for (int q = threadIdx.x; q <= N / 2; q += S::NT) {
    const int jx = q <= N / 4 ? q : q + N / 2 - 1;
    const double kv[2] = {two_pi * signed_index(jx, N) / N, two_pi * jy / A.Ny};
    double r[3][2], o[3][2];
    cpx<CT>* c = const_cast<cpx<CT>*>(base) + jx;
#pragma unroll
    for (int g = 0; g < 3; ++g) {
      r[g][0] = (double)c[g * N].x;
      r[g][1] = (double)c[g * N].y;
    }
    if (A.adjoint)
      schur_solve_adjoint<2>(kv, r, A.a, A.nu, A.inv_ns, o);
    else
      schur_solve<2>(kv, r, A.a, A.nu, A.inv_ns, o);
#pragma unroll
    for (int g = 0; g < 3; ++g) c[g * N] = {(CT)o[g][0], (CT)o[g][1]};
  }
  __syncthreads();
  if (f >= 3) return;  // only where lines need no barrier
#pragma unroll
  for (int i = 0; i < E; ++i)
    v[i] = in_band(signed_index(t + i * TPL, N), N) ? s[t + i * TPL] : cpx<CT>{0, 0};
  if constexpr (F::WAVE)
    wave_fence();
  F::template run<+1>(v, t, (F::NX & 1) ? a : b, s, w);
#pragma unroll
  for (int i = 0; i < E; ++i) A.spec[f * FS + Spec2<CT>::at(t + i * TPL, jy, N)] = v[i];
}

// Pass 3: inverse transform along y from the half band to real rows.  The
// band of field f at x is extended by conjugate symmetry (Z(N - j) =
// conj Z(j)); fields 0 and 1 share one complex inverse transform (real and
// imaginary parts), field 2 uses the real part of a second one.
template <class CT, class TM, int LG>
__global__ __launch_bounds__((RowsShape<CT, LG>::NT)) void k_fft2_rows_inv(Fft2Args<CT, TM> A) {
  fetch_kernargs<sizeof(A)>();
  using S = RowsShape<CT, LG>;
  using F = typename S::F;
  constexpr int N = F::N, E = F::E, TPL = F::TPL;
  __shared__ cpx<CT> lds[S::LDS];
  const int line = threadIdx.x / TPL, t = threadIdx.x & (TPL - 1);
  const int x = blockIdx.x * S::R + (line >> 1);
  cpx<CT> w[F::NTW];
  F::load_tw(A.twy, t, w);
  if (A.g.skip()) return;
  if (F::WAVE && x >= A.Nx) return;
  const int NB = A.NBy;
  const int64_t FS = Spec2<CT>::field(A.Nx, NB);
  cpx<CT> v[E];
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const int j = t + i * TPL;
    const bool lower = j < NB;
    const int jj = lower ? j : N - j;
    v[i] = {0, 0};
    if (jj < NB) {
      const int64_t o = Spec2<CT>::at(x, jj, A.Nx);
      cpx<CT> a0 = A.spec[((line & 1) ? 2 * FS : 0) + o];
      cpx<CT> a1 = (line & 1) ? cpx<CT>{0, 0} : A.spec[FS + o];
      if (j == 0) {
        a0.y = 0;
        a1.y = 0;
      } else if (!lower) {
        a0.y = -a0.y;
        a1.y = -a1.y;
      }
      v[i] = {a0.x - a1.y, a0.y + a1.x};  // pack a0 + i a1
    }
  }
  cpx<CT>* a = lds + line * N;
  F::template run<+1>(v, t, a, F::WAVE ? a : a + S::LDS / 2, w);
  const int64_t NS = (int64_t)A.Nx * N, s0 = (int64_t)x * N;
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const int64_t s = s0 + t + i * TPL;
    if (line & 1) {
      A.dm[2 * NS + s] = (TM)v[i].x;
    } else {
      A.dm[s] = (TM)v[i].x;
      A.dm[NS + s] = (TM)v[i].y;
    }
  }
}

// ---------------------------------------------------------------- 3D ----
// Five passes over the band |j_alpha| <= N_alpha/4: forward along z (real
// input, keeps j_z = 0..N_z/4), forward along y (keeps the y band), along x
// with the FP64 4x4 Schur solve of Eq. (schur) between the forward and
// inverse transforms, inverse along y, inverse along z to real fields.  spec1
// holds the band after the z passes, spec2 after the y passes (Spec3).
template <class CT, class TM>
struct Fft3Args {
  CorrGuard g;
  int do_accept;
  int adjoint;
  int Nx, Ny, Nz;
  int NBz;  // N_z/4 + 1
  int NBy;  // 2 (N_y/4) + 1 retained y indices
  const TM* Pr;        // 4 x N_sites
  TM* dm;              // 4 x N_sites
  cpx<CT>* spec1;      // 4 fields, every y
  cpx<CT>* spec2;      // 4 fields, band of y
  const cpx<CT>* twx;
  const cpx<CT>* twy;
  const cpx<CT>* twz;
  double a, nu, inv_ns;
};

// The spectra keep groups of G = 64 bytes of neighbouring j_z together, with
// the axis that the y passes run along next: [field][x][j_z / G][y][j_z % G]
// and [field][j_z / G][x][band y][j_z % G].  A y line then reads consecutive
// 64-byte pieces, an x line pieces N_By apart.
template <class CT>
struct Spec3 {
  static constexpr int G = 64 / (int)sizeof(cpx<CT>);
  static __host__ __device__ int groups(int NBz) { return (NBz + G - 1) / G; }
  static __host__ __device__ int64_t field(int Nx, int Ny, int NBz) { return (int64_t)Nx * groups(NBz) * Ny * G; }
  static __device__ __forceinline__ int64_t at1(int x, int y, int j, int Ny, int NG) {
    return (((int64_t)x * NG + j / G) * Ny + y) * G + (j & (G - 1));
  }
  static __device__ __forceinline__ int64_t at2(int x, int by, int j, int Nx, int NBy) {
    return (((int64_t)(j / G) * Nx + x) * NBy + by) * G + (j & (G - 1));
  }
};

__device__ inline int band_to_j(int i, int N, int NB) { return (i <= N / 4) ? i : N - (NB - i); }

// log2 of the elements per thread in the 3D passes, which have thousands of
// lines: eight from N = 128 up (fewer exchanges per line)
constexpr int line_le3(int lg) { return lg <= 6 ? 2 : 3; }

// z passes: the two packed lines (fields 0, 1 and 2, 3) of PB pencils per block
template <class CT, int LG>
struct ZShape {
  using F = LineFft<CT, LG, line_le3(LG)>;
  static constexpr int NT = 2 * F::TPL > 256 ? 2 * F::TPL : 256;
  static constexpr int LPB = NT / F::TPL, PB = LPB / 2;
  static constexpr int LDS = LPB * F::N * (F::WAVE ? 1 : 2);
};

// y and x passes: CW neighbouring j_z columns of the four fields per block,
// one wavefront per field with the column fastest over its lanes (one column
// and more threads where a line is longer than a wavefront holds).  The lines
// of a wavefront are padded apart so that lanes of different columns use
// different banks.
template <class CT, int LG>
struct ColShape3 {
  using F = LineFft<CT, LG, line_le3(LG)>;
  static constexpr int CW = F::WAVE ? 64 / F::TPL : 1;
  static constexpr int FT = CW * F::TPL, NT = 4 * FT;
  static constexpr int PAD = CW == 1 ? 0 : (256 / (CW * (int)sizeof(cpx<CT>)) > 1 ? 256 / (CW * (int)sizeof(cpx<CT>)) : 1);
  static constexpr int PITCH = F::N + PAD;
  static constexpr int LDS = 4 * CW * PITCH * (F::WAVE ? 1 : 2);
};

// pass 1: forward along z.  The grid holds as many blocks as the device runs
// at once and each block loops over groups of pencils, so that the acceptance
// decision (a chain of dependent loads) is taken once per block rather than
// once per group.
template <class L, class T, class CT, class TM, int LG>
__global__ __launch_bounds__((ZShape<CT, LG>::NT)) void k_fft3_z_fwd(Fft3Args<CT, TM> A, AcceptArgs<L, T> Ac,
                                                                    FinishArgs Fin) {
  fetch_kernargs<sizeof(A) + sizeof(Ac) + sizeof(Fin)>();
  using S = ZShape<CT, LG>;
  using F = typename S::F;
  constexpr int N = F::N, E = F::E, TPL = F::TPL;
  __shared__ cpx<CT> lds[S::LDS];
  const int line = threadIdx.x / TPL, t = threadIdx.x & (TPL - 1), hf = line & 1;
  cpx<CT> w[F::NTW];
  F::load_tw(A.twz, t, w);
  if (A.do_accept) {
    __shared__ double red[S::NT / 64];
    const int dec = finish_block(Fin, red);
    if (dec != DEC_RUNNING) {
      if (dec == DEC_ACCEPTED)
        accept_sites<L, T>(Ac, (int64_t)blockIdx.x * blockDim.x + threadIdx.x, Ac.NS,
                           (int64_t)gridDim.x * blockDim.x);
      return;
    }
  } else if (A.g.skip()) {
    return;
  }
  const int NP = A.Nx * A.Ny, ngrp = (NP + S::PB - 1) / S::PB;
  const int64_t NS = (int64_t)NP * N;
  const int NB = A.NBz, NG = Spec3<CT>::groups(NB);
  const int64_t FS = Spec3<CT>::field(A.Nx, A.Ny, NB);
  cpx<CT>* a = lds + line * N;
  cpx<CT>* b = F::WAVE ? a : a + S::LDS / 2;
  cpx<CT>* nat = (F::NX & 1) ? b : a;
  for (int g = blockIdx.x; g < ngrp; g += gridDim.x) {
    const int p = g * S::PB + (line >> 1);
    if (F::WAVE && p >= NP) break;  // fewer pencils than one block's
    const TM* src = A.Pr + 2 * hf * NS + (int64_t)p * N;
    cpx<CT> v[E];
#pragma unroll
    for (int i = 0; i < E; ++i) v[i] = {(CT)src[t + i * TPL], (CT)src[NS + t + i * TPL]};
    F::template run<-1>(v, t, a, b, w);
#pragma unroll
    for (int i = 0; i < E; ++i) nat[t + i * TPL] = v[i];
    if constexpr (F::WAVE)
      wave_fence();
    else
      __syncthreads();
    const int x = p / A.Ny, y = p - x * A.Ny;
    auto store = [&](int j, cpx<CT> z) {
      const cpx<CT> zc = nat[(N - j) & (N - 1)];
      const int64_t o = 2 * hf * FS + Spec3<CT>::at1(x, y, j, A.Ny, NG);
      A.spec1[o] = {(CT)0.5 * (z.x + zc.x), (CT)0.5 * (z.y - zc.y)};
      A.spec1[FS + o] = {(CT)0.5 * (z.y + zc.y), (CT)0.5 * (zc.x - z.x)};
    };
#pragma unroll
    for (int i = 0; i < E / 4; ++i) store(t + i * TPL, v[i]);
    if (t == 0) store(N / 4, v[E / 4]);
    if constexpr (F::WAVE)
      wave_fence();
    else
      __syncthreads();  // the line's LDS is refilled by the next group
  }
}

// This thread's field, column and place in its line in a y or x pass.
template <class S>
struct Lane3 {
  int f, c, t;
  __device__ Lane3() {
    const int l = threadIdx.x % S::FT;
    f = threadIdx.x / S::FT;
    c = l % S::CW;
    t = l / S::CW;
  }
};

// pass 2: forward along y for a group of j_z columns at one x; keep the band
template <class CT, class TM, int LG>
__global__ __launch_bounds__((ColShape3<CT, LG>::NT)) void k_fft3_y_fwd(Fft3Args<CT, TM> A) {
  fetch_kernargs<sizeof(A)>();
  using S = ColShape3<CT, LG>;
  using F = typename S::F;
  constexpr int N = F::N, E = F::E, TPL = F::TPL;
  __shared__ cpx<CT> lds[S::LDS];
  const Lane3<S> l;
  cpx<CT> w[F::NTW], v[E];
  F::load_tw(A.twy, l.t, w);
  if (A.g.skip()) return;
  const int NBz = A.NBz, NG = Spec3<CT>::groups(NBz), nc = (NBz + S::CW - 1) / S::CW;
  const int item = xcd_item(blockIdx.x, gridDim.x);
  if (item >= A.Nx * nc) return;  // grid padding
  const int x = item / nc, j = (item % nc) * S::CW + l.c;
  const int64_t FS1 = Spec3<CT>::field(A.Nx, N, NBz), FS2 = Spec3<CT>::field(A.Nx, A.NBy, NBz);
#pragma unroll
  for (int i = 0; i < E; ++i)
    v[i] = (j < NBz) ? A.spec1[l.f * FS1 + Spec3<CT>::at1(x, l.t + i * TPL, j, N, NG)] : cpx<CT>{0, 0};
  cpx<CT>* a = lds + (l.f * S::CW + l.c) * S::PITCH;
  F::template run<-1>(v, l.t, a, F::WAVE ? a : a + S::LDS / 2, w);
  if (j >= NBz) return;
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const int jy = l.t + i * TPL;
    const int by = (jy <= N / 4) ? jy : ((N - jy <= N / 4) ? A.NBy - (N - jy) : -1);
    if (by >= 0) A.spec2[l.f * FS2 + Spec3<CT>::at2(x, by, j, A.Nx, A.NBy)] = v[i];
  }
}

// pass 3: along x for a group of j_z columns at one band-y index: forward,
// FP64 Schur solve on |j_x| <= N_x/4 (zero elsewhere), inverse; in place
template <class CT, class TM, int LG>
__global__ __launch_bounds__((ColShape3<CT, LG>::NT)) void k_fft3_x_solve(Fft3Args<CT, TM> A) {
  fetch_kernargs<sizeof(A)>();
  using S = ColShape3<CT, LG>;
  using F = typename S::F;
  constexpr int N = F::N, E = F::E, TPL = F::TPL, CW = S::CW;
  __shared__ cpx<CT> lds[S::LDS];
  const Lane3<S> l;
  cpx<CT> w[F::NTW], v[E];
  F::load_tw(A.twx, l.t, w);
  if (A.g.skip()) return;
  const int NBz = A.NBz, NBy = A.NBy, nc = (NBz + CW - 1) / CW;
  const int item = xcd_item(blockIdx.x, gridDim.x);
  if (item >= NBy * nc) return;  // grid padding
  const int by = item / nc, j0 = (item % nc) * CW, j = j0 + l.c;
  const int64_t FS2 = Spec3<CT>::field(N, NBy, NBz);
#pragma unroll
  for (int i = 0; i < E; ++i)
    v[i] = (j < NBz) ? A.spec2[l.f * FS2 + Spec3<CT>::at2(l.t + i * TPL, by, j, N, NBy)] : cpx<CT>{0, 0};
  cpx<CT>* a = lds + (l.f * CW + l.c) * S::PITCH;
  cpx<CT>* b = F::WAVE ? a : a + S::LDS / 2;
  F::template run<-1>(v, l.t, a, b, w);
  // the band of the four spectra meets in LDS (see the 2D column pass)
  cpx<CT>* s = (F::NX & 1) ? b : a;
  cpx<CT>* base = lds + ((!F::WAVE && (F::NX & 1)) ? S::LDS / 2 : 0);
#pragma unroll
  for (int i = 0; i < E; ++i)
    if (in_band(signed_index(l.t + i * TPL, N), N)) s[l.t + i * TPL] = v[i];
  __syncthreads();
  const double two_pi = 6.283185307179586476925286766559;
  const int sjy = signed_index(band_to_j(by, A.Ny, NBy), A.Ny);
  for (int i = threadIdx.x; i < CW * (N / 2 + 1); i += S::NT) {
    const int c = i % CW, q = i / CW;
    if (j0 + c >= NBz) continue;
    const int jx = q <= N / 4 ? q : q + N / 2 - 1;
    const double kv[3] = {two_pi * signed_index(jx, N) / N, two_pi * sjy / A.Ny, two_pi * (j0 + c) / A.Nz};
    double r[4][2], o[4][2];
    cpx<CT>* e = base + c * S::PITCH + jx;
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      r[f][0] = (double)e[f * CW * S::PITCH].x;
      r[f][1] = (double)e[f * CW * S::PITCH].y;
    }
    if (A.adjoint)
      schur_solve_adjoint<3>(kv, r, A.a, A.nu, A.inv_ns, o);
    else
      schur_solve<3>(kv, r, A.a, A.nu, A.inv_ns, o);
#pragma unroll
    for (int f = 0; f < 4; ++f) e[f * CW * S::PITCH] = {(CT)o[f][0], (CT)o[f][1]};
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < E; ++i)
    v[i] = in_band(signed_index(l.t + i * TPL, N), N) ? s[l.t + i * TPL] : cpx<CT>{0, 0};
  if constexpr (F::WAVE) wave_fence();
  F::template run<+1>(v, l.t, (F::NX & 1) ? a : b, s, w);
  if (j >= NBz) return;
#pragma unroll
  for (int i = 0; i < E; ++i) A.spec2[l.f * FS2 + Spec3<CT>::at2(l.t + i * TPL, by, j, N, NBy)] = v[i];
}

// pass 4: inverse along y from the band to every y, for a group of j_z at x
template <class CT, class TM, int LG>
__global__ __launch_bounds__((ColShape3<CT, LG>::NT)) void k_fft3_y_inv(Fft3Args<CT, TM> A) {
  fetch_kernargs<sizeof(A)>();
  using S = ColShape3<CT, LG>;
  using F = typename S::F;
  constexpr int N = F::N, E = F::E, TPL = F::TPL;
  __shared__ cpx<CT> lds[S::LDS];
  const Lane3<S> l;
  cpx<CT> w[F::NTW], v[E];
  F::load_tw(A.twy, l.t, w);
  if (A.g.skip()) return;
  const int NBz = A.NBz, NG = Spec3<CT>::groups(NBz), nc = (NBz + S::CW - 1) / S::CW;
  const int item = xcd_item(blockIdx.x, gridDim.x);
  if (item >= A.Nx * nc) return;  // grid padding
  const int x = item / nc, j = (item % nc) * S::CW + l.c;
  const int64_t FS1 = Spec3<CT>::field(A.Nx, N, NBz), FS2 = Spec3<CT>::field(A.Nx, A.NBy, NBz);
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const int jy = l.t + i * TPL;
    const int by = (jy <= N / 4) ? jy : ((N - jy <= N / 4) ? A.NBy - (N - jy) : -1);
    v[i] = (j < NBz && by >= 0) ? A.spec2[l.f * FS2 + Spec3<CT>::at2(x, by, j, A.Nx, A.NBy)] : cpx<CT>{0, 0};
  }
  cpx<CT>* a = lds + (l.f * S::CW + l.c) * S::PITCH;
  F::template run<+1>(v, l.t, a, F::WAVE ? a : a + S::LDS / 2, w);
  if (j >= NBz) return;
#pragma unroll
  for (int i = 0; i < E; ++i) A.spec1[l.f * FS1 + Spec3<CT>::at1(x, l.t + i * TPL, j, N, NG)] = v[i];
}

// pass 5: inverse along z from j_z = 0..N_z/4 (conjugate-symmetric
// extension, real part at j_z = 0) to real fields; (0,1) and (2,3) packed
template <class CT, class TM, int LG>
__global__ __launch_bounds__((ZShape<CT, LG>::NT)) void k_fft3_z_inv(Fft3Args<CT, TM> A) {
  fetch_kernargs<sizeof(A)>();
  using S = ZShape<CT, LG>;
  using F = typename S::F;
  constexpr int N = F::N, E = F::E, TPL = F::TPL;
  __shared__ cpx<CT> lds[S::LDS];
  const int line = threadIdx.x / TPL, t = threadIdx.x & (TPL - 1), hf = line & 1;
  cpx<CT> w[F::NTW], v[E];
  F::load_tw(A.twz, t, w);
  if (A.g.skip()) return;
  const int NP = A.Nx * A.Ny, p = blockIdx.x * S::PB + (line >> 1);
  if (F::WAVE && p >= NP) return;
  const int64_t NS = (int64_t)NP * N;
  const int NB = A.NBz, NG = Spec3<CT>::groups(NB);
  const int64_t FS = Spec3<CT>::field(A.Nx, A.Ny, NB);
  const int x = p / A.Ny, y = p - x * A.Ny;
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const int j = t + i * TPL;
    const bool lower = j < NB;
    const int jj = lower ? j : N - j;
    v[i] = {0, 0};
    if (jj < NB) {
      const int64_t o = 2 * hf * FS + Spec3<CT>::at1(x, y, jj, A.Ny, NG);
      cpx<CT> a0 = A.spec1[o], a1 = A.spec1[FS + o];
      if (j == 0) {
        a0.y = 0;
        a1.y = 0;
      } else if (!lower) {
        a0.y = -a0.y;
        a1.y = -a1.y;
      }
      v[i] = {a0.x - a1.y, a0.y + a1.x};  // pack a0 + i a1
    }
  }
  cpx<CT>* a = lds + line * N;
  F::template run<+1>(v, t, a, F::WAVE ? a : a + S::LDS / 2, w);
  TM* dst = A.dm + 2 * hf * NS + (int64_t)p * N;
#pragma unroll
  for (int i = 0; i < E; ++i) {
    dst[t + i * TPL] = (TM)v[i].x;
    dst[NS + t + i * TPL] = (TM)v[i].y;
  }
}

}  // namespace msc
