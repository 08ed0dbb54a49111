// Discrete adjoint of the dual-time march: the transpose of the unrolled
// computation of each physical step at its recorded inner count.  The step's
// inner iterates are recomputed from its checkpoint (kept in the storage
// precision) in FP64, and the adjoint runs in FP64, whatever the storage
// precision: the corrected iteration's transpose cancels terms amplified by
// the shadow solve (up to 1/a_q at low wavenumbers), so it is linearised at
// FP64 iterates.
//
// Stages (transposes of the forward stages):
//   sweep: push streaming transposes to a pull, mu_k(x) = lamT_k(x + c_k);
//     the TRT collision with source, Eq. (collision), transposes sitewise
//     through the even/odd projections, the derivatives of Eq. (feq) and Eq.
//     (source-distribution) in m and s, s = h - a m and
//     m = (P f + h/2)/(1 + a/2) (Eq. macro-reconstruct);
//   correction: f' = f_T + E Sh P (f_T - f) with Sh the shadow multiplier;
//     its transpose uses E^T, Sh^T = F^{-1}[chi H^{-H} F[.]] (same transform
//     kernels, conjugate-transposed Schur solve) and P^T;
//   acceptance m^{n+1} = (P f_T + h/2)/(1 + a/2), the rotation of the
//   histories, the BDF history term h_q (Eq. bdf2) and the trial
//   extrapolation.
#pragma once

#include "msc_fft.h"

namespace msc {

struct AdjGeom {
  int N0, N1, N2;
  int64_t NS;
};

__device__ __forceinline__ int64_t adj_neighbor(const AdjGeom& g, int64_t s, int cx, int c1, int c2) {
  const int p2 = (int)(s % g.N2);
  const int p1 = (int)((s / g.N2) % g.N1);
  const int x = (int)(s / ((int64_t)g.N1 * g.N2));
  return ((int64_t)wrapi(x + cx, g.N0) * g.N1 + wrapi(p1 + c1, g.N1)) * g.N2 + wrapi(p2 + c2, g.N2);
}

// One transposed sweep with what surrounds it at the same sites, so that each
// field passes once per launch.  With f the forward trial of sweep ell,
//   LF = carry + (dT/df)^T LT,   lam_h += (dT/dh)^T LT,
// where
//   f  = fin, or fin + E dm (Eq. lift) with dm the correction of sweep ell - 1;
//   LT = Lt + P^T zt, and the carry is 0, at the last sweep K of the step: the
//        seed, Lt and zt the adjoints of the new f^n and of m^{n+1} / (1 + a/2),
//        and lam_h starts at that of m^{n+1} / (2 + a);
//   LT = Lt + P^T zt and the carry is -P^T zt below it: Lt the LF of sweep
//        ell + 1 and zt = Sh^T E^T Lt its transposed correction;
//   LT = Lt without the shadow corrector.
// Above the first sweep LF is stored with y = E^T LF, the input of the
// transposed correction.  At the first sweep (last = 1) it is the adjoint of the
// trial, and the rotation of the histories, the trial's extrapolation and h_q
// (Eq. bdf2) are transposed in place: of0 .. om1 receive the adjoint of the old
// state (f^n, f^{n-1}, f^{n-2}, m^n, m^{n-1}).
struct AdjArgs {
  AdjGeom g;
  const double* fin;
  const double* dm;    // or null
  const double* h;
  const double* Lt;
  const double* zt;    // or null
  double zscale;       // zt times this
  int seed;
  double* LF;
  double* y;           // or null
  double* lam_h;
  double a, wp, wm;
  int last, order, q;
  double dt;
  const double* lf1n;  // adjoint of f^{n-1}' (= old f^n)
  const double* lf2n;  // adjoint of f^{n-2}' (= old f^{n-1})
  const double* lm1n;  // adjoint of m^{n-1}' (= old m^n)
  double* of0;
  double* of1;
  double* of2;
  double* om0;
  double* om1;
  // k_adj_rows: the spectra (Spec2, 2D band) of the correction of sweep ell - 1
  // and of the transposed correction of sweep ell + 1, solved, in place of dm
  // and zt; and of y, out
  const cpx<double>* dm_spec;
  const cpx<double>* z_spec;
  cpx<double>* y_spec;
  const cpx<double>* twy;
};

// The site's part: fs the trial, hs and lhs h and lam_h so far, mu the pulled LT
// (mu_k(x) = LT_k(x + c_k)), zz the scaled zt at the site.  Leaves y = E^T LF.
template <class L>
__device__ __forceinline__ void adj_site(const AdjArgs& A, int64_t x, const double* fs, const double* hs,
                                         const double* lhs, const double* mu, const double* zz, double* y) {
  constexpr int Q = L::Q, D = L::D;
  const double a = A.a, wp = A.wp, wm = A.wm;
  const double inv1pa2 = 1.0 / (1.0 + a / 2.0);  // as the forward sweep forms m
  const int64_t NS = A.g.NS;
  double M[4] = {0, 0, 0, 0}, m[4], s[4];
#pragma unroll
  for (int k = 0; k < Q; ++k) {
    M[0] += fs[k];
#pragma unroll
    for (int b = 0; b < D; ++b) M[1 + b] += (double)ca<L>(k, b) * fs[k];
  }
#pragma unroll
  for (int b = 0; b <= D; ++b) {
    m[b] = (M[b] + 0.5 * hs[b]) * inv1pa2;
    s[b] = hs[b] - a * m[b];
  }
  // gk = the even/odd projections' adjoint of feq, pk of Phi (Eq. collision);
  // feq and Phi in m and s (Eq. feq, source-distribution) with 1/cs2 = 3
  double lm[4] = {0, 0, 0, 0}, ls[4] = {0, 0, 0, 0};
#pragma unroll
  for (int k = 0; k < Q; ++k) {
    const double np = 0.5 * (mu[k] + mu[L::opp(k)]), nm = 0.5 * (mu[k] - mu[L::opp(k)]);
    const double wg = L::w(k) * (wp * np + wm * nm);
    const double wq = L::w(k) * ((1.0 - wp / 2.0) * np + (1.0 - wm / 2.0) * nm);
    double cu = 0.0, cs = 0.0;
#pragma unroll
    for (int b = 0; b < D; ++b) {
      cu += (double)ca<L>(k, b) * m[1 + b];
      cs += (double)ca<L>(k, b) * s[1 + b];
    }
    lm[0] += wg;
    ls[0] += wq;
#pragma unroll
    for (int b = 0; b < D; ++b) {
      const double c = (double)ca<L>(k, b);
      lm[1 + b] += (3.0 * (c - m[1 + b]) + 9.0 * cu * c) * wg;
      lm[1 + b] += (9.0 * c * cs - 3.0 * s[1 + b]) * wq;
      ls[1 + b] += (3.0 * (c - m[1 + b]) + 9.0 * cu * c) * wq;
    }
  }
  double lmt[4], lh[4], cz[4];
#pragma unroll
  for (int b = 0; b <= D; ++b) {
    lmt[b] = (lm[b] - a * ls[b]) * inv1pa2;
    lh[b] = (A.seed ? 0.5 * zz[b] : lhs[b]) + ls[b] + 0.5 * lmt[b];
  }
#pragma unroll
  for (int b = 0; b <= D; ++b) {
    y[b] = 0.0;
    cz[b] = A.seed ? 0.0 : zz[b];
  }
#pragma unroll
  for (int k = 0; k < Q; ++k) {
    const double np = 0.5 * (mu[k] + mu[L::opp(k)]), nm = 0.5 * (mu[k] - mu[L::opp(k)]);
    double v = lmt[0], c = cz[0];
#pragma unroll
    for (int b = 0; b < D; ++b) {
      v += (double)ca<L>(k, b) * lmt[1 + b];
      c += (double)ca<L>(k, b) * cz[1 + b];
    }
    const double l = (mu[k] - wp * np - wm * nm) - c + v;
    const int64_t i = (int64_t)k * NS + x;
    if (A.last) {
      double a0 = A.lf1n[i], a1 = A.lf2n[i], a2 = 0.0;
      if (A.order == 0) {
        a0 += l;
      } else if (A.order == 1) {
        a0 += 2.0 * l;
        a1 -= l;
      } else {
        a0 += 3.0 * l;
        a1 -= 3.0 * l;
        a2 += l;
      }
      A.of0[i] = a0;
      A.of1[i] = a1;
      A.of2[i] = a2;
    } else {
      A.LF[i] = l;
      y[0] += L::w(k) * l;
#pragma unroll
      for (int b = 0; b < D; ++b) y[1 + b] += 3.0 * L::w(k) * (double)ca<L>(k, b) * l;
    }
  }
#pragma unroll
  for (int b = 0; b <= D; ++b) {
    const int64_t i = b * NS + x;
    if (!A.last) {
      A.lam_h[i] = lh[b];
    } else if (A.q == 1) {
      A.om0[i] = A.lm1n[i] + lh[b] / A.dt;
      A.om1[i] = 0.0;
    } else {
      A.om0[i] = A.lm1n[i] + 4.0 * lh[b] / (2.0 * A.dt);
      A.om1[i] = -lh[b] / (2.0 * A.dt);
    }
  }
}

// f + E dm of one direction, as the sweep lifts (Eq. lift)
template <class L>
__device__ __forceinline__ double adj_lifted(int k, double f, const double* dmv) {
  double cu = 0.0;
#pragma unroll
  for (int b = 0; b < L::D; ++b) cu += (double)ca<L>(k, b) * dmv[1 + b];
  return f + L::w(k) * (dmv[0] + 3.0 * cu);
}

template <class L>
__global__ __launch_bounds__(256) void k_adj_sweep(AdjArgs A) {
  constexpr int Q = L::Q, D = L::D;
  const int64_t NS = A.g.NS;
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < NS; x += (int64_t)gridDim.x * blockDim.x) {
    double fs[Q], mu[Q], hs[4], lhs[4] = {0, 0, 0, 0}, dmv[4], zz[4] = {0, 0, 0, 0}, y[4];
#pragma unroll
    for (int b = 0; b <= D; ++b) {
      hs[b] = A.h[b * NS + x];
      if (!A.seed) lhs[b] = A.lam_h[b * NS + x];
      if (A.zt) zz[b] = A.zt[b * NS + x] * A.zscale;
    }
#pragma unroll
    for (int k = 0; k < Q; ++k) fs[k] = A.fin[(int64_t)k * NS + x];
    if (A.dm) {
#pragma unroll
      for (int b = 0; b <= D; ++b) dmv[b] = A.dm[b * NS + x];
#pragma unroll
      for (int k = 0; k < Q; ++k) fs[k] = adj_lifted<L>(k, fs[k], dmv);
    }
#pragma unroll
    for (int k = 0; k < Q; ++k) {
      const int64_t xn = adj_neighbor(A.g, x, L::cx(k), L::c1(k), L::c2(k));
      mu[k] = A.Lt[(int64_t)k * NS + xn];
      if (A.zt) {
        double z = A.zt[xn];
#pragma unroll
        for (int b = 0; b < D; ++b)
          if (ca<L>(k, b) != 0) z += (double)ca<L>(k, b) * A.zt[(1 + b) * NS + xn];
        mu[k] += z * A.zscale;
      }
    }
    adj_site<L>(A, x, fs, hs, lhs, mu, zz, y);
    if (A.y && !A.last) {
#pragma unroll
      for (int b = 0; b <= D; ++b) A.y[b * NS + x] = y[b];
    }
  }
}

// The same on a 2D grid whose rows fit a block (the sweep's own row
// transforms are on), one row per block: the rows of dm and of zt come from
// their solved band spectra (dm on this row, zt on it and its two neighbours,
// all lines at once), and y goes out as its row's band spectrum, so a
// transposed correction is one column pass between two of these.  Every block
// runs at once, so a launch takes one block's chain: the eight lines of the
// three transforms side by side, the site's loads issued before them (N = 256:
// 12.2 us, for 19 MB).
constexpr int adj_rows_threads(int T2) { return T2 >= 32 ? 2 * T2 : 64; }

template <int T2>
__global__ __launch_bounds__(adj_rows_threads(T2)) void k_adj_rows(AdjArgs A) {
  fetch_kernargs<sizeof(A)>();
  using L = D2Q9;
  constexpr int Q = L::Q, D = L::D, LG = ilog2c(T2);
  using F = LineFft<double, LG, 2>;
  // lines 0 .. 5: zt on rows x - 1, x, x + 1 (fields 0 and 1 packed, then 2);
  // 6, 7: dm on row x, and then y's row
  __shared__ cpx<double> buf[8 * T2];
  const int x0 = blockIdx.x, N0 = A.g.N0, tid = threadIdx.x;
  const int64_t NS = A.g.NS;
  const int NB = T2 / 4 + 1;
  const int64_t FS = Spec2<double>::field(N0, NB);
  const int t = tid & (F::TPL - 1);
  const int64_t x = (int64_t)x0 * T2 + tid;
  const bool site = tid < T2;
  // the site's own loads, in flight during the transforms
  double fs[Q], mu[Q], hs[4], lhs[4] = {0, 0, 0, 0}, zz[4] = {0, 0, 0, 0};
  if (site) {
#pragma unroll
    for (int k = 0; k < Q; ++k) {
      fs[k] = A.fin[(int64_t)k * NS + x];
      mu[k] = A.Lt[(int64_t)k * NS + (int64_t)((x0 + L::cx(k)) & (N0 - 1)) * T2 + ((tid + L::cy(k)) & (T2 - 1))];
    }
#pragma unroll
    for (int b = 0; b <= D; ++b) {
      hs[b] = A.h[b * NS + x];
      if (!A.seed) lhs[b] = A.lam_h[b * NS + x];
    }
  }
  cpx<double> w[F::NTW];
  F::load_tw(A.twy, t, w);
  const int line = tid / F::TPL;
  const cpx<double>* spec = line < 6 ? A.z_spec : A.dm_spec;
  if (line < 8 && spec) {
    const int xl = line < 6 ? (x0 - 1 + (line >> 1)) & (N0 - 1) : x0;
    cpx<double> v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      // element j of the conjugate-symmetric extension of the half band
      const int j = t + i * F::TPL, jj = j < NB ? j : T2 - j;
      v[i] = {0.0, 0.0};
      if (jj < NB) {
        const int64_t o = Spec2<double>::at(xl, jj, N0);
        cpx<double> a0 = spec[((line & 1) ? 2 * FS : 0) + o], a1 = {0.0, 0.0};
        if (!(line & 1)) a1 = spec[FS + o];
        const double sg = j == 0 ? 0.0 : (j < NB ? 1.0 : -1.0);
        v[i] = {a0.x - sg * a1.y, sg * a0.y + a1.x};
      }
    }
    cpx<double>* ln = buf + line * T2;
    F::template run<+1>(v, t, ln, ln, w);
#pragma unroll
    for (int i = 0; i < 4; ++i) ln[t + i * F::TPL] = v[i];
  }
  __syncthreads();
  double y[4] = {0, 0, 0, 0};
  if (site) {
    if (A.dm_spec) {
      const double dmv[3] = {buf[6 * T2 + tid].x, buf[6 * T2 + tid].y, buf[7 * T2 + tid].x};
#pragma unroll
      for (int k = 0; k < Q; ++k) fs[k] = adj_lifted<L>(k, fs[k], dmv);
    }
    if (A.z_spec) {
#pragma unroll
      for (int k = 0; k < Q; ++k) {
        const int yn = (tid + L::cy(k)) & (T2 - 1);
        const cpx<double>* ln = buf + 2 * (1 + L::cx(k)) * T2;
        mu[k] += ln[yn].x + (double)L::cx(k) * ln[yn].y + (double)L::cy(k) * ln[T2 + yn].x;
      }
      zz[0] = buf[2 * T2 + tid].x;
      zz[1] = buf[2 * T2 + tid].y;
      zz[2] = buf[3 * T2 + tid].x;
    } else if (A.zt) {
#pragma unroll
      for (int k = 0; k < Q; ++k) {
        const int64_t xn = (int64_t)((x0 + L::cx(k)) & (N0 - 1)) * T2 + ((tid + L::cy(k)) & (T2 - 1));
        mu[k] += (A.zt[xn] + (double)L::cx(k) * A.zt[NS + xn] + (double)L::cy(k) * A.zt[2 * NS + xn]) * A.zscale;
      }
#pragma unroll
      for (int b = 0; b <= D; ++b) zz[b] = A.zt[b * NS + x] * A.zscale;
    }
    adj_site<L>(A, x, fs, hs, lhs, mu, zz, y);
  }
  if (A.last || !A.y_spec) return;  // uniform
  cpx<double>* fbuf = buf + 6 * T2;
  if (site) {  // (lines 6 and 7: only this thread has read its dm)
    fbuf[tid] = {y[0], y[1]};
    fbuf[T2 + tid] = {y[2], 0.0};
  }
  __syncthreads();
  row_spectrum<T2>(A.y_spec, N0, NB, fbuf, tid, x0, w);
}

// Record of step n's start, enqueued behind its first sweep (and, like it, run
// only if the march gets there): the populations f^n, for a call's first
// records also the older ones, and the step's history term h, 16 bytes at a
// time.  Null targets are not copied.
template <class T>
struct CkptArgs {
  const DevCtl* ctl;
  int n;
  FBufs<T> fb;
  const double* h;
  uint4* rf[3];    // f^n, f^{n-1}, f^{n-2}
  uint4* rh;
  int64_t nf, nh;  // 16-byte words of one population and of h
};

template <class T>
__global__ __launch_bounds__(256) void k_checkpoint(CkptArgs<T> A) {
  if (!phase_ready(A.ctl->phase, A.n, 1)) return;
  const Roles& ro = A.ctl->roles[A.n & 1];
  const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    if (!A.rf[r]) continue;
    const uint4* src = reinterpret_cast<const uint4*>(A.fb.p[ro.slot_hist[r]]);
    for (int64_t i = i0; i < A.nf; i += stride) A.rf[r][i] = src[i];
  }
  const uint4* hs = reinterpret_cast<const uint4*>(A.h);
  for (int64_t i = i0; i < A.nh; i += stride) A.rh[i] = hs[i];
}

// Forward recompute helpers: the trial by extrapolation and h_q (Eq. bdf2),
// from checkpointed populations of type T into FP64 iterates.
template <class L, class T>
__global__ void k_adj_trial(int64_t NS, int order, const T* __restrict__ f0, const T* __restrict__ f1,
                            const T* __restrict__ f2, float sig, double* __restrict__ trial) {
  using CT = typename CompT<T>::type;
  constexpr int Q = L::Q;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; s < NS; s += stride) {
    CT a0[Q], a1[Q], a2[Q];
    site_load<L, T>(f0, NS, s, sig, a0);
    if (order >= 1) site_load<L, T>(f1, NS, s, sig, a1);
    if (order >= 2) site_load<L, T>(f2, NS, s, sig, a2);
#pragma unroll
    for (int k = 0; k < Q; ++k) {
      double v;
      if (order == 0)
        v = (double)a0[k];
      else if (order == 1)
        v = 2.0 * (double)a0[k] - (double)a1[k];
      else
        v = 3.0 * (double)a0[k] - 3.0 * (double)a1[k] + (double)a2[k];
      trial[(int64_t)k * NS + s] = v;
    }
  }
}

// Adjoint of the initial map: state (f0, f0, f0, P f0, P f0), f0 = feq(p0, u0).
template <class L>
__global__ void k_adj_init(int64_t NS, const double* __restrict__ p0, const double* __restrict__ u0,
                           const double* __restrict__ lam, double* __restrict__ lp, double* __restrict__ lu) {
  constexpr int Q = L::Q, D = L::D;
  const double cs2 = 1.0 / 3.0;
  const int64_t FQ = (int64_t)Q * NS, FM = (int64_t)(D + 1) * NS;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < NS; x += stride) {
    double m[4] = {p0[x], 0, 0, 0};
#pragma unroll
    for (int b = 0; b < D; ++b) m[1 + b] = u0[b * NS + x];
    double acc_p = 0.0, acc_u[3] = {0, 0, 0};
#pragma unroll
    for (int k = 0; k < Q; ++k) {
      double lk = lam[k * NS + x] + lam[FQ + k * NS + x] + lam[2 * FQ + k * NS + x];
      lk += lam[3 * FQ + x] + lam[3 * FQ + FM + x];
      double cu = 0.0;
#pragma unroll
      for (int b = 0; b < D; ++b) {
        lk += (double)ca<L>(k, b) * (lam[3 * FQ + (1 + b) * NS + x] + lam[3 * FQ + FM + (1 + b) * NS + x]);
        cu += (double)ca<L>(k, b) * m[1 + b];
      }
      acc_p += L::w(k) * lk;
#pragma unroll
      for (int b = 0; b < D; ++b) {
        const double c = (double)ca<L>(k, b);
        acc_u[b] += L::w(k) * (c / cs2 + cu * c / (cs2 * cs2) - m[1 + b] / cs2) * lk;
      }
    }
    lp[x] = acc_p;
#pragma unroll
    for (int b = 0; b < D; ++b) lu[b * NS + x] = acc_u[b];
  }
}

}  // namespace msc
