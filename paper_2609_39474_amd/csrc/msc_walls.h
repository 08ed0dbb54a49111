// Wall-bounded kinetic correction (paper Sec. 3.3, Algorithm 2) on the D2Q9
// lid-driven cavity: (I - L) df = r with L = B_Gamma S blkdiag(J^C(x))
// (Eq. wall-global-jacobian).  J^C(x) is the local collision Jacobian of Eq.
// (wall-local-jacobian) at a reference field (m, s): with G of Eq. (wall-G),
// J^C_kk' = (G_k0 + sum_a G_ka c_k'a) / (1 + a/2), i.e. (J^C z)_k =
// sum_b G_kb mu_b with mu = P z / (1 + a/2).  S streams with the periodic
// wrap, B_Gamma replaces the wall rows in the order of Eq. (bounceback-rows)
// (the lid constants have zero derivative).
//
// The paper factors I - L with a sparse direct solver.  Here it is solved by
// restarted GMRES, preconditioned on the right with M = I - L_0, L_0 the
// periodic map at rest.  At omega+- = 1, J^C at rest is g E P of rank three,
// g = (1 - a/2)/(1 + a/2), so M needs the moments only: with z the three
// fields that solve (I - g P Z(k) E) z^ = F[P v] at every wavevector,
//   M^{-1} v = v + g S E z,   P M^{-1} v = z,
// three transforms each way instead of nine and a 3 x 3 system that is real
// after scaling the velocities by i.  With the operator at rest L and L_0
// differ in the wall rows only, so
//   (I - L) M^{-1} v = v + (1 - B_Gamma) g S E z
// is v except at the wall nodes.
//
// One GMRES iteration is three launches, each with one block per row of the
// grid (or per column): k_wall_orth (Gram-Schmidt from the dot products'
// partial sums, the next basis vector, its moments' row transforms, the
// Hessenberg bookkeeping), k_wall_cols (column transforms and the solve) and
// k_wall_rows (inverse row transforms of the three planes around the row, the
// wall rows, the dot products with the basis).  They are latency-bound chains
// (N = 128: 20 us per iteration; 60 us as ten launches with nine-field
// transforms), so launches and passes count, not bytes.  Every sum has a fixed
// order.  Convergence is decided on the device: the launches after it return
// at once.
#pragma once

#include "msc_fullsym.h"

namespace msc {

// Eq. (wall-G) at omega+- = 1 for direction k (D2Q9): G[0] = dC_k/dp,
// G[1 + b] = dC_k/du_b at the reference moments m and source s.
__device__ inline void wall_G(int k, const double* m, const double* s, double a, double* G) {
  const double cs2 = 1.0 / 3.0, cs4 = cs2 * cs2;
  const double wk = D2Q9::w(k);
  const double c0 = (double)D2Q9::cx(k), c1 = (double)D2Q9::cy(k);
  const double cu = c0 * m[1] + c1 * m[2];
  G[0] = wk * (1.0 - 0.5 * a);
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const double cb = (b == 0) ? c0 : c1, ub = m[1 + b];
    double g = wk * (cb / cs2 + cu * cb / cs4 - ub / cs2);
    double src = 0.0;
#pragma unroll
    for (int al = 0; al < 2; ++al) {
      const double ca_ = (al == 0) ? c0 : c1;
      src += (-(al == b ? 1.0 : 0.0) / cs2 + ca_ * cb / cs4) * s[1 + al];
    }
    src -= a * ((cb - ub) / cs2 + cu * cb / cs4);
    G[1 + b] = g + 0.5 * wk * src;
  }
}

// Reference field of a refresh (Algorithm 2): the current iterate f = f_T - r
// reconstructed with the unchanged history term, m = (P f + h/2)/(1 + a/2),
// s = h - a m.
template <int UNUSED = 0>
__global__ __launch_bounds__(256) void k_wall_reference(const double* __restrict__ fT, const double* __restrict__ r,
                                                        const double* __restrict__ h, double a, int64_t NS,
                                                        double* __restrict__ mref, double* __restrict__ sref) {
  const double inv = 1.0 / (1.0 + 0.5 * a);
  for (int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; s < NS; s += (int64_t)gridDim.x * blockDim.x) {
    double M[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      const double f = fT[k * NS + s] - r[k * NS + s];
      M[0] += f;
      M[1] += (double)D2Q9::cx(k) * f;
      M[2] += (double)D2Q9::cy(k) * f;
    }
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const double m = (M[b] + 0.5 * h[b * NS + s]) * inv;
      mref[b * NS + s] = m;
      sref[b * NS + s] = h[b * NS + s] - a * m;
    }
  }
}

// ---------------------------------------------------------- one solve --
struct WallState {
  int done;  // launch index j of the k_wall_orth whose column converged or broke down, or 0
  int jend;  // the columns of the solution then
};

struct WallArgs {
  int Nx, Ny;          // rows of Ny sites
  int64_t NS;
  double a, g;         // a_A and (1 - a_A/2)/(1 + a_A/2)
  const double* mref;  // reference field of a re-linearised operator, or null at rest
  const double* sref;
  double* vc;          // FP64 copy of the newest basis vector; becomes w = (I - L) M^{-1} v
  cpx<double>* spec;   // three half spectra (Spec2, j_y <= N_y/2)
  const cpx<double>* twx;
  const cpx<double>* twy;
  double* part;        // dot-product partials: entry i of row x at part[i Nx + x]
  WallState* state;
  // Hessenberg bookkeeping of the cycle (m columns, row stride m)
  int m;
  double* Hd;
  double* cs;
  double* sn;
  double* gv;
  double stop;         // tolerance times the initial norm
};

// h[i] = the sum of the n <= 256 partials of entry i, i < nv, one wavefront
// per entry (each lane its strided partials, then a butterfly: a fixed order).
__device__ inline void wall_sums(const double* __restrict__ part, int n, int nv, double* h) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int i = wv; i < nv; i += (int)(blockDim.x >> 6)) {
    double x[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) x[q] = (lane + 64 * q < n) ? part[(int64_t)i * n + lane + 64 * q] : 0.0;
    double acc = ((x[0] + x[1]) + x[2]) + x[3];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (lane == 0) h[i] = acc;
  }
  __syncthreads();
}

constexpr int kWallGroup = 16;

// acc -/+= sum_k coef[k] V_k[t], k < G in order, with G fixed at compile time
// so that the G loads of element t issue together; the _n form dispatches a
// run-time group width g <= G.
template <int G, bool SUB, class VT>
__device__ inline double comb_rows(double acc, const VT* __restrict__ v, int64_t stride,
                                   const double* __restrict__ coef, int64_t t) {
  double x[G];
#pragma unroll
  for (int k = 0; k < G; ++k) x[k] = (double)v[k * stride + t];
#pragma unroll
  for (int k = 0; k < G; ++k) {
    if constexpr (SUB)
      acc -= coef[k] * x[k];
    else
      acc += coef[k] * x[k];
  }
  return acc;
}

template <int G, bool SUB, class VT>
__device__ inline double comb_rows_n(int g, double acc, const VT* __restrict__ v, int64_t stride,
                                     const double* __restrict__ coef, int64_t t) {
  if constexpr (G > 0) {
    if (g == G) return comb_rows<G, SUB, VT>(acc, v, stride, coef, t);
    return comb_rows_n<G - 1, SUB, VT>(g, acc, v, stride, coef, t);
  } else {
    return acc;
  }
}

template <bool SUB, class VT>
__device__ inline double comb_all(double acc, const VT* __restrict__ V, int64_t stride, int nv,
                                  const double* __restrict__ coef, int64_t t) {
  for (int i0 = 0; i0 < nv; i0 += kWallGroup) {
    const int g = (nv - i0 < kWallGroup) ? nv - i0 : kWallGroup;
    acc = comb_rows_n<kWallGroup, SUB, VT>(g, acc, V + (int64_t)i0 * stride, stride, coef + i0, t);
  }
  return acc;
}

// w -= sum_i coef[i] V_i (coef on the device), i < nv.
template <class VT>
__global__ __launch_bounds__(256) void k_axpy_multi(double* __restrict__ w, const VT* __restrict__ V, int64_t stride,
                                                    int nv, const double* __restrict__ coef, int64_t n) {
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x)
    w[t] = comb_all<true, VT>(w[t], V, stride, nv, coef, t);
}

// Threads of the row kernels: on rows of 512 twice as many wavefronts share the
// basis vectors (256 x 512, tolerance 1e-2: 96 -> 72 us per iteration, with the
// shorter loops of wall_row_dots).
constexpr int wall_threads(int lgy) { return lgy <= 8 ? 512 : 1024; }

// Lines along y: each in one wavefront (eight elements per thread at 512).
template <int LGY>
using WallLine = LineFft<double, LGY, line_le(LGY)>;

// Forward row transforms of P v for the row whose nine populations are in
// vrow (9 x T2): two packed lines, half spectrum j_y <= N_y/2.
template <int LGY>
__device__ __forceinline__ void wall_rows_fwd(const WallArgs& A, const double* vrow, cpx<double>* buf, int x) {
  constexpr int T2 = 1 << LGY;
  using F = WallLine<LGY>;
  static_assert(F::WAVE, "lines of at most 512");
  for (int y = threadIdx.x; y < T2; y += blockDim.x) {
    double M[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      const double f = vrow[k * T2 + y];
      M[0] += f;
      M[1] += (double)D2Q9::cx(k) * f;
      M[2] += (double)D2Q9::cy(k) * f;
    }
    buf[y] = {M[0], M[1]};
    buf[T2 + y] = {M[2], 0.0};
  }
  __syncthreads();
  if ((int)threadIdx.x >= 2 * F::TPL) return;
  const int line = threadIdx.x / F::TPL, t = threadIdx.x & (F::TPL - 1);
  cpx<double> w[F::NTW], v[F::E];
  F::load_tw(A.twy, t, w);
  cpx<double>* ln = buf + line * T2;
#pragma unroll
  for (int i = 0; i < F::E; ++i) v[i] = ln[t + i * F::TPL];
  wave_fence();
  F::template run<-1>(v, t, ln, ln, w);
#pragma unroll
  for (int i = 0; i < F::E; ++i) ln[t + i * F::TPL] = v[i];
  wave_fence();
  const int64_t FS = Spec2<double>::field(A.Nx, T2 / 2 + 1);
  auto store = [&](int j, cpx<double> z) {
    const int64_t o = Spec2<double>::at(x, j, A.Nx);
    if (line) {
      A.spec[2 * FS + o] = z;
      return;
    }
    const cpx<double> zc = ln[(T2 - j) & (T2 - 1)];
    A.spec[o] = {0.5 * (z.x + zc.x), 0.5 * (z.y - zc.y)};
    A.spec[FS + o] = {0.5 * (z.y + zc.y), 0.5 * (zc.x - z.x)};
  };
#pragma unroll
  for (int i = 0; i < F::E / 2; ++i) store(t + i * F::TPL, v[i]);
  if (t == 0) store(T2 / 2, v[F::E / 2]);
}

// z on the three rows x - 1, x, x + 1: line 2p holds z_0 + i z_1 of row
// x - 1 + p, line 2p + 1 z_2 (real part), by the block's first 6 TPL threads.
template <int LGY>
__device__ __forceinline__ void wall_rows_inv(const WallArgs& A, cpx<double>* buf, int x) {
  constexpr int T2 = 1 << LGY;
  using F = WallLine<LGY>;
  static_assert(F::WAVE, "lines of at most 512");
  const int line = threadIdx.x / F::TPL, t = threadIdx.x & (F::TPL - 1);
  if (line < 6) {
    cpx<double> w[F::NTW], v[F::E];
    F::load_tw(A.twy, t, w);
    const int64_t FS = Spec2<double>::field(A.Nx, T2 / 2 + 1);
    const int xl = (x - 1 + (line >> 1)) & (A.Nx - 1);
#pragma unroll
    for (int i = 0; i < F::E; ++i) {
      const int j = t + i * F::TPL;
      const bool lower = 2 * j <= T2, real_term = j == 0 || 2 * j == T2;
      const int64_t o = Spec2<double>::at(xl, lower ? j : T2 - j, A.Nx);
      cpx<double> a0 = A.spec[((line & 1) ? 2 * FS : 0) + o];
      cpx<double> a1 = (line & 1) ? cpx<double>{0.0, 0.0} : A.spec[FS + o];
      if (real_term) {
        a0.y = 0.0;
        a1.y = 0.0;
      } else if (!lower) {
        a0.y = -a0.y;
        a1.y = -a1.y;
      }
      v[i] = {a0.x - a1.y, a0.y + a1.x};
    }
    cpx<double>* ln = buf + line * T2;
    F::template run<+1>(v, t, ln, ln, w);
#pragma unroll
    for (int i = 0; i < F::E; ++i) ln[t + i * F::TPL] = v[i];
  }
  __syncthreads();
}

// g (S E z)_k at node (x, y) from the rows of wall_rows_inv: the streamed
// value of direction k comes from x - c_k.
template <int T2>
__device__ __forceinline__ void wall_stream(const cpx<double>* buf, double g, int y, double* v) {
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const cpx<double>* ln = buf + 2 * (1 - D2Q9::cx(k)) * T2;
    const int yu = (y - D2Q9::cy(k)) & (T2 - 1);
    const cpx<double> z = ln[yu];
    const double u2 = ln[T2 + yu].x;
    v[k] = g * D2Q9::w(k) * (z.x + 3.0 * ((double)D2Q9::cx(k) * z.y + (double)D2Q9::cy(k) * u2));
  }
}

// L u at node (x, y), u = M^{-1} v with z = P u in the rows of
// wall_rows_inv: the wall rows applied to the streamed J^C u.  gs: the
// streamed values of wall_stream (J^C at rest).
template <int T2>
__device__ __forceinline__ void wall_Lu(const WallArgs& A, const cpx<double>* buf, int x, int y, const double* gs,
                                        double* Lu) {
#pragma unroll
  for (int k = 0; k < 9; ++k) Lu[k] = gs[k];
  if (A.mref) {
    const double inv = 1.0 / (1.0 + 0.5 * A.a);
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      const int xu = (x - D2Q9::cx(k)) & (A.Nx - 1), yu = (y - D2Q9::cy(k)) & (T2 - 1);
      const int64_t su = (int64_t)xu * T2 + yu;
      double m[3], s[3], G[3];
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        m[b] = A.mref[b * A.NS + su];
        s[b] = A.sref[b * A.NS + su];
      }
      wall_G(k, m, s, A.a, G);
      const cpx<double>* ln = buf + 2 * (1 - D2Q9::cx(k)) * T2;
      const cpx<double> z = ln[yu];
      Lu[k] = (G[0] * z.x + G[1] * z.y + G[2] * ln[T2 + yu].x) * inv;
    }
  }
  cavity_rows<double>(Lu, x, y, A.Nx, T2, 0.0);
}

// The Gram-Schmidt step of column j - 1 and basis vector j (one block per row):
// h_i = <V_i, w> (i < j) and <w, w> from the partials, v_j = (w - sum h_i V_i)
// / |w - V h| into V_j and vc, and its rows' transforms.  One more block keeps
// the books, a serial chain as long as another block's whole work: column j - 1
// of the Hessenberg matrix (hcol + h, with hcol the first projection's
// coefficients where there were two), the earlier Givens rotations applied, a
// new one zeroes its last entry, g is rotated.  j = 0: v_0 = src scale0, and the
// cycle's books are opened with g_0 = 1 / scale0.
template <int LGY, class VT>
__global__ __launch_bounds__(wall_threads(LGY)) void k_wall_orth(WallArgs A, VT* V, int j, const double* hcol, const double* src,
                                                  double scale0) {
  fetch_kernargs<sizeof(A)>();
  constexpr int T2 = 1 << LGY;
  __shared__ double vrow[9 * T2];
  __shared__ cpx<double> buf[2 * T2];
  __shared__ double h[72], c_s[72], s_s[72];
  // (the launch that sets the flag goes on: its other blocks may read either)
  const int done = j > 0 ? A.state->done : 0;
  if (done && done < j) return;
  const int x = blockIdx.x;
  const int64_t n = 9 * A.NS;
  double scale = scale0;
  if (j > 0) {
    wall_sums(A.part, A.Nx, j + 1, h);
    double hh = 0.0;
    for (int i = 0; i < j; ++i) hh += h[i] * h[i];
    const double d = h[j] - hh;  // |w - V h|^2 = <w, w> - |h|^2
    const double hn = sqrt(d > 0.0 ? d : 0.0);
    scale = hn > 0.0 ? 1.0 / hn : 1.0;
    if (x == A.Nx) {
      const int c = j - 1;
      double* col = h;
      __syncthreads();  // every thread has summed h
      for (int i = threadIdx.x; i < c; i += blockDim.x) {
        c_s[i] = A.cs[i];
        s_s[i] = A.sn[i];
      }
      if (hcol)
        for (int i = threadIdx.x; i < j; i += blockDim.x) col[i] += hcol[i];
      __syncthreads();
      if (threadIdx.x == 0) {
        double cur = col[0];
        for (int i = 0; i < c; ++i) {
          const double nxt = col[i + 1];
          col[i] = c_s[i] * cur + s_s[i] * nxt;
          cur = -s_s[i] * cur + c_s[i] * nxt;
        }
        const double den = hypot(cur, hn);
        const double cj = den > 0.0 ? cur / den : 1.0, sj = den > 0.0 ? hn / den : 0.0;
        A.cs[c] = cj;
        A.sn[c] = sj;
        col[c] = den;
        const double gj = A.gv[c], res = fabs(sj * gj);
        A.gv[j] = -sj * gj;
        A.gv[c] = cj * gj;
        // converged with this column, or broken down in it
        if (!(den > 0.0) || !isfinite(res)) {
          A.state->jend = c;
          A.state->done = j;
        } else if (res <= A.stop) {
          A.state->jend = j;
          A.state->done = j;
        }
      }
      __syncthreads();
      for (int i = threadIdx.x; i < j; i += blockDim.x) A.Hd[(int64_t)i * A.m + c] = col[i];
    }
  } else if (x == A.Nx && threadIdx.x == 0) {
    A.state->done = 0;
    A.state->jend = 0;
    A.gv[0] = 1.0 / scale0;
  }
  if (x == A.Nx) return;
  for (int e = threadIdx.x; e < 9 * T2; e += blockDim.x) {
    const int64_t t = (int64_t)(e >> LGY) * A.NS + (int64_t)x * T2 + (e & (T2 - 1));
    double v;
    if (j > 0)
      v = comb_all<true, VT>(A.vc[t], V, n, j, h, t) * scale;
    else
      v = src[t] * scale;
    V[(int64_t)j * n + t] = (VT)v;
    A.vc[t] = v;
    vrow[e] = v;
  }
  __syncthreads();
  wall_rows_fwd<LGY>(A, vrow, buf, x);
}

// Column pass of M^{-1}: per retained j_y, forward along x, the 3 x 3 solve at
// every wavevector, inverse along x (1/N_sites folded in), in place.  With
// E, P and the streaming factors of D2Q9, P Z(k) E is built from the 1D sums
// A = 2/3 + cos(k)/3, B = -i sin(k)/3, C = cos(k)/3 per axis; dividing the
// velocity rows by i and multiplying its columns by i makes the matrix real.
// run_on: 0 within the iteration (nothing to do once converged), 1 at its end
// (only if converged), 2 always.
template <int LGX>
__global__ __launch_bounds__(256) void k_wall_cols(WallArgs A, int run_on) {
  fetch_kernargs<sizeof(A)>();
  constexpr int N = 1 << LGX;
  using F = LineFft<double, LGX, 2>;
  __shared__ cpx<double> lds[3 * N];
  if (run_on != 2 && (A.state->done != 0) != (run_on == 1)) return;
  const int NH = A.Ny / 2 + 1, jy = xcd_item(blockIdx.x, gridDim.x);
  if (jy >= NH) return;
  const int f = threadIdx.x / F::TPL, t = threadIdx.x & (F::TPL - 1);
  const int64_t FS = Spec2<double>::field(N, NH);
  cpx<double> w[F::NTW], v[4];
  cpx<double>* ln = lds + f * N;
  if (f < 3) {
    F::load_tw(A.twx, t, w);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = A.spec[f * FS + Spec2<double>::at(t + i * F::TPL, jy, N)];
    F::template run<-1>(v, t, ln, ln, w);
#pragma unroll
    for (int i = 0; i < 4; ++i) ln[t + i * F::TPL] = v[i];
  }
  __syncthreads();
  double sy, cy;
  sincospi(2.0 * jy / A.Ny, &sy, &cy);
  const double Ay = (2.0 + cy) / 3.0, by = sy / 3.0, Cy = cy / 3.0, ins = 1.0 / (double)A.NS;
  for (int jx = threadIdx.x; jx < N; jx += 256) {
    double sx, cx;
    sincospi(2.0 * signed_index(jx, N) / N, &sx, &cx);
    const double Ax = (2.0 + cx) / 3.0, bx = sx / 3.0, Cx = cx / 3.0, g = A.g;
    // rows p, x, y of the real system for (z_p, z_x / i, z_y / i)
    const double m00 = 1.0 - g * Ax * Ay, m01 = -3.0 * g * bx * Ay, m02 = -3.0 * g * Ax * by;
    const double m10 = g * bx * Ay, m11 = 1.0 - 3.0 * g * Cx * Ay, m12 = 3.0 * g * bx * by;
    const double m20 = g * Ax * by, m22 = 1.0 - 3.0 * g * Ax * Cy;
    const double c00 = m11 * m22 - m12 * m12, c01 = m12 * m20 - m10 * m22, c02 = m10 * m12 - m11 * m20;
    const double id = ins / (m00 * c00 + m01 * c01 + m02 * c02);
    const double c10 = m02 * m12 - m01 * m22, c11 = m00 * m22 - m02 * m20, c12 = m01 * m20 - m00 * m12;
    const double c20 = m01 * m12 - m02 * m11, c21 = m02 * m10 - m00 * m12, c22 = m00 * m11 - m01 * m10;
    const cpx<double> r0 = lds[jx], r1 = lds[N + jx], r2 = lds[2 * N + jx];
    // right side (r_p, r_x / i, r_y / i): 1/i (x + i y) = y - i x
    const double q0[2] = {r0.x, r0.y}, q1[2] = {r1.y, -r1.x}, q2[2] = {r2.y, -r2.x};
    double z[3][2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      z[0][e] = (c00 * q0[e] + c10 * q1[e] + c20 * q2[e]) * id;
      z[1][e] = (c01 * q0[e] + c11 * q1[e] + c21 * q2[e]) * id;
      z[2][e] = (c02 * q0[e] + c12 * q1[e] + c22 * q2[e]) * id;
    }
    lds[jx] = {z[0][0], z[0][1]};
    lds[N + jx] = {-z[1][1], z[1][0]};
    lds[2 * N + jx] = {-z[2][1], z[2][0]};
  }
  __syncthreads();
  if (f >= 3) return;
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = ln[t + i * F::TPL];
  wave_fence();
  F::template run<+1>(v, t, ln, ln, w);
#pragma unroll
  for (int i = 0; i < 4; ++i) A.spec[f * FS + Spec2<double>::at(t + i * F::TPL, jy, N)] = v[i];
}

// partials of <V_i, w>, i < nv, and of <w, w> (entry nv) over one row of w (9 x
// T2, in LDS): one wavefront per vector, up to 36 of its loads in flight per lane
// (18 on rows of 512, whose 72 at once spilled 107 registers).
template <int T2, class VT>
__device__ __forceinline__ void wall_row_dots(const WallArgs& A, const VT* V, int nv, const double* wrow, int x) {
  constexpr int PER = (9 * T2 + 63) / 64, CH = PER > 36 ? PER / 4 : PER;
  static_assert(PER % CH == 0 && CH <= 36, "rows of at most 512");
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int i = wv; i <= nv; i += (int)(blockDim.x >> 6)) {
    double acc = 0.0;
    const VT* v = V + (int64_t)i * 9 * A.NS + (int64_t)x * T2;
#pragma unroll 1
    for (int q0 = 0; q0 < PER; q0 += CH) {
#pragma unroll
      for (int q = 0; q < CH; ++q) {
        const int e = lane + 64 * (q0 + q);
        if (9 * T2 % 64 == 0 || e < 9 * T2) {
          const double we = wrow[e];
          acc += (i < nv ? (double)v[(int64_t)(e / T2) * A.NS + (e & (T2 - 1))] : we) * we;
        }
      }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (lane == 0) A.part[(int64_t)i * A.Nx + x] = acc;
  }
}

// w = (I - L) M^{-1} v_j on row x, in place of v_j in vc, and the partials of
// its dot products with V_0 .. V_j and itself.
template <int LGY, class VT>
__global__ __launch_bounds__(wall_threads(LGY)) void k_wall_rows(WallArgs A, const VT* V, int j) {
  fetch_kernargs<sizeof(A)>();
  constexpr int T2 = 1 << LGY;
  __shared__ cpx<double> buf[6 * T2];
  __shared__ double wrow[9 * T2];
  if (A.state->done) return;
  const int x = blockIdx.x;
  for (int e = threadIdx.x; e < 9 * T2; e += blockDim.x)
    wrow[e] = A.vc[(int64_t)(e >> LGY) * A.NS + (int64_t)x * T2 + (e & (T2 - 1))];
  wall_rows_inv<LGY>(A, buf, x);
  for (int y = threadIdx.x; y < T2; y += blockDim.x) {
    if (!A.mref && !(x == 0 || x == A.Nx - 1 || y == 0 || y == T2 - 1)) continue;
    double gs[9], Lu[9];
    wall_stream<T2>(buf, A.g, y, gs);
    wall_Lu<T2>(A, buf, x, y, gs, Lu);
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      const double wn = wrow[k * T2 + y] + gs[k] - Lu[k];
      wrow[k * T2 + y] = wn;
      A.vc[k * A.NS + (int64_t)x * T2 + y] = wn;
    }
  }
  __syncthreads();
  wall_row_dots<T2, VT>(A, V, j + 1, wrow, x);
}

// The dot products alone (after a first projection).
template <int LGY, class VT>
__global__ __launch_bounds__(wall_threads(LGY)) void k_wall_dots(WallArgs A, const VT* V, int j) {
  constexpr int T2 = 1 << LGY;
  __shared__ double wrow[9 * T2];
  const int x = blockIdx.x;
  for (int e = threadIdx.x; e < 9 * T2; e += blockDim.x)
    wrow[e] = A.vc[(int64_t)(e >> LGY) * A.NS + (int64_t)x * T2 + (e & (T2 - 1))];
  __syncthreads();
  wall_row_dots<T2, VT>(A, V, j + 1, wrow, x);
}

// The first projection's coefficients h = <V_i, w>, i < nv -> coef and hcol.
template <int UNUSED = 0>
__global__ __launch_bounds__(1024) void k_gs_first(const double* __restrict__ partials, int n, int nv,
                                                  double* __restrict__ coef, double* __restrict__ hcol) {
  __shared__ double h[72];
  wall_sums(partials, n, nv, h);
  for (int i = threadIdx.x; i < nv; i += blockDim.x) {
    coef[i] = h[i];
    hcol[i] = h[i];
  }
}

// The end of a cycle (one block per row): y = R^{-1} g of the jend columns
// (every block solves the small triangular system itself), Y = sum y_i V_i
// into vc, and its rows' transforms.  force: end after that many columns
// although the estimate has not converged (0: only if it has).
template <int LGY, class VT>
__global__ __launch_bounds__(512) void k_wall_combine(WallArgs A, const VT* V, int force) {
  constexpr int T2 = 1 << LGY;
  __shared__ double vrow[9 * T2];
  __shared__ cpx<double> buf[2 * T2];
  __shared__ double R[72 * 72 / 2 + 72], y[72];
  const int done = A.state->done;
  if (!done && !force) return;
  const int jend = done ? A.state->jend : force;
  const int x = blockIdx.x;
  const int64_t n = 9 * A.NS;
  // the upper triangle by columns: R(i, k) at k (k + 1) / 2 + i
  for (int e = threadIdx.x; e < jend * jend; e += blockDim.x) {
    const int i = e / jend, k = e - i * jend;
    if (i <= k) R[k * (k + 1) / 2 + i] = A.Hd[(int64_t)i * A.m + k];
  }
  for (int i = threadIdx.x; i < jend; i += blockDim.x) y[i] = A.gv[i];
  __syncthreads();
  if (threadIdx.x < 64) {
    // back substitution, column by column, the updates over the lanes
    const int lane = threadIdx.x;
    for (int k = jend - 1; k >= 0; --k) {
      const double yk = y[k] / R[k * (k + 1) / 2 + k];
      wave_fence();
      for (int i = lane; i <= k; i += 64) y[i] = (i == k) ? yk : y[i] - R[k * (k + 1) / 2 + i] * yk;
      wave_fence();
    }
  }
  __syncthreads();
  for (int e = threadIdx.x; e < 9 * T2; e += blockDim.x) {
    const int64_t t = (int64_t)(e >> LGY) * A.NS + (int64_t)x * T2 + (e & (T2 - 1));
    const double v = comb_all<false, VT>(0.0, V, n, jend, y, t);
    A.vc[t] = v;
    vrow[e] = v;
  }
  __syncthreads();
  wall_rows_fwd<LGY>(A, vrow, buf, x);
}

// u = M^{-1} Y is added to the correction delta (first cycle: delta = u), the
// residual R (first cycle: rhs) loses (I - L) u, and the partials of |R|^2 go to
// entry 0.  With fT the estimate's convergence also ends the solve: f_T <- f_T +
// (delta - rhs) = f + delta.
template <int LGY>
__global__ __launch_bounds__(512) void k_wall_finish(WallArgs A, const double* rhs, double* delta, double* R,
                                                    double* fT, int first, int force) {
  constexpr int T2 = 1 << LGY;
  __shared__ cpx<double> buf[6 * T2];
  __shared__ double red[8];
  const int done = A.state->done;
  if (!done && !force) return;
  const int x = blockIdx.x;
  wall_rows_inv<LGY>(A, buf, x);
  double r2 = 0.0;
  for (int y = threadIdx.x; y < T2; y += blockDim.x) {
    double gs[9], Lu[9];
    wall_stream<T2>(buf, A.g, y, gs);
    wall_Lu<T2>(A, buf, x, y, gs, Lu);
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      const int64_t t = k * A.NS + (int64_t)x * T2 + y;
      const double Y = A.vc[t], u = Y + gs[k], rh = rhs[t];
      const double d = first ? u : delta[t] + u;
      const double r = (first ? rh : R[t]) - (Y + (gs[k] - Lu[k]));
      delta[t] = d;
      R[t] = r;
      r2 += r * r;
      if (done && fT) fT[t] = fT[t] + (d - rh);
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) r2 += __shfl_xor(r2, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = r2;
  __syncthreads();
  if (threadIdx.x == 0) {
    double acc = 0.0;
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) acc += red[i];
    A.part[x] = acc;
  }
}

// f_T <- f_T + (delta - rhs), where the solve took more than one cycle.
template <int UNUSED = 0>
__global__ __launch_bounds__(256) void k_wall_update(double* fT, const double* delta, const double* rhs, int64_t n) {
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x)
    fT[t] = fT[t] + (delta[t] - rhs[t]);
}

}  // namespace msc
