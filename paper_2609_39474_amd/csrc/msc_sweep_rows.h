// The fused sweep (see msc_sweep.h) on a 2D grid whose rows fit one tile, with
// one destination plane per block: the three source rows of a destination row
// in parallel, one group of T2 threads each, instead of one after the other.
//
// On these grids (N_y <= 256, at most 512 rows) every block runs at once, so
// the sweep takes as long as one block's chain of dependent work.  k_sweep's
// chain is three plane steps of load, collision and barrier; here it is one.
// The groups push their post-collision values to one array in LDS, and the
// middle group, which holds the trial populations of the destination row,
// finalises it.  The arithmetic is k_sweep's, so populations and P r are
// bit-identical to it.
//
// A step's first sweep can take the decision on the step before it along (rows
// of at least 64 sites): its loads, from the buffers that an acceptance leaves
// f^n and the histories in, and the fold of the residual run side by side, and
// the march saves the launch that only decides
// (N = 256 FP32: 25.5 -> 23.8 us per step)
//
// The lift mode inverts the band spectrum rows of the three source planes
// before the collision (six lines at once), and with fuse_rows the block
// transforms its row of P r forward.
#pragma once

#include "msc_sweep.h"

namespace msc {

// sqrt(sum of the grid's partials * inv_count) by the last block to get here, in
// a fixed order.  Thread 0 of each block has written its partial.
template <int NT>
__device__ __forceinline__ void rows_rms(const double* partials, double* rms, unsigned* arrived, unsigned before,
                                         double inv_count) {
  __shared__ double sum[NT];
  __shared__ int last;
  const int tid = threadIdx.x, n = gridDim.x;
  if (tid == 0)
    last = __hip_atomic_fetch_add(arrived, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) - before == (unsigned)n - 1;
  __syncthreads();
  if (!last) return;  // uniform
  double acc = 0.0;
  for (int i = tid; i < n; i += NT)
    acc += __hip_atomic_load(&partials[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if constexpr (NT % 64 == 0) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  }
  sum[tid] = acc;
  __syncthreads();
  if (tid == 0) {
    constexpr int STEP = NT % 64 == 0 ? 64 : 1;
    double tot = 0.0;
    for (int i = 0; i < NT; i += STEP) tot += sum[i];
    *rms = sqrt(tot * inv_count);
  }
}

template <class T, class TM, int T2, int MODE>
__global__ __launch_bounds__(3 * T2) void k_sweep_rows(SweepArgs<T, TM> A) {
  fetch_kernargs<sizeof(A)>();
  using L = D2Q9;
  using CT = typename CompT<T>::type;
  using LT = typename std::conditional<PopDev<T>::value, float, T>::type;
  constexpr int Q = L::Q, D = L::D;
  constexpr bool DV = PopDev<T>::value;
  constexpr bool ROWINV = (MODE == SW_DTS_LIFT_ROWS);
  constexpr bool DUAL = (MODE != SW_EXPLICIT);
  constexpr int NRED = T2 < 64 ? T2 : T2 / 64;
  constexpr int LG = ilog2c(T2);
  __shared__ LT val[Q][T2];  // post-collision values by destination
  __shared__ cpx<CT> fbuf[DUAL ? 2 * T2 : 1];  // the row of P r, then its spectrum
  __shared__ cpx<CT> ibuf[ROWINV ? 6 * T2 : 1];
  __shared__ double red[NRED];

  SrcPtrs<T> P{A.src, nullptr, nullptr, nullptr, nullptr, nullptr};
  T* __restrict__ dst = A.dst;
  constexpr bool MERGE = setup_mode(MODE) && T2 >= 64;  // whole wavefronts, for the fold
  FinishPre pre;
  bool pending = false;
  if (A.ctl) {
    if (MERGE && A.merge) {
      pre = finish_begin(A.fin);
      if (!merged_sources(A, P, dst, pending)) return;
    } else if (!sweep_sources<MODE>(A, P, dst)) {
      return;
    }
  }
  if (!pending && A.did_run && blockIdx.x == 0 && threadIdx.x == 0) *A.did_run = 1;

  const int N0 = A.N0;
  const int64_t NS = A.NS;
  const int x0 = xcd_item(blockIdx.x, gridDim.x);  // adjacent rows on one XCD
  const int tid = threadIdx.x;
  const int pl = tid / T2, y = tid & (T2 - 1);  // source plane x0 - 1 + pl
  const int xs = (x0 - 1 + pl) & (N0 - 1);
  const int64_t site = (int64_t)xs * T2 + y;
  RawSite<L, T, TM, MODE> raw;
  load_raw<L, T, TM, MODE>(A, P, site, raw);
  if constexpr (MERGE) {
    // (nothing has been written yet)
    __shared__ double fold[3 * T2 / 64];
    if (pending) {
      if (finish_end(A.fin, pre, fold) != DEC_ACCEPTED) return;
      if (A.did_run && blockIdx.x == 0 && threadIdx.x == 0) *A.did_run = 1;
    }
  }
  using F = LineFft<CT, LG, 2>;
  cpx<CT> tw[F::NTW];
  // (the table is there only for sweeps that transform rows)
  if (DUAL && A.fuse_rows && tid < (ROWINV ? 6 : 2) * F::TPL) F::load_tw(A.twr, tid & (F::TPL - 1), tw);
  if constexpr (ROWINV) {
    // inverse transform along y of the band spectrum rows of the three source
    // planes (the conjugate-symmetric extension of each field's half band,
    // fields 0 and 1 packed in line 2p of plane p, field 2 in line 2p + 1)
    const int line = tid / F::TPL, t = tid & (F::TPL - 1);
    if (line < 6) {
      const int NB = A.NBr;
      const int64_t FS = Spec2<CT>::field(N0, NB);
      const int xl = (x0 - 1 + (line >> 1)) & (N0 - 1);
      // element j of the line, j <= N_y/4
      auto elem = [&](int j) -> cpx<CT> {
        const int64_t o = Spec2<CT>::at(xl, j, N0);
        if (line & 1) {
          const cpx<CT> a2 = A.spec_in[2 * FS + o];
          return {a2.x, j == 0 ? (CT)0 : a2.y};
        }
        const cpx<CT> a0 = A.spec_in[o], a1 = A.spec_in[FS + o];
        return j == 0 ? cpx<CT>{a0.x, a1.x} : cpx<CT>{a0.x - a1.y, a0.y + a1.x};
      };
      // its conjugate-symmetric partner N_y - j
      auto conj_elem = [&](int j) -> cpx<CT> {
        const int64_t o = Spec2<CT>::at(xl, j, N0);
        if (line & 1) {
          const cpx<CT> a2 = A.spec_in[2 * FS + o];
          return {a2.x, -a2.y};
        }
        const cpx<CT> a0 = A.spec_in[o], a1 = A.spec_in[FS + o];
        return {a0.x + a1.y, a1.x - a0.y};
      };
      cpx<CT> v[4] = {elem(t), {0, 0}, {0, 0}, conj_elem(F::TPL - t)};
      if (t == 0) v[1] = elem(F::TPL);
      cpx<CT>* ln = ibuf + line * T2;
      F::template run<+1>(v, t, ln, ln, tw);
#pragma unroll
      for (int i = 0; i < 4; ++i) ln[t + i * F::TPL] = v[i];
    }
    __syncthreads();
    const cpx<CT>* dmr = ibuf + 2 * pl * T2;
    raw.dmv[0] = (TM)dmr[y].x;
    raw.dmv[1] = (TM)dmr[y].y;
    raw.dmv[2] = (TM)dmr[T2 + y].x;
  }

  CT f[Q], C[Q];
  double hs[4], mns[4], mtr[4];
  collide_raw<L, T, TM, MODE>(A, raw, f, C, hs, mtr, mns);
  if (setup_mode(MODE) && pl == 1) {
#pragma unroll
    for (int b = 0; b <= D; ++b) A.h[b * NS + site] = hs[b];
    if (A.recon) {
#pragma unroll
      for (int b = 0; b <= D; ++b) P.mw[b * NS + site] = mns[b];
    }
  }
  // push (Eq. sweep): the directions that carry this plane into x0
#pragma unroll
  for (int k = 0; k < Q; ++k)
    if (L::cx(k) == 1 - pl) val[k][(y + L::cy(k)) & (T2 - 1)] = (LT)C[k];
  __syncthreads();

  double r2 = 0.0;
  if (pl == 1) {
    CT vv[Q], pr[4] = {0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < Q; ++k) vv[k] = (CT)val[k][y];
    if (A.walls) cavity_rows<CT>(vv, x0, y, N0, T2, (CT)A.ulid);
    float Mq[DV ? D + 1 : 1];
    if constexpr (DV) {
      // store (g, M); the residual is taken against the stored output
      T gq[Q];
      dev_split<L, typename std::conditional<DUAL, double, float>::type>(vv, A.isig, gq, Mq);
#pragma unroll
      for (int k = 0; k < Q; ++k) __builtin_nontemporal_store(gq[k], &dst[k * NS + site]);
      float* dM = dev_moments(dst, Q, NS);
#pragma unroll
      for (int b = 0; b <= D; ++b) __builtin_nontemporal_store(Mq[b], &dM[b * NS + site]);
      if (DUAL) dev_rebuild<L>(gq, Mq, A.sig, vv);
    }
#pragma unroll
    for (int k = 0; k < Q; ++k) {
      const CT v = vv[k];
      if constexpr (!DV) __builtin_nontemporal_store((T)v, &dst[k * NS + site]);
      if (DUAL) {
        const CT r = v - f[k];
        if (A.rout) __builtin_nontemporal_store((TM)r, &A.rout[k * NS + site]);
        pr[0] += r;
#pragma unroll
        for (int b = 0; b < D; ++b)
          if (ca<L>(k, b) != 0) pr[1 + b] += (CT)ca<L>(k, b) * r;
        r2 += (double)r * (double)r;
      }
    }
    if constexpr (DV && DUAL) {
      // P r exactly: the stored output moments minus the trial's
#pragma unroll
      for (int b = 0; b <= D; ++b) pr[b] = (CT)((double)Mq[b] - mtr[b]);
    }
    if constexpr (DUAL) {
      if (A.fuse_rows) {
        fbuf[y] = {pr[0], pr[1]};
        fbuf[T2 + y] = {pr[2], (CT)0};
      } else if (!A.rout && !A.skip_pr) {
#pragma unroll
        for (int b = 0; b <= D; ++b) __builtin_nontemporal_store((TM)pr[b], &A.Pr[b * NS + site]);
      }
    }
  }
  if constexpr (DUAL) {
    if (pl == 1) {
      // FP64 sum of r^2 over the row, as k_sweep's block sum
      if constexpr (T2 >= 64) {
        double v = r2;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        if ((y & 63) == 0) red[y >> 6] = v;
      } else {
        red[y] = r2;
      }
    }
    __syncthreads();
    if (tid == 0) {
      double acc = 0.0;
      for (int i = 0; i < NRED; ++i) acc += red[i];
      A.partials[blockIdx.x] = acc;
    }
    if (MODE == SW_DTS && A.rms) rows_rms<3 * T2>(A.partials, A.rms, A.arrived, A.arrivals, A.inv_count);
    if (A.fuse_rows) row_spectrum<T2>(A.spec, N0, A.NBr, fbuf, tid, x0, tw);
  }
}

}  // namespace msc
