// Solver<L, T>: device buffers and kernel sequencing for one lattice and
// storage type.  Included by one translation unit per instantiation.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstring>
#include <initializer_list>
#include <memory>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include <hip/hip_ext.h>

#include "msc_march2.h"
#include "msc_adjoint.h"
#include "msc_sweep_launch.h"
#include "msc_fullsym.h"
#include "msc_walls.h"
#include "msc_solver.h"

namespace msc {

#define MSC_HIPCK(x)                                                                 \
  do {                                                                               \
    hipError_t e_ = (x);                                                             \
    if (e_ != hipSuccess) throw DeviceError{e_, std::string(#x) + ": " + hipGetErrorString(e_)}; \
  } while (0)

struct OomError {};

inline int ilog2(int n) {
  int l = 0;
  while ((1 << l) < n) ++l;
  return l;
}

// Buffers of one run of the correction transforms in one precision.
template <class CX, class TX>
struct XformBufs {
  const TX* in;
  TX* out;
  cpx<CX>* spec1;
  cpx<CX>* spec2;
  const cpx<CX>* tw[3];
};

// ----------------------------------------------------------------- solver --
template <class L, class T>
class Solver : public SolverBase {
 public:
  using CT = typename CompT<T>::type;
  using TM = CT;
  static constexpr int Q = L::Q, D = L::D;
  static constexpr bool DV = PopDev<T>::value;  // FP16 deviation storage

  Solver(const msc_params& p, const Geometry& g, hipStream_t s) : P(p), G(g), st(s) {
    wp = 1.0 / P.tau_plus;
    wm = 1.0 / P.tau_minus;
    nu = (P.tau_plus - 0.5) / 3.0;  // Eq. (trt): nu = cs^2 (tau+ - 1/2)
  }
  ~Solver() override { release(); }

  Tuning& tuning() override { return tune; }

  void krylov_stats(int64_t* solves, int64_t* iters, int64_t* refreshes, double* worst) const override {
    if (solves) *solves = kr_solves;
    if (iters) *iters = kr_iters;
    if (refreshes) *refreshes = kr_refresh;
    if (worst) *worst = kr_worst;
  }

  msc_status reconfigure() override {
    return guard([&]() {
      sync();
      choose_sweep();
      ensure_partials(sweep_grid_max());
      for (auto& g : graphs) drop_graph(g);
      return MSC_OK;
    });
  }

  // ----------------------------------------------------------------- init --
  msc_status init(const double* phat0, const double* u0, bool on_device) override {
    return guard([&]() -> msc_status {
      if (P.corrector == MSC_CORRECTOR_SHADOW && !corrector_supported()) {
        last_error = "the shadow corrector is not available for this lattice/grid size";
        return MSC_ERR_UNSUPPORTED;
      }
      if (wallkin() && !wall_supported()) {
        last_error = "the wall-kinetic corrector needs the D2Q9 cavity, FP64 storage, tau+ = tau- = 1 and "
                     "extents up to 256 x 512";
        return MSC_ERR_UNSUPPORTED;
      }
      if (fullsym() && !fs_supported()) {
        last_error = "the full-symbol corrector needs D2Q9 with FP64 or FP32 storage and extents up to "
                     "256 x 512 (FP64) or 512 x 1024 (FP32)";
        return MSC_ERR_UNSUPPORTED;
      }
      allocate();
      // Algorithm 2: the initial wall operator is assembled at rest with the
      // BDF2 coefficient
      wk_aA = 1.5 / P.dt;
      wk_rest = true;
      const int64_t NS = G.NS;
      double* pd = nullptr;
      double* ud = nullptr;
      if (on_device) {
        after_default_stream();
        pd = const_cast<double*>(phat0);
        ud = const_cast<double*>(u0);
      } else {
        double* stg = staging();
        MSC_HIPCK(hipMemcpyAsync(stg, phat0, sizeof(double) * NS, hipMemcpyHostToDevice, st));
        MSC_HIPCK(hipMemcpyAsync(stg + NS, u0, sizeof(double) * D * NS, hipMemcpyHostToDevice, st));
        pd = stg;
        ud = stg + NS;
      }
      // control block: slots 0,1,2 hold f^n, f^{n-1}, f^{n-2}; 3,4 work.
      std::memset(ctl_h, 0, sizeof(DevCtl));
      ctl_h->phase = make_phase(-1, 0, PH_ACCEPTED);
      for (int r = 0; r < 2; ++r) {
        Roles& ro = ctl_h->roles[r];
        for (int i = 0; i < 3; ++i) ro.slot_hist[i] = i;
        ro.slot_w[0] = 3;
        ro.slot_w[1] = 4;
        for (int i = 0; i < 3; ++i) ro.slot_m[i] = i;
      }
      n_next = 0;
      MSC_HIPCK(hipMemcpyAsync(ctl, ctl_h, sizeof(DevCtl), hipMemcpyHostToDevice, st));
      if (DV) sig = choose_sigma(0.0, std::max(absmax(pd, NS), absmax(ud, (int64_t)D * NS)));
      hipLaunchKernelGGL((k_init_feq<L, T>), dim3(ew_grid()), dim3(256), 0, st, pd, ud, fb.p[0], NS);
      MSC_HIPCK(hipGetLastError());
      reset_history_from_current();
      sync();
      for (auto& t : tw_host) t = {};
      return MSC_OK;
    });
  }

  // ------------------------------------------------------- BDF dual time --
  msc_status bdf2_step(int32_t nsteps, msc_step_stats* out) override {
    if (wallkin()) return bdf2_step_walls(nsteps, out);
    return guard([&]() -> msc_status {
      if (nsteps <= 0) return MSC_OK;
      ensure_stats(nsteps);
      const int stat_base = n_next;
      const int n_end = n_next + nsteps;
      RecordScope recs(*this);  // drops the records of steps that were not accepted
      handed_on.ctl = nullptr;
      // schedule replay for these steps
      const bool use_sched = sched_pos < (int64_t)sched_h.size();
      if (use_sched) {
        std::vector<int32_t> K(nsteps, 0);
        for (int i = 0; i < nsteps; ++i) {
          const int64_t j = sched_pos + i;
          K[i] = (j < (int64_t)sched_h.size()) ? sched_h[j] : P.k_max;
        }
        ensure_sched(nsteps);
        MSC_HIPCK(hipMemcpyAsync(sched_d, K.data(), sizeof(int32_t) * nsteps, hipMemcpyHostToDevice, st));
        sched_host_view = K;
      }
      if (replayed && !use_sched) batch = 1;
      replayed = use_sched;
      int n_dev = n_next, ell_dev = 1;
      int64_t bdf_dev = bdf_count;
      msc_status rc = MSC_OK;
      while (n_dev < n_end) {
        // (key 2 may have been lowered since the batch grew)
        int B = std::min({batch, std::max(1, tune.batch_steps), n_end - n_dev});
        if (recording) {
          // only steps that have a record are enqueued
          B = reserve_records(n_dev, bdf_dev, B, stat_base, n_end - n_dev);
          if (B == 0) {
            // (a step that still iterates has one: the march stands at an
            // accepted step, whose m^n was left to the step that does not come)
            if (n_dev > stat_base) reconstruct(n_dev, bdf_dev);
            copy_stats(out, stat_base, n_dev - stat_base);
            recs.accept(n_dev - stat_base);
            n_next = n_dev;
            bdf_count = bdf_dev;
            if (use_sched) sched_pos += n_dev - stat_base;
            sync();
            last_error = "device allocation failed for the record of physical step " + std::to_string(n_dev);
            return MSC_ERR_OUT_OF_MEMORY;
          }
        }
        for (int i = 0; i < B; ++i) {
          const int n = n_dev + i;
          const int64_t bc = bdf_dev + i;
          const int q = (bc == 0) ? 1 : 2;
          const int max_order = (P.extrap_states == 0) ? 2 : P.extrap_states - 1;
          const int order = (int)std::min<int64_t>(bc, max_order);
          const double a = (q == 1) ? 1.0 / P.dt : 3.0 / (2.0 * P.dt);
          const int ell0 = (i == 0) ? ell_dev : 1;
          int want;
          if (use_sched)
            want = sched_host_view[n - stat_base];
          else
            want = std::max(P.n_min, last_iters + tune.spec_extra);
          int ell1 = (ell0 == 1) ? want : ell0 - 1 + std::max(8, want);
          ell1 = std::min(std::max(ell1, ell0), P.k_max);
          // resuming a step: the previous batch ended it at sweep ell0 - 1
          // without the correction's later passes
          if (ell0 > 1) enqueue_correction_tail(n, ell0 - 1, a);
          // within one call, each step's acceptance leaves m^{n+1} to the next
          // step's setup sweep (which reads the same populations anyway); the
          // call's last step reconstructs it so that the state is complete
          // when the call returns
          const bool recon = n > stat_base;
          const double a_prev = (bc - 1 == 0) ? 1.0 / P.dt : 3.0 / (2.0 * P.dt);
          const bool defer = n < n_end - 1;
          CkptArgs<T>* rec = nullptr;
          CkptArgs<T> ck;
          if (recording && ell0 == 1) {
            ck = checkpoint_args(n, recs.base + (size_t)(n - stat_base));
            rec = &ck;
          }
          // the decision on this step's last sweep goes with the next step's
          // first sweep where that one follows at once and can take it
          const bool hand_on = i < B - 1 && merge_ok();
          for (int ell = ell0; ell <= ell1; ++ell)
            enqueue_iteration(n, ell, q, order, a, use_sched, stat_base, ell == ell1, recon, a_prev, defer, rec,
                              hand_on);
        }
        fetch_ctl(nsteps);
        const uint64_t ph = ctl_h->phase;
        const int pn = phase_n(ph), pell = phase_ell(ph);
        const uint32_t ps = phase_state(ph);
        if (ps == PH_FAILED) {
          bdf_dev += (pn - n_dev);
          rc = (ctl_h->fail_code == 5) ? MSC_ERR_NONCONVERGED : MSC_ERR_NONFINITE;
          last_error = std::string(rc == MSC_ERR_NONCONVERGED ? "nonconvergent" : "non-finite residual") +
                       " at physical step " + std::to_string(pn) + ", inner iteration " + std::to_string(pell);
          // the march stays at the last accepted step
          ctl_h->phase = make_phase(pn - 1, 0, PH_ACCEPTED);
          ctl_h->fail_code = 0;
          MSC_HIPCK(hipMemcpyAsync(ctl, ctl_h, sizeof(DevCtl), hipMemcpyHostToDevice, st));
          copy_stats(out, stat_base, pn - stat_base + 1);
          recs.accept(pn - stat_base);
          n_next = pn;
          bdf_count = bdf_dev;
          batch = 1;
          sched_pos += (pn - stat_base);
          sync();
          return rc;
        }
        if (ps == PH_ACCEPTED) {
          bdf_dev += (pn - n_dev + 1);
          n_dev = pn + 1;
          ell_dev = 1;
          last_iters = pell;
          batch = std::min(batch * 2, std::max(1, tune.batch_steps));
        } else {
          // still iterating step pn after pell sweeps
          bdf_dev += (pn - n_dev);
          n_dev = pn;
          ell_dev = pell + 1;
          last_iters = std::max(last_iters, pell + 1);
          batch = 1;
        }
      }
      copy_stats(out, stat_base, nsteps);
      recs.accept(nsteps);
      n_next = n_end;
      bdf_count = bdf_dev;
      if (use_sched) sched_pos += nsteps;
      return rc;
    });
  }

  // -------------------------------------------------------- explicit march --
  msc_status explicit_step(int64_t nsteps) override {
    return guard([&]() -> msc_status {
      T* A = fb.p[cur_roles().slot_hist[0]];
      T* B = fb.p[cur_roles().slot_w[0]];
      SweepArgs<T, TM> S = sweep_args(0.0);
      const int64_t chunk = 64;
      int64_t done = 0;
      const int kind = explicit_kind();
      // steps that the chosen kernels take before the tiled sweep takes the
      // rest one by one: all of them (tiled), or pairs of steps
      const int64_t paired = (kind == EX_TILED) ? 0 : (nsteps & ~(int64_t)1);
      const int64_t graphed = (kind == EX_TILED) ? nsteps : paired;
      if (tune.use_graph && graphed >= chunk && !timing) {
        hipGraphExec_t ge = explicit_graph(A, B, (int)chunk, kind);
        for (; done + chunk <= graphed; done += chunk) MSC_HIPCK(hipGraphLaunch(ge, st));
      }
      T* cur = A;
      T* oth = B;
      if (kind == EX_MULTI) {
        const int sm = march2_steps(march2_tile());
        for (; done + sm <= paired; done += sm) {
          launch_march2(cur, oth);
          std::swap(cur, oth);
        }
      }
      for (; done < paired; done += 2) {
        launch_aa(cur, false);
        launch_aa(cur, true);
      }
      for (; done < nsteps; ++done) {
        S.src = cur;
        S.dst = oth;
        launch_sweep_timed(SW_EXPLICIT, S, 1);
        std::swap(cur, oth);
      }
      if (cur != A) std::swap(cur_roles().slot_hist[0], cur_roles().slot_w[0]);
      MSC_HIPCK(hipMemcpyAsync(ctl, ctl_h, sizeof(DevCtl), hipMemcpyHostToDevice, st));
      // non-finite check on the final state
      if (!std::isfinite(reset_history_from_current(true))) {
        last_error = "non-finite population after the explicit march";
        return MSC_ERR_NONFINITE;
      }
      return MSC_OK;
    });
  }

  // How the explicit march runs: the tiled two-buffer sweep; the in-place AA
  // march; or, in 2D, several steps per launch (the AA pattern in LDS), with
  // AA pairs for what is left of the count.  Kernel timing reports single
  // steps, so it takes the AA march.
  enum { EX_TILED = 0, EX_AA = 1, EX_MULTI = 2 };
  int explicit_kind() const {
    if (!aa_ok()) return EX_TILED;
    return (!timing && march2_tile() >= 0) ? EX_MULTI : EX_AA;
  }

  // Tile of k_march2, or -1 where the grid is smaller than a tile.  Measured
  // us per step (single-step AA march; 8 x 16 tile; 16 x 16; the large one):
  // FP64 N = 128 2.9; 0.93; 1.07; 1.6, N = 256 3.3; 1.40; 1.19; 1.7, N = 512
  // 6.4; 4.4; 3.2; 2.9, N = 2048 100; -; -; 45; FP32 N = 128 2.8; 0.87; 1.0;
  // 1.5, N = 256 2.8; 1.28; 1.07; 2.0, N = 512 4.3; 3.0; 2.9; 2.2, N = 2048
  // 44; -; -; 28.  Small tiles fill the chip and keep a step's chain short;
  // with more tiles than compute units the halo work decides.
  int march2_tile() const {
    if (D != 2 || DV) return -1;
    if (G.NS <= 32768 && G.N0 >= 8 && G.N2 >= 16) return 0;
    if (G.NS <= 131072 && G.N0 >= 16 && G.N2 >= 16) return 1;
    if (G.NS > 131072 && G.N0 >= 32 && G.N2 >= 32) return 2;
    return -1;
  }
  static int march2_steps(int tile) { return tile == 2 ? 4 : 8; }

  // march2_steps(tile) steps from in to out
  void launch_march2(const T* in, T* out) {
    if constexpr (D == 2 && !DV) {
      March2Args<T> A{};
      A.in = in;
      A.out = out;
      A.Nx = G.N0;
      A.Ny = G.N2;
      A.lgy = ilog2(G.N2);
      A.wp = wp;
      A.wm = wm;
      const int tile = march2_tile();
      if (tile == 0)
        launch_march2_tile<8, 16, 8, 512>(A);
      else if (tile == 1)
        launch_march2_tile<16, 16, 8, 1024>(A);
      else if constexpr (sizeof(T) == 8)
        launch_march2_tile<16, 32, 4, 512>(A);
      else
        launch_march2_tile<32, 32, 4, 1024>(A);
    }
  }
  template <int BX, int BY, int SM, int NT>
  void launch_march2_tile(March2Args<T>& A) {
    A.lgty = ilog2(G.N2 / BY);
    const dim3 grid((G.N0 / BX) * (G.N2 / BY));
    if (A.wp == 1.0 && A.wm == 1.0)
      hipLaunchKernelGGL((k_march2<T, true, BX, BY, SM, NT>), grid, dim3(NT), 0, st, A);
    else
      hipLaunchKernelGGL((k_march2<T, false, BX, BY, SM, NT>), grid, dim3(NT), 0, st, A);
    MSC_HIPCK(hipGetLastError());
  }

  // The in-place (AA) explicit march: periodic boundaries and full-population
  // storage (FP64, FP32); the cavity and FP16-deviation storage keep the
  // two-buffer sweep.
  bool aa_ok() const { return tune.explicit_aa && !walls() && !PopDev<T>::value && G.NS < ((int64_t)1 << 31); }

  // one AA kernel (odd = false: the even kernel) on the population array f
  void launch_aa(T* f, bool odd) {
    if constexpr (!PopDev<T>::value) {
      AaArgs<T> A{};
      A.f = f;
      A.N0 = G.N0;
      A.N1 = G.N1;
      A.N2 = G.N2;
      A.lg1 = ilog2(G.N1);
      A.lg2 = ilog2(G.N2);
      A.NS = (int)G.NS;
      A.wp = 1.0 / P.tau_plus;
      A.wm = 1.0 / P.tau_minus;
      EvPair ep{};
      if (timing) {
        ep = timed_pair(1, 2.0 * Q * (double)G.NS * sizeof(T));
        A.did_run = run_flags + ep.flag;
        MSC_HIPCK(hipEventRecord(ep.a, st));
      }
      const int grid = (int)((G.NS + 255) / 256);
      if (odd)
        hipLaunchKernelGGL((k_aa_odd<L, T>), dim3(grid), dim3(256), 0, st, A);
      else
        hipLaunchKernelGGL((k_aa_even<L, T>), dim3(grid), dim3(256), 0, st, A);
      MSC_HIPCK(hipGetLastError());
      if (timing) {
        MSC_HIPCK(hipEventRecord(ep.b, st));
        ev_live.push_back(ep);
        if ((int)ev_live.size() >= kFlagCap) collect_timing();
      }
    }
  }

  // -------------------------------------------------------------- outputs --
  msc_status moments(double* phat, double* u, bool on_device) override {
    return guard([&]() {
      if (on_device) after_default_stream();
      const double* m = mb[cur_roles().slot_m[0]];
      const hipMemcpyKind kind = on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost;
      if (phat && u == phat + G.NS) {
        MSC_HIPCK(hipMemcpyAsync(phat, m, sizeof(double) * (D + 1) * G.NS, kind, st));
      } else {
        if (phat) MSC_HIPCK(hipMemcpyAsync(phat, m, sizeof(double) * G.NS, kind, st));
        if (u) MSC_HIPCK(hipMemcpyAsync(u, m + G.NS, sizeof(double) * D * G.NS, kind, st));
      }
      sync();
      return MSC_OK;
    });
  }

  msc_status export_tables(int32_t* nbr, int32_t* sidx, uint8_t* mask) override {
    return guard([&]() {
      const int64_t NS = G.NS;
      const int nsum = G.n[0] + G.n[1] + (D == 3 ? G.n[2] : 0);
      int32_t* dn = (int32_t*)dalloc(sizeof(int32_t) * Q * NS);
      uint8_t* dmk = (uint8_t*)dalloc(NS);
      int32_t* ds = (int32_t*)dalloc(sizeof(int32_t) * nsum);
      hipLaunchKernelGGL((k_tables<L>), dim3(ew_grid()), dim3(256), 0, st, G.N0, G.N1, G.N2, dn, dmk, ds);
      MSC_HIPCK(hipGetLastError());
      if (nbr) MSC_HIPCK(hipMemcpyAsync(nbr, dn, sizeof(int32_t) * Q * NS, hipMemcpyDeviceToHost, st));
      if (mask) MSC_HIPCK(hipMemcpyAsync(mask, dmk, NS, hipMemcpyDeviceToHost, st));
      if (sidx) MSC_HIPCK(hipMemcpyAsync(sidx, ds, sizeof(int32_t) * nsum, hipMemcpyDeviceToHost, st));
      sync();
      dfree(dn);
      dfree(dmk);
      dfree(ds);
      return MSC_OK;
    });
  }

  msc_status get_populations(double* f) override {
    return guard([&]() {
      download_pop(fb.p[cur_roles().slot_hist[0]], f);
      return MSC_OK;
    });
  }

  msc_status set_populations(const double* f) override {
    return guard([&]() {
      if (DV) sig = sigma_for({f});
      upload_pop(f, fb.p[cur_roles().slot_hist[0]]);
      reset_history_from_current();
      sync();
      return MSC_OK;
    });
  }

  // ------------------------------------------------------------ diagnostics --
  msc_status sweep(const double* f, const double* h_in, double a, double* fT, double* Pr_out,
                   double* R) override {
    return guard([&]() {
      T* A = fb.p[cur_roles().slot_w[0]];
      T* B = fb.p[cur_roles().slot_w[1]];
      const float sig_state = sig;  // the work buffers may take another scale
      if (DV) sig = sigma_for({f});
      upload_pop(f, A);
      upload_h(h_in);
      SweepArgs<T, TM> S = sweep_args(a);
      S.src = A;
      S.dst = B;
      launch_sweep_timed(SW_DTS, S, 0);
      const double Rv = reduce_partials(S);
      if (R) *R = Rv;
      if (fT) download_pop(B, fT);
      if (Pr_out) download_tm(Pr, Pr_out, (int64_t)(D + 1) * G.NS);
      sync();
      sig = sig_state;
      return MSC_OK;
    });
  }

  msc_status correct(const double* f, const double* h_in, double a, double* fnext, double* dm_out,
                     double* R) override {
    if (fullsym()) return correct_fullsym(f, h_in, a, fnext, dm_out, R);
    if (wallkin()) return correct_walls(f, h_in, a, fnext, dm_out, R);
    return guard([&]() -> msc_status {
      if (!corrector_supported()) {
        last_error = "the shadow corrector is not available for this lattice/grid";
        return MSC_ERR_UNSUPPORTED;
      }
      T* A = fb.p[cur_roles().slot_w[0]];
      T* B = fb.p[cur_roles().slot_w[1]];
      const float sig_state = sig;
      if (DV) sig = sigma_for({f});
      upload_pop(f, A);
      upload_h(h_in);
      SweepArgs<T, TM> S = sweep_args(a);
      S.src = A;
      S.dst = B;
      launch_sweep_timed(SW_DTS, S, 0);
      const double Rv = reduce_partials(S);
      if (R) *R = Rv;
      enqueue_correction(nullptr, 0, 0, a, nullptr);
      // f_next = f_T + E dm: the same lift the next sweep applies on load,
      // here through an explicit no-op-collision pass is not available, so
      // apply it element-wise.
      hipLaunchKernelGGL((k_lift<L, T, TM>), dim3(ew_grid()), dim3(256), 0, st, B, dm, A, G.NS, sig, 1.0f / sig);
      MSC_HIPCK(hipGetLastError());
      if (fnext) download_pop(A, fnext);
      if (dm_out) download_tm(dm, dm_out, (int64_t)(D + 1) * G.NS);
      sync();
      sig = sig_state;
      return MSC_OK;
    });
  }

  // One full-symbol corrected iteration from host arrays: f_T = T(f), the
  // correction of Eq. (full-symbol), f_next = f + df; dm_out (no macroscopic
  // correction field here) is zeroed.
  msc_status correct_fullsym(const double* f, const double* h_in, double a, double* fnext, double* dm_out,
                             double* R) {
    return guard([&]() -> msc_status {
      T* A = fb.p[cur_roles().slot_w[0]];
      T* B = fb.p[cur_roles().slot_w[1]];
      upload_pop(f, A);
      upload_h(h_in);
      SweepArgs<T, TM> S = sweep_args(a);
      S.src = A;
      S.dst = B;
      S.rout = rfs;
      launch_sweep_timed(SW_DTS, S, 0);
      const double Rv = reduce_partials(S);
      if (R) *R = Rv;
      enqueue_fullsym(nullptr, 0, 0, a, nullptr, nullptr, true, true, B);
      if (fnext) download_pop(B, fnext);
      sync();
      if (dm_out) std::memset(dm_out, 0, sizeof(double) * (D + 1) * G.NS);
      return MSC_OK;
    });
  }

  // ------------------------------------------- wall-bounded correction --
  template <class W>
  void wall_parts(W&& want) {
    const int64_t n = (int64_t)Q * G.NS;
    wk_m = P.wall_restart > 0 ? P.wall_restart : 50;
    std::fill(wk_pred, wk_pred + kWallPred, 8);
    want(wk_V, sizeof(double) * (wk_m + 1) * n);
    want(wk_R, sizeof(double) * n);
    want(wk_D, sizeof(double) * n);
    want(wk_vc, sizeof(double) * n);
    want(wk_spec, sizeof(cpx<double>) * 3 * Spec2<double>::field(G.N0, G.N2 / 2 + 1));
    want(wk_mref, sizeof(double) * 3 * G.NS);
    want(wk_sref, sizeof(double) * 3 * G.NS);
    // the state word, then the dot-product partials (one entry of N_x per vector)
    want(wk_part, sizeof(double) * (1 + (size_t)G.N0 * (wk_m + 2)));
    want(wk_coef, sizeof(double) * (wk_m + 2));
    // Hd (m x m), cs, sn (m each), g (m + 1), hcol (m + 2)
    want(wk_small, sizeof(double) * ((size_t)wk_m * wk_m + 4 * wk_m + 3));
  }

  WallArgs wall_args() const {
    WallArgs A{};
    A.Nx = G.N0;
    A.Ny = G.N2;
    A.NS = G.NS;
    A.a = wk_aA;
    A.g = (1.0 - 0.5 * wk_aA) / (1.0 + 0.5 * wk_aA);
    A.mref = wk_rest ? nullptr : wk_mref;
    A.sref = wk_rest ? nullptr : wk_sref;
    A.vc = wk_vc;
    A.spec = wk_spec;
    if constexpr (std::is_same<CT, double>::value) {
      A.twx = tw[0];
      A.twy = tw[2];
    }
    A.state = reinterpret_cast<WallState*>(wk_part);
    A.part = wk_part + 1;
    A.m = wk_m;
    A.Hd = wk_small;
    A.cs = A.Hd + (size_t)wk_m * wk_m;
    A.sn = A.cs + wk_m;
    A.gv = A.sn + wk_m;
    return A;
  }

  // Restarted GMRES(m), right-preconditioned (msc_walls.h), classical
  // Gram-Schmidt (with one re-orthogonalisation when krylov_tol < 1e-8; a
  // single projection otherwise, which halves the passes over the basis):
  // delta ~ (I - L)^{-1} rhs to the relative residual krylov_tol, beta0 =
  // |rhs|; then f_T <- f_T + (delta - rhs) = f + delta, f the sweep's input.
  // The basis is stored in FP32 when krylov_tol >= 1e-5 (half the bytes of the
  // passes over it; its rounding, ~1e-7 relative, stays far below such
  // tolerances), else in FP64; the new vector, the coefficients and every sum
  // are FP64.  The host enqueues as many iterations as the last solve took and
  // the solution's assembly, which the device skips unless the estimate has
  // converged, and reads the state once.  ell: the inner iteration.
  void wall_solve(const double* rhs, double beta0, double* fT, int ell) {
    const double tol = P.krylov_tol > 0.0 ? P.krylov_tol : 1e-12;
    if (!(beta0 > 0.0) || !std::isfinite(beta0)) return;  // delta = 0
    int& pred = wk_pred[std::min(ell, kWallPred) - 1];
    with_lg<2, LineMax<double>::wall_rows>(ilog2(G.N2), [&](auto lgy) {
      with_lg<2, LineMax<double>::wall_cols>(ilog2(G.N0), [&](auto lgx) {
        if (tol >= 1e-5)
          wall_solve_t<lgx.value, lgy.value, float>(rhs, beta0, fT, tol, pred);
        else
          wall_solve_t<lgx.value, lgy.value, double>(rhs, beta0, fT, tol, pred);
      });
    });
  }

  template <int LGX, int LGY, class VT>
  void wall_solve_t(const double* rhs, double beta0, double* fT, double tol, int& pred) {
    const int64_t n = (int64_t)Q * G.NS;
    const int m = wk_m, rows = G.N0;
    const int max_restarts = 40;
    const bool reorth = tol < 1e-8;
    VT* V = reinterpret_cast<VT*>(wk_V);
    WallArgs A = wall_args();
    A.stop = tol * beta0;
    double* hcol = reorth ? A.gv + (m + 1) : nullptr;
    const int vgrid = (int)std::min<int64_t>((n + 255) / 256, 2048);
    auto cols = [&](int run_on) {
      hipLaunchKernelGGL((k_wall_cols<LGX>), dim3(pad8(G.N2 / 2 + 1)), dim3(256), 0, st, A, run_on);
    };
    auto orth = [&](int j, const double* src, double scale0) {
      hipLaunchKernelGGL((k_wall_orth<LGY, VT>), dim3(rows + 1), dim3(wall_threads(LGY)), 0, st, A, V, j,
                         (const double*)hcol, src, scale0);
    };
    double beta = beta0, rel = 0.0;
    int iters = 0;
    bool updated = false;
    for (int rs = 0; rs < max_restarts; ++rs) {
      orth(0, rs == 0 ? rhs : (const double*)wk_R, 1.0 / beta);
      int j = 0;
      bool done = false;
      WallState ws{};
      do {
        const int upto = std::min(m, j == 0 ? pred : j + 2);
        for (; j < upto; ++j) {
          cols(0);
          hipLaunchKernelGGL((k_wall_rows<LGY, VT>), dim3(rows), dim3(wall_threads(LGY)), 0, st, A, (const VT*)V,
                             j);
          if (reorth) {
            hipLaunchKernelGGL(k_gs_first<0>, dim3(1), dim3(1024), 0, st, (const double*)A.part, rows, j + 1, wk_coef,
                               hcol);
            hipLaunchKernelGGL(k_axpy_multi<VT>, dim3(vgrid), dim3(256), 0, st, wk_vc, (const VT*)V, n, j + 1,
                               (const double*)wk_coef, n);
            hipLaunchKernelGGL((k_wall_dots<LGY, VT>), dim3(rows), dim3(wall_threads(LGY)), 0, st, A,
                               (const VT*)V, j);
          }
          orth(j + 1, nullptr, 0.0);
        }
        const int force = (j == m) ? m : 0;
        hipLaunchKernelGGL((k_wall_combine<LGY, VT>), dim3(rows), dim3(512), 0, st, A, (const VT*)V, force);
        cols(force ? 2 : 1);
        hipLaunchKernelGGL((k_wall_finish<LGY>), dim3(rows), dim3(512), 0, st, A, rhs, wk_D, wk_R, fT, rs == 0 ? 1 : 0,
                           force);
        MSC_HIPCK(hipGetLastError());
        MSC_HIPCK(hipMemcpyAsync(wk_part_h, wk_part, sizeof(double) * (1 + rows), hipMemcpyDeviceToHost, st));
        sync();
        std::memcpy(&ws, wk_part_h, sizeof(ws));
        done = ws.done != 0;
      } while (!done && j < m);
      const int took = done ? ws.jend : m;
      iters += took;
      if (rs == 0) pred = std::max(1, took);
      double r2 = 0.0;
      for (int x = 0; x < rows; ++x) r2 += wk_part_h[1 + x];
      beta = std::sqrt(r2);
      rel = beta / beta0;
      updated = done;
      if (done || rel <= tol || !(beta > 0.0)) break;
    }
    if (!updated) {
      hipLaunchKernelGGL(k_wall_update<0>, dim3(vgrid), dim3(256), 0, st, fT, (const double*)wk_D, rhs, n);
      MSC_HIPCK(hipGetLastError());
    }
    kr_solves += 1;
    kr_iters += iters;
    kr_worst = std::max(kr_worst, rel);
  }

  // Algorithm 2 driven from the host: each inner iteration is the sweep (with
  // the wall rows) and the device-side acceptance decision, then, when the
  // step goes on, the residual guard (adaptive branch) and the correction.
  msc_status bdf2_step_walls(int32_t nsteps, msc_step_stats* out) {
    return guard([&]() -> msc_status {
      if constexpr (std::is_same<T, double>::value) {
        if (nsteps <= 0) return MSC_OK;
        ensure_stats(nsteps);
        const int stat_base = n_next;
        const bool use_sched = sched_pos < (int64_t)sched_h.size();
        if (use_sched) {
          std::vector<int32_t> K(nsteps, 0);
          for (int i = 0; i < nsteps; ++i) {
            const int64_t j = sched_pos + i;
            K[i] = (j < (int64_t)sched_h.size()) ? sched_h[j] : P.k_max;
          }
          ensure_sched(nsteps);
          MSC_HIPCK(hipMemcpyAsync(sched_d, K.data(), sizeof(int32_t) * nsteps, hipMemcpyHostToDevice, st));
        }
        wall_refreshes.assign(nsteps, 0);
        const int64_t NS = G.NS;
        double Rdev = 0.0;
        for (int i = 0; i < nsteps; ++i) {
          const int n = n_next;
          const int64_t bc = bdf_count;
          const int q = (bc == 0) ? 1 : 2;
          const int max_order = (P.extrap_states == 0) ? 2 : P.extrap_states - 1;
          const int order = (int)std::min<int64_t>(bc, max_order);
          const double a = (q == 1) ? 1.0 / P.dt : 3.0 / (2.0 * P.dt);
          int n_grow = 0, n_ref = 0;
          double Rref = 0.0, Rprev = 0.0;
          for (int ell = 1; ell <= P.k_max; ++ell) {
            enqueue_iteration(n, ell, q, order, a, use_sched, stat_base, true);
            MSC_HIPCK(hipMemcpyAsync(&Rdev, Rhist + (ell - 1), sizeof(double), hipMemcpyDeviceToHost, st));
            fetch_ctl(nsteps);
            const uint32_t ps = phase_state(ctl_h->phase);
            if (ps == PH_ACCEPTED) {
              bdf_count += 1;
              n_next = n + 1;
              last_iters = ell;
              break;
            }
            if (ps == PH_FAILED) {
              const msc_status rc = (ctl_h->fail_code == 5) ? MSC_ERR_NONCONVERGED : MSC_ERR_NONFINITE;
              last_error = std::string(rc == MSC_ERR_NONCONVERGED ? "nonconvergent" : "non-finite residual") +
                           " at physical step " + std::to_string(n) + ", inner iteration " + std::to_string(ell);
              ctl_h->phase = make_phase(n - 1, 0, PH_ACCEPTED);
              ctl_h->fail_code = 0;
              MSC_HIPCK(hipMemcpyAsync(ctl, ctl_h, sizeof(DevCtl), hipMemcpyHostToDevice, st));
              copy_stats(out, stat_base, n - stat_base + 1);
              if (use_sched) sched_pos += (n - stat_base);
              sync();
              return rc;
            }
            // Algorithm 2: residual guard of the adaptive operator
            const double R = Rdev;
            if (ell == 1) Rref = R;
            n_grow = (ell > 1 && R > Rprev) ? n_grow + 1 : 0;
            Rprev = R;
            T* fT = fb.p[ctl_h->roles[n & 1].slot_w[ell & 1]];
            if (P.wall_operator == MSC_WALL_ADAPTIVE && n_ref < 3 &&
                (n_grow >= 2 || R > 10.0 * Rref || (P.wall_forced > 0 && ell % P.wall_forced == 0))) {
              hipLaunchKernelGGL(k_wall_reference<0>, dim3(ew_grid()), dim3(256), 0, st, (const double*)fT,
                                 (const double*)rfs, (const double*)h, a, NS, wk_mref, wk_sref);
              MSC_HIPCK(hipGetLastError());
              wk_aA = a;
              wk_rest = false;
              ++n_ref;
              ++kr_refresh;
              wall_refreshes[i] = n_ref;
              n_grow = 0;
              Rref = R;
            }
            wall_solve(rfs, R * std::sqrt((double)Q * (double)NS), fT, ell);
          }
        }
        copy_stats(out, stat_base, nsteps);
        if (use_sched) sched_pos += nsteps;
        return MSC_OK;
      } else {
        (void)nsteps, (void)out;
        return MSC_ERR_UNSUPPORTED;
      }
    });
  }

  // One wall-corrected iteration from host arrays with the current operator.
  msc_status correct_walls(const double* f, const double* h_in, double a, double* fnext, double* dm_out,
                           double* R) {
    return guard([&]() -> msc_status {
      if constexpr (std::is_same<T, double>::value) {
        T* A = fb.p[cur_roles().slot_w[0]];
        T* B = fb.p[cur_roles().slot_w[1]];
        upload_pop(f, A);
        upload_h(h_in);
        SweepArgs<T, TM> S = sweep_args(a);
        S.src = A;
        S.dst = B;
        S.rout = rfs;
        launch_sweep_timed(SW_DTS, S, 0);
        const double Rv = reduce_partials(S);
        if (R) *R = Rv;
        wall_solve(rfs, Rv * std::sqrt((double)Q * (double)G.NS), B, 1);
        if (fnext) download_pop(B, fnext);
        sync();
        if (dm_out) std::memset(dm_out, 0, sizeof(double) * (D + 1) * G.NS);
        return MSC_OK;
      } else {
        (void)f, (void)h_in, (void)a, (void)fnext, (void)dm_out, (void)R;
        return MSC_ERR_UNSUPPORTED;
      }
    });
  }

  msc_status set_schedule(const int32_t* K, int32_t nsteps) override {
    sched_h.clear();
    sched_pos = 0;
    if (K && nsteps > 0) {
      for (int i = 0; i < nsteps; ++i) {
        if (K[i] < 1) {
          last_error = "schedule entries must be >= 1";
          sched_h.clear();
          return MSC_ERR_INVALID_ARG;
        }
        sched_h.push_back(std::min(K[i], P.k_max));
      }
    }
    return MSC_OK;
  }

  int64_t state_size() const override {
    return 3 * (int64_t)Q * G.NS + 2 * (int64_t)(D + 1) * G.NS;
  }

  msc_status get_state(double* state, int64_t* bc) override {
    return guard([&]() {
      complete_history();
      const int64_t FQ = (int64_t)Q * G.NS, FM = (int64_t)(D + 1) * G.NS;
      for (int i = 0; i < 3; ++i) download_pop(fb.p[cur_roles().slot_hist[i]], state + i * FQ);
      MSC_HIPCK(hipMemcpyAsync(state + 3 * FQ, mb[cur_roles().slot_m[0]], sizeof(double) * FM,
                               hipMemcpyDeviceToHost, st));
      MSC_HIPCK(hipMemcpyAsync(state + 3 * FQ + FM, mb[cur_roles().slot_m[1]], sizeof(double) * FM,
                               hipMemcpyDeviceToHost, st));
      sync();
      if (bc) *bc = bdf_count;
      return MSC_OK;
    });
  }

  msc_status set_state(const double* state, int64_t bc) override {
    return guard([&]() {
      const int64_t FQ = (int64_t)Q * G.NS, FM = (int64_t)(D + 1) * G.NS;
      if (DV) sig = sigma_for({state, state + FQ, state + 2 * FQ});
      for (int i = 0; i < 3; ++i) upload_pop(state + i * FQ, fb.p[cur_roles().slot_hist[i]]);
      MSC_HIPCK(hipMemcpyAsync(mb[cur_roles().slot_m[0]], state + 3 * FQ, sizeof(double) * FM,
                               hipMemcpyHostToDevice, st));
      MSC_HIPCK(hipMemcpyAsync(mb[cur_roles().slot_m[1]], state + 3 * FQ + FM, sizeof(double) * FM,
                               hipMemcpyHostToDevice, st));
      sync();
      lazy_history = false;
      bdf_count = bc;
      batch = 1;
      return MSC_OK;
    });
  }

  // ------------------------------------------------------------- adjoint --
  msc_status set_recording(int enable) override {
    return guard([&]() {
      sync();
      clear_records();
      recording = enable != 0;
      if (!recording) free_adjoint_buffers();
      return MSC_OK;
    });
  }

  int32_t recorded_steps() const override { return (int32_t)records.size(); }

  msc_status bdf2_adjoint(int32_t nsteps, double* lam, bool on_device) override {
    return guard([&]() -> msc_status {
      if (nsteps < 1 || nsteps > (int32_t)records.size()) {
        last_error = "nsteps must be between 1 and the number of recorded steps (" +
                     std::to_string(records.size()) + ")";
        return MSC_ERR_INVALID_ARG;
      }
      if (P.corrector == MSC_CORRECTOR_SHADOW && !fft_fits<double>()) {
        last_error = "the FP64 transforms of the adjoint correction do not fit this grid size";
        return MSC_ERR_UNSUPPORTED;
      }
      if (fullsym() || wallkin() || walls()) {
        last_error = "the adjoint covers the periodic Picard and shadow marches only";
        return MSC_ERR_UNSUPPORTED;
      }
      int kmax = 1;
      for (int r = 0; r < nsteps; ++r) kmax = std::max(kmax, records[records.size() - 1 - r].K);
      ensure_adjoint_buffers(kmax);
      if (on_device) after_default_stream();
      const int64_t SZ = state_size();
      // device memory of the caller is read by the first step and written by
      // the last, with the two buffers in between (a step's in and out differ)
      const double* cur = lam;
      if (!on_device) {
        MSC_HIPCK(hipMemcpyAsync(adj_lam[1], lam, sizeof(double) * SZ, hipMemcpyHostToDevice, st));
        cur = adj_lam[1];
      }
      for (int r = 0; r < nsteps; ++r) {
        double* nxt = (on_device && r > 0 && r == nsteps - 1) ? lam : adj_lam[r & 1];
        backward_step(records[records.size() - 1 - r], cur, nxt);
        cur = nxt;
      }
      if (cur != lam)
        MSC_HIPCK(hipMemcpyAsync(lam, cur, sizeof(double) * SZ,
                                 on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost, st));
      sync();
      records.resize(records.size() - nsteps);
      return MSC_OK;
    });
  }

  msc_status init_adjoint(const double* phat0, const double* u0, const double* lam, double* lam_phat0,
                          double* lam_u0, bool on_device) override {
    return guard([&]() -> msc_status {
      if (on_device) after_default_stream();
      const int64_t NS = G.NS, SZ = state_size();
      const double *pd = phat0, *ud = u0, *ld = lam;
      double *lp = lam_phat0, *lu = lam_u0;
      double* tmp = nullptr;
      if (!on_device) {
        tmp = (double*)dalloc(sizeof(double) * (SZ + 2 * (D + 1) * NS));
        double* t = tmp;
        MSC_HIPCK(hipMemcpyAsync(t, phat0, sizeof(double) * NS, hipMemcpyHostToDevice, st));
        MSC_HIPCK(hipMemcpyAsync(t + NS, u0, sizeof(double) * D * NS, hipMemcpyHostToDevice, st));
        MSC_HIPCK(hipMemcpyAsync(t + (D + 1) * NS, lam, sizeof(double) * SZ, hipMemcpyHostToDevice, st));
        pd = t;
        ud = t + NS;
        ld = t + (D + 1) * NS;
        lp = t + (D + 1) * NS + SZ;
        lu = lp + NS;
      }
      hipLaunchKernelGGL((k_adj_init<L>), dim3(ew_grid()), dim3(256), 0, st, NS, pd, ud, ld, lp, lu);
      MSC_HIPCK(hipGetLastError());
      if (!on_device) {
        MSC_HIPCK(hipMemcpyAsync(lam_phat0, lp, sizeof(double) * NS, hipMemcpyDeviceToHost, st));
        MSC_HIPCK(hipMemcpyAsync(lam_u0, lu, sizeof(double) * D * NS, hipMemcpyDeviceToHost, st));
      }
      sync();
      if (tmp) dfree(tmp);
      return MSC_OK;
    });
  }

  msc_status set_kernel_timing(int enable) override {
    return guard([&]() {
      sync();
      collect_timing();
      timing = enable != 0;
      for (int k = 0; k < 2; ++k) {
        t_sum[k] = 0.0;
        t_count[k] = 0;
        t_bytes[k] = 0.0;
      }
      return MSC_OK;
    });
  }

  msc_status kernel_time(int kind, double* seconds, int64_t* launches, double* bytes) override {
    return guard([&]() -> msc_status {
      if (kind < 0 || kind > 1) return MSC_ERR_INVALID_ARG;
      sync();
      collect_timing();
      if (seconds) *seconds = t_sum[kind];
      if (launches) *launches = t_count[kind];
      if (bytes) *bytes = t_count[kind] ? t_bytes[kind] / (double)t_count[kind] : sweep_bytes(kind == 1 ? SW_EXPLICIT : SW_DTS_LIFT);
      return MSC_OK;
    });
  }

 private:
  msc_params P;
  Geometry G;
  hipStream_t st;
  Tuning tune;
  double wp, wm, nu;

  FBufs<T> fb{};
  double* mb[3] = {nullptr, nullptr, nullptr};
  double* h = nullptr;
  // history term of odd physical steps (even steps use h): a setup sweep that
  // forms m^n from the previous step's h writes its own step's h meanwhile
  double* h_alt = nullptr;
  TM* Pr = nullptr;
  TM* dm = nullptr;
  cpx<CT>* spec = nullptr;
  cpx<CT>* spec2 = nullptr;
  cpx<CT>* spec_alt = nullptr;  // 2D: second band spectrum (inverse rows in the sweep)
  TM* rfs = nullptr;           // full symbol / wall corrector: residual of every field (Q x NS)
  // wall-bounded kinetic corrector (Algorithm 2): Krylov basis and work
  // vectors (FP64, Q x NS each), the moment spectra, the reference field of the
  // current operator and the assembly coefficient a_A, the state word with
  // the dot-product partials, and the cycle's bookkeeping
  double* wk_V = nullptr;
  double* wk_R = nullptr;
  double* wk_D = nullptr;
  double* wk_vc = nullptr;  // FP64 copy of the newest basis vector
  cpx<double>* wk_spec = nullptr;
  double* wk_mref = nullptr;
  double* wk_sref = nullptr;
  double* wk_part = nullptr;
  double* wk_part_h = nullptr;
  double* wk_coef = nullptr;
  double* wk_small = nullptr;
  // iterations enqueued before the host looks, by inner iteration: what that
  // inner iteration's solve took in the previous step
  static constexpr int kWallPred = 16;
  int wk_pred[kWallPred];
  int wk_m = 50;
  double wk_aA = 0.0;
  bool wk_rest = true;
  int64_t kr_solves = 0, kr_iters = 0, kr_refresh = 0;
  double kr_worst = 0.0;
  std::vector<int32_t> wall_refreshes;
  cpx<CT>* spec_fs = nullptr;  // full symbol: half spectrum (Q x N_x x (N_y/2 + 1))
  double* partials = nullptr;
  double* partials_h = nullptr;
  double* presum = nullptr;                   // folded partials for large sweep grids
  static constexpr int kFusedParts = 4096;    // decision kernels sum at most this many partials
  int nparts_cap = 0, nparts_h = 0;
  DevCtl* ctl = nullptr;
  DevCtl* ctl_h = nullptr;
  double* Rhist = nullptr;
  StepStat* stats_d = nullptr;  // of the current call
  StepStat* stats_h = nullptr;
  StepStat* stats_long = nullptr;
  std::vector<StepStat> stats_long_h;
  int stats_cap = 0;
  int32_t* sched_d = nullptr;
  int sched_cap = 0;
  std::vector<int32_t> sched_h, sched_host_view;
  int64_t sched_pos = 0;
  cpx<CT>* tw[3] = {nullptr, nullptr, nullptr};
  std::vector<cpx<CT>> tw_host[3];
  double* stage = nullptr;
  std::vector<void*> allocs;

  hipEvent_t order_ev = nullptr;  // see after_default_stream
  int n_next = 0;
  int64_t bdf_count = 0;
  bool lazy_history = false;  // complete_history has copies to make
  // physical steps enqueued before the next synchronisation: one where the
  // steps' counts are not to be expected from those before (a new state, a free
  // march behind a replay), twice as many after each accepted batch
  int batch = 1;
  bool replayed = false;  // the last march replayed a schedule
  int last_iters = 4;
  float sig = 1.0f;  // scale of FP16 deviation storage (unused otherwise)

  // Captured chunks of the explicit march, each with the arguments it holds by
  // value (buffers, chunk length, the deviation-storage scale).  Two: behind a
  // chunk an odd number of launches from one buffer to the other exchanges
  // them, so that calls of one length alternate between both orders.
  struct ExplicitGraph {
    hipGraphExec_t exec;
    hipGraph_t graph;
    const T* a;
    const T* b;  // null where the march is in place
    int chunk, kind;
    float sig;
  };
  ExplicitGraph graphs[2] = {};
  int graph_used = 0;  // the one used last

  // kernel timing
  bool timing = false;
  struct EvPair {
    hipEvent_t a, b;
    int kind;
    int flag;
    double bytes;
  };
  int* run_flags = nullptr;  // device, one per timed launch since the last collection
  int32_t* run_flags_h = nullptr;
  static constexpr int kFlagCap = 4096;
  double t_bytes[2] = {0, 0};
  std::vector<EvPair> ev_live;
  std::vector<hipEvent_t> ev_free;
  double t_sum[2] = {0, 0};
  int64_t t_count[2] = {0, 0};

  // adjoint records and buffers
  // A recorded step.  Each keeps f^n and h; the older populations of its trial
  // are f^n of the call's earlier records, and only a call's first records keep
  // their own (other entry points may change the state between calls).
  struct Record {
    std::shared_ptr<void> mem;  // the slab it lies in
    const T* f[3];              // f^n, f^{n-1}, f^{n-2} (storage format), null beyond the order
    const double* h;            // history term h_q
    int own;                    // how many of the last of these are its own (f^n always is)
    int64_t bc;                 // BDF steps accepted before this step
    int K;                      // inner sweeps at acceptance; 0 while the step is in flight
    float sig;                  // deviation-storage scale of the populations
  };
  // slab of the records being made: its next free byte and its end
  std::shared_ptr<void> slab;
  char* slab_at = nullptr;
  char* slab_end = nullptr;
  bool recording = false;
  std::vector<Record> records;
  std::vector<void*> adj_allocs;
  double* adj_lam[2] = {nullptr, nullptr};  // state-layout adjoints (in, out)
  double* adj_L[2] = {nullptr, nullptr};    // LF of the transposed sweeps in turn
  double* adj_lh = nullptr;
  // trial f^(1) and FP64 sweep outputs f_T of sweeps 1 .. K-1 of the step being
  // reversed, and their corrections dm of sweeps 1 .. K-1 or (adj_rows) the
  // solved band spectra of these, then of two transposed corrections
  double* adj_it = nullptr;
  double* adj_dm = nullptr;
  cpx<double>* adj_spec = nullptr;
  int adj_it_cap = 0, adj_dm_cap = 0, adj_spec_cap = 0;
  // FP64 transform buffers: P r of a recomputed sweep, or y = E^T Lambda, in
  // adj_y; z = Sh^T y out in adj_z
  double* adj_y = nullptr;
  double* adj_z = nullptr;
  XformBufs<double, double> adj_x{};

  // ------------------------------------------------------------- helpers --
  template <class F>
  msc_status guard(F&& fn) {
    if (broken) return MSC_ERR_STATE;
    try {
      return fn();
    } catch (const DeviceError& e) {
      broken = true;
      last_error = e.what;
      return MSC_ERR_DEVICE;
    } catch (const OomError&) {
      last_error = "device allocation failed";
      return MSC_ERR_OUT_OF_MEMORY;
    } catch (const std::bad_alloc&) {
      last_error = "host allocation failed";
      return MSC_ERR_OUT_OF_MEMORY;
    }
  }

  void sync() { MSC_HIPCK(hipStreamSynchronize(st)); }

  // A context without a caller's stream works on one of its own, which nothing
  // orders after the default stream, where such a caller's program fills the
  // tensors it passes and where memory that its allocator hands out again may
  // still be in use.  Called where device memory comes in from the caller.
  void after_default_stream() {
    if (P.stream) return;
    const hipError_t q = hipStreamQuery(nullptr);
    if (q == hipSuccess) return;
    (void)hipGetLastError();  // (not ready is no error here)
    if (!order_ev) MSC_HIPCK(hipEventCreateWithFlags(&order_ev, hipEventDisableTiming));
    MSC_HIPCK(hipEventRecord(order_ev, nullptr));
    MSC_HIPCK(hipStreamWaitEvent(st, order_ev, 0));
  }

  // (the failed call's error is not one of the launches that follow)
  [[noreturn]] static void out_of_memory() {
    (void)hipGetLastError();
    throw OomError{};
  }

  void* dalloc(size_t bytes) {
    void* p = nullptr;
    if (bytes == 0) bytes = 1;
    if (P.alloc_fn) {
      p = P.alloc_fn(bytes, P.alloc_user);
      if (!p) out_of_memory();
      after_default_stream();
    } else {
      hipError_t e = hipMalloc(&p, bytes);
      if (e == hipErrorOutOfMemory) out_of_memory();
      if (e != hipSuccess) throw DeviceError{e, std::string("hipMalloc: ") + hipGetErrorString(e)};
    }
    return p;
  }
  void dfree(void* p) {
    if (!p) return;
    if (P.alloc_fn) {
      if (P.free_fn) P.free_fn(p, P.alloc_user);
    } else {
      (void)hipFree(p);
    }
  }
  template <class X>
  X* keep(X* p) {
    allocs.push_back((void*)p);
    return p;
  }

  int ew_grid() const {
    const int64_t b = (G.NS + 255) / 256;
    return (int)std::min<int64_t>(std::max<int64_t>(b, 1), 4096);
  }

  bool corrector_supported() const { return fft_fits(); }

  bool fullsym() const { return P.corrector == MSC_CORRECTOR_FULL_SYMBOL; }
  // Shadow corrector with FP64 or FP32 populations, 3D or 2D with the row
  // transforms as passes of their own: the lift sweep enqueued as the last of
  // its step leaves P r out (the step is predicted to accept there);
  // k_recompute_pr forms it if the step goes on
  bool skip_pr_ok() const {
    return tune.skip_pr != 0 && P.corrector == MSC_CORRECTOR_SHADOW && !PopDev<T>::value &&
           (D == 3 || !fuse_rows);
  }
  bool wallkin() const { return P.corrector == MSC_CORRECTOR_WALL_KINETIC; }
  bool walls() const { return P.boundary == MSC_BOUNDARY_CAVITY; }
  bool wall_supported() const {
    return D == 2 && std::is_same<T, double>::value && walls() && P.tau_plus == 1.0 && P.tau_minus == 1.0 &&
           ilog2(G.N2) <= LineMax<double>::wall_rows && ilog2(G.N0) <= LineMax<double>::wall_cols;
  }
  bool fs_supported() const {
    return D == 2 && !DV && ilog2(G.N2) <= LineMax<CT>::fs_rows && ilog2(G.N0) <= LineMax<CT>::fs_cols;
  }

  // the shadow correction's passes, in the context's precision or (the
  // adjoint's) in FP64
  template <class CX = CT>
  bool fft_fits() const {
    if (D == 2) return ilog2(G.N2) <= LineMax<CX>::rows2 && ilog2(G.N0) <= LineMax<CX>::cols2;
    return ilog2(std::max(G.n[0], std::max(G.n[1], G.n[2]))) <= LineMax<CX>::line3;
  }

  // The context's buffers: the small ones share one device allocation (256-byte
  // aligned parts), because a context per solve is ordinary use and each
  // allocation is a call into the caller's allocator; the large ones have their
  // own, so that an allocator finds room for them in what it holds.
  static constexpr size_t kOwnBlock = (size_t)8 << 20;
  struct Part {
    void* p;  // the pointer to set
    size_t bytes;
  };
  void allocate() {
    const int64_t NS = G.NS;
    std::vector<Part> parts;
    auto want = [&](auto*& p, size_t bytes) { parts.push_back({&p, bytes}); };
    const size_t fields = sizeof(double) * (D + 1) * NS;
    want(h, fields);
    want(h_alt, fields);
    want(dm, sizeof(TM) * (D + 1) * NS);
    for (int i = 0; i < 5; ++i) want(fb.p[i], pop_bytes());
    for (int i = 0; i < 3; ++i) want(mb[i], fields);
    want(Pr, sizeof(TM) * (D + 1) * NS);
    want(ctl, kCtlBytes);
    want(Rhist, sizeof(double) * std::max(P.k_max, 1));
    want(presum, sizeof(double));
    choose_sweep();
    nparts_cap = std::max(sweep_grid_max(), 1024);
    want(partials, 2 * sizeof(double) * nparts_cap);
    const bool fs = (fullsym() || wallkin()) && fs_supported();
    bool axis[3] = {false, false, false};
    if (corrector_supported()) {
      if (D == 2) {
        const size_t bytes = sizeof(cpx<CT>) * 3 * Spec2<CT>::field(G.N0, G.N2 / 4 + 1);
        want(spec, bytes);
        want(spec_alt, bytes);
      } else {
        const int NBz = G.n[2] / 4 + 1, NBy = 2 * (G.n[1] / 4) + 1;
        want(spec, sizeof(cpx<CT>) * 4 * Spec3<CT>::field(G.n[0], G.n[1], NBz));
        want(spec2, sizeof(cpx<CT>) * 4 * Spec3<CT>::field(G.n[0], NBy, NBz));
        axis[1] = true;
      }
      axis[0] = axis[2] = true;
    }
    if (fs) {
      want(rfs, sizeof(TM) * (int64_t)Q * NS);
      if (fullsym()) want(spec_fs, sizeof(cpx<CT>) * Q * Spec2<CT>::field(G.N0, G.N2 / 2 + 1));
      axis[0] = axis[2] = true;
    }
    for (int i = 0; i < 3; ++i)
      if (axis[i]) {
        tw_host[i] = twiddle_tables<CT>(ilog2(i == 0 ? G.N0 : (i == 1 ? G.N1 : G.N2)));
        want(tw[i], sizeof(cpx<CT>) * tw_host[i].size());
      }
    if (wallkin() && wall_supported()) wall_parts(want);

    size_t total = 0;
    for (const Part& q : parts)
      if (q.bytes < kOwnBlock) total += (q.bytes + 255) / 256 * 256;
    char* base = keep((char*)dalloc(total));
    for (size_t i = 0; i < parts.size(); ++i) {
      const Part& q = parts[i];
      char* at = base;
      if (q.bytes < kOwnBlock)
        base += (q.bytes + 255) / 256 * 256;
      else
        at = keep((char*)dalloc(q.bytes));
      std::memcpy(q.p, &at, sizeof(at));
    }
    // the history terms and the correction start at zero (one fill where they
    // share the block)
    const size_t tmb = sizeof(TM) * (D + 1) * NS;
    if (fields < kOwnBlock) {
      MSC_HIPCK(hipMemsetAsync(h, 0, (char*)dm - (char*)h + tmb, st));
    } else {
      MSC_HIPCK(hipMemsetAsync(h, 0, fields, st));
      MSC_HIPCK(hipMemsetAsync(h_alt, 0, fields, st));
      MSC_HIPCK(hipMemsetAsync(dm, 0, tmb, st));
    }
    // (the host tables are kept until the copies are done: init waits)
    for (int i = 0; i < 3; ++i)
      if (axis[i])
        MSC_HIPCK(hipMemcpyAsync(tw[i], tw_host[i].data(), sizeof(cpx<CT>) * tw_host[i].size(),
                                 hipMemcpyHostToDevice, st));
    MSC_HIPCK(hipHostMalloc((void**)&ctl_h, kCtlBytes, hipHostMallocDefault));
    if (wallkin() && wall_supported())
      MSC_HIPCK(hipHostMalloc((void**)&wk_part_h, sizeof(double) * (1 + G.N0), hipHostMallocDefault));
  }

  void release() {
    for (auto& g : graphs) drop_graph(g);
    for (auto& e : ev_live) {
      (void)hipEventDestroy(e.a);
      (void)hipEventDestroy(e.b);
    }
    for (auto& e : ev_free) (void)hipEventDestroy(e);
    if (order_ev) (void)hipEventDestroy(order_ev);
    order_ev = nullptr;
    ev_live.clear();
    ev_free.clear();
    if (st) (void)hipStreamSynchronize(st);
    clear_records();
    for (void* p : adj_allocs) dfree(p);
    adj_allocs.clear();
    for (void* p : allocs) dfree(p);
    allocs.clear();
    if (ctl_h) (void)hipHostFree(ctl_h);
    if (partials_h) (void)hipHostFree(partials_h);
    if (run_flags_h) (void)hipHostFree(run_flags_h);
    run_flags_h = nullptr;
    if (wk_part_h) (void)hipHostFree(wk_part_h);
    wk_part_h = nullptr;
    ctl_h = nullptr;
    partials_h = nullptr;
  }

  // FP64 twiddle tables of the adjoint's transforms
  cpx<double>* adj_twiddles(int N) {
    const std::vector<cpx<double>> t = twiddle_tables<double>(ilog2(N));
    cpx<double>* d = (cpx<double>*)dalloc(sizeof(cpx<double>) * t.size());
    adj_allocs.push_back((void*)d);
    MSC_HIPCK(hipMemcpyAsync(d, t.data(), sizeof(cpx<double>) * t.size(), hipMemcpyHostToDevice, st));
    sync();  // t goes out of scope
    return d;
  }

  double* staging() {
    if (!stage) stage = keep((double*)dalloc(sizeof(double) * std::max<int64_t>(Q, 2 * (D + 1)) * G.NS));
    return stage;
  }

  void ensure_partials(int n) {
    if (n <= nparts_cap) return;
    partials = keep((double*)dalloc(2 * sizeof(double) * n));
    nparts_cap = n;
  }

  // pinned host memory for n partials (diagnostics and checks only)
  double* host_partials(int n) {
    if (n > nparts_h) {
      if (partials_h) (void)hipHostFree(partials_h);
      partials_h = nullptr;
      nparts_h = std::max(n, 1024);
      MSC_HIPCK(hipHostMalloc((void**)&partials_h, sizeof(double) * nparts_h, hipHostMallocDefault));
    }
    return partials_h;
  }

  // Step statistics: the first kInlineStats lie behind the control block, so
  // that one copy brings both; longer calls take buffers of their own.
  static constexpr int kInlineStats = 64;
  static constexpr size_t kCtlBytes = sizeof(DevCtl) + kInlineStats * sizeof(StepStat);
  void ensure_stats(int n) {
    if (n <= kInlineStats) {
      stats_d = reinterpret_cast<StepStat*>(ctl + 1);
      stats_h = reinterpret_cast<StepStat*>(ctl_h + 1);
      return;
    }
    if (n > stats_cap) {
      stats_long = keep((StepStat*)dalloc(sizeof(StepStat) * n));
      stats_long_h.resize(n);
      stats_cap = n;
    }
    stats_d = stats_long;
    stats_h = stats_long_h.data();
  }
  // the control block and, of a short call, its n steps' statistics; waits
  void fetch_ctl(int n) {
    const size_t more = n <= kInlineStats ? n * sizeof(StepStat) : 0;
    MSC_HIPCK(hipMemcpyAsync(ctl_h, ctl, sizeof(DevCtl) + more, hipMemcpyDeviceToHost, st));
    sync();
  }

  void ensure_sched(int n) {
    if (n <= sched_cap) return;
    sched_d = keep((int32_t*)dalloc(sizeof(int32_t) * n));
    sched_cap = n;
  }

  void copy_stats(msc_step_stats* out, int base, int count) {
    (void)base;
    if ((!out && !recording) || count <= 0) return;
    if (stats_d == stats_long) {
      MSC_HIPCK(hipMemcpyAsync(stats_h, stats_d, sizeof(StepStat) * count, hipMemcpyDeviceToHost, st));
      sync();
    }
    if (!out) return;
    for (int i = 0; i < count; ++i) {
      out[i].q = stats_h[i].q;
      out[i].iters = stats_h[i].iters;
      out[i].R_first = stats_h[i].R_first;
      out[i].R_final = stats_h[i].R_final;
      out[i].rho_obs = stats_h[i].rho_obs;
      out[i].converged = stats_h[i].converged;
      out[i].refreshes = (i < (int)wall_refreshes.size()) ? wall_refreshes[i] : 0;
    }
  }

  // Buffer roles of the next step to run.  Between calls the host's copy of the
  // control block equals the device's: every call that changes it ends with a
  // copy one way or the other.
  Roles& cur_roles() { return ctl_h->roles[n_next & 1]; }

  // m^n = P f^n and the BDF history reset (next step BDF1, whose trial uses
  // f^n alone): m^{n-1} = m^n, f^{n-1} = f^{n-2} = f^n, which are left to
  // complete_history, because the march never reads a state older than its
  // step count.  Returns sum f^2 (non-finite if a value is) where asked.
  double reset_history_from_current(bool check = false) {
    const T* f = fb.p[cur_roles().slot_hist[0]];
    const int grid = check ? 1024 : ew_grid();
    if (check) ensure_partials(grid);
    hipLaunchKernelGGL((k_moments<L, T>), dim3(grid), dim3(256), 0, st, f, mb[cur_roles().slot_m[0]], G.NS,
                       check ? partials : nullptr);
    MSC_HIPCK(hipGetLastError());
    bdf_count = 0;
    batch = 1;
    lazy_history = true;
    return check ? sum_partials_host(grid) : 0.0;
  }

  // The states older than the march's step count since the last reset.
  void complete_history() {
    if (!lazy_history) return;
    lazy_history = false;
    if (bdf_count >= 2) return;
    const Roles& ro = cur_roles();
    for (int i = (int)bdf_count + 1; i < 3; ++i)
      MSC_HIPCK(hipMemcpyAsync(fb.p[ro.slot_hist[i]], fb.p[ro.slot_hist[bdf_count]], pop_bytes(),
                               hipMemcpyDeviceToDevice, st));
    if (bdf_count == 0)
      MSC_HIPCK(hipMemcpyAsync(mb[ro.slot_m[1]], mb[ro.slot_m[0]], sizeof(double) * (D + 1) * G.NS,
                               hipMemcpyDeviceToDevice, st));
  }

  // bytes of one population buffer: Q N_sites values, plus the FP32 moments
  // of deviation storage
  size_t pop_bytes() const {
    return sizeof(T) * (size_t)Q * G.NS + (DV ? sizeof(float) * (size_t)(D + 1) * G.NS : 0);
  }

  void upload_pop(const double* f, T* dst) {
    double* stg = staging();
    const int64_t n = (int64_t)Q * G.NS;
    MSC_HIPCK(hipMemcpyAsync(stg, f, sizeof(double) * n, hipMemcpyHostToDevice, st));
    hipLaunchKernelGGL((k_pop_from_f64<L, T>), dim3(ew_grid()), dim3(256), 0, st, (const double*)stg, dst, G.NS,
                       1.0f / sig);
    MSC_HIPCK(hipGetLastError());
  }
  void download_pop(const T* src, double* f) {
    double* stg = staging();
    const int64_t n = (int64_t)Q * G.NS;
    hipLaunchKernelGGL((k_pop_to_f64<L, T>), dim3(ew_grid()), dim3(256), 0, st, src, stg, G.NS, sig);
    MSC_HIPCK(hipGetLastError());
    MSC_HIPCK(hipMemcpyAsync(f, stg, sizeof(double) * n, hipMemcpyDeviceToHost, st));
    sync();
  }
  void download_tm(const TM* src, double* out, int64_t n) {
    double* stg = staging();
    hipLaunchKernelGGL((k_convert<TM, double>), dim3(ew_grid()), dim3(256), 0, st, src, stg, n);
    MSC_HIPCK(hipGetLastError());
    MSC_HIPCK(hipMemcpyAsync(out, stg, sizeof(double) * n, hipMemcpyDeviceToHost, st));
    sync();
  }
  void upload_h(const double* h_in) {
    const int64_t n = (int64_t)(D + 1) * G.NS;
    if (h_in)
      MSC_HIPCK(hipMemcpyAsync(h, h_in, sizeof(double) * n, hipMemcpyHostToDevice, st));
    else
      MSC_HIPCK(hipMemsetAsync(h, 0, sizeof(double) * n, st));
  }

  // Scale of deviation storage: a power of two with |g| <= 2^12 for the
  // given populations (max deviation from equilibrium) and <= 2^10 times the
  // deviation over the largest moment (headroom for the march: a post-stream
  // deviation is a difference of neighbouring equilibria, a few times the
  // largest moment at most); FP16 overflows at 65504.
  static float choose_sigma(double maxdev, double maxm) {
    const double want = std::max(std::max(maxdev * 0x1p-12, maxm * 0x1p-10), 0x1p-100);
    return (float)std::exp2(std::ceil(std::log2(want)));
  }

  // Scale for populations uploaded from host FP64 arrays.
  float sigma_for(std::initializer_list<const double*> fs) {
    double md = 0.0, mm = 0.0;
    double* stg = staging();
    const int grid = 512;
    ensure_partials(2 * grid);
    for (const double* f : fs) {
      MSC_HIPCK(hipMemcpyAsync(stg, f, sizeof(double) * Q * G.NS, hipMemcpyHostToDevice, st));
      hipLaunchKernelGGL((k_pop_maxdev<L>), dim3(grid), dim3(256), 0, st, (const double*)stg, G.NS, partials);
      MSC_HIPCK(hipGetLastError());
      const double* ph = host_partials(2 * grid);
      MSC_HIPCK(hipMemcpyAsync((void*)ph, partials, sizeof(double) * 2 * grid, hipMemcpyDeviceToHost, st));
      sync();
      for (int i = 0; i < grid; ++i) {
        md = std::max(md, ph[2 * i]);
        mm = std::max(mm, ph[2 * i + 1]);
      }
    }
    return choose_sigma(md, mm);
  }

  double absmax(const double* v, int64_t n) {
    const int grid = 512;
    ensure_partials(grid);
    hipLaunchKernelGGL(k_absmax<0>, dim3(grid), dim3(256), 0, st, v, n, partials);
    MSC_HIPCK(hipGetLastError());
    const double* ph = host_partials(grid);
    MSC_HIPCK(hipMemcpyAsync((void*)ph, partials, sizeof(double) * grid, hipMemcpyDeviceToHost, st));
    sync();
    double m = 0.0;
    for (int i = 0; i < grid; ++i) m = std::max(m, ph[i]);
    return m;
  }

  // the first n partials' sum, in order
  double sum_partials_host(int n) {
    double* h = host_partials(n);
    MSC_HIPCK(hipMemcpyAsync(h, partials, sizeof(double) * n, hipMemcpyDeviceToHost, st));
    sync();
    double s = 0.0;
    for (int i = 0; i < n; ++i) s += h[i];
    return s;
  }

  double reduce_partials(const SweepArgs<T, TM>& S) {
    (void)S;
    return std::sqrt(sum_partials_host(sweep_grid()) / ((double)Q * (double)G.NS));
  }

  // ------------------------------------------------------ adjoint pieces --
  // Records for the steps n0 .. n0 + B - 1 (bc0 accepted steps before the first)
  // of the call that began at step base, made before any of them is enqueued;
  // how many have one (fewer than B, or none, where the memory ends).  A step
  // enqueued again, because the march had not reached it, has its record.
  int reserve_records(int n0, int64_t bc0, int B, int base, int remaining) {
    const int max_order = (P.extrap_states == 0) ? 2 : P.extrap_states - 1;
    for (int i = 0; i < B; ++i) {
      const size_t idx = rec_base + (size_t)(n0 + i - base);
      if (idx < records.size()) continue;
      try {
        make_record(bc0 + i, (int)std::min<int64_t>(bc0 + i, max_order), remaining - i);
      } catch (const OomError&) {
        return i;
      } catch (const std::bad_alloc&) {
        return i;
      }
    }
    return B;
  }

  // older populations that the record of a trial of that order keeps itself:
  // the others are f^n of the call's earlier records
  int own_populations(size_t idx, int order) const {
    return std::max(order - (int)std::min<size_t>(idx - rec_base, 2), 0);
  }

  // The next record of the list, in a slab with room for it: for up to 32 of
  // the call's remaining steps, or for as many fewer as there is memory.
  void make_record(int64_t bc, int order, int remaining) {
    const size_t fq = pop_bytes(), fm = sizeof(double) * (size_t)(D + 1) * G.NS;
    const size_t idx = records.size();
    const int own = own_populations(idx, order);
    const size_t need = fm + (size_t)(1 + own) * fq;
    if (!slab || slab_at + need > slab_end) {
      for (int steps = std::min(remaining, 32);; steps /= 2) {
        // (a call's second record may keep an older population as well)
        const size_t bytes = need + (size_t)(steps - 1) * (fm + fq) + (steps > 1 && idx == rec_base ? fq : 0);
        try {
          slab = std::shared_ptr<void>(dalloc(bytes), [this](void* p) { dfree(p); });
        } catch (const OomError&) {
          if (steps == 1) throw;
          continue;
        }
        slab_at = (char*)slab.get();
        slab_end = slab_at + bytes;
        break;
      }
    }
    Record r{};
    r.mem = slab;
    char* at = slab_at;
    auto take = [&](size_t bytes) {
      char* p = at;
      at += bytes;
      return p;
    };
    for (int i = 0; i <= order; ++i) {
      if (i == 0 || i > order - own)
        r.f[i] = (const T*)take(fq);
      else
        r.f[i] = records[idx - 1].f[i - 1];
    }
    r.own = own;
    r.h = (const double*)take(fm);
    r.bc = bc;
    r.sig = sig;
    records.push_back(std::move(r));
    slab_at = at;
  }

  // Arguments of the copy into the record of step n, the idx-th in the list.
  CkptArgs<T> checkpoint_args(int n, size_t idx) {
    const Record& r = records[idx];
    CkptArgs<T> A{};
    A.ctl = ctl;
    A.n = n;
    A.fb = fb;
    A.h = h_of(n);
    const int last = r.f[2] ? 2 : (r.f[1] ? 1 : 0);
    for (int i = 0; i <= last; ++i)
      if (i == 0 || i > last - r.own) A.rf[i] = (uint4*)r.f[i];
    A.rh = (uint4*)r.h;
    A.nf = (int64_t)(pop_bytes() / sizeof(uint4));
    A.nh = (int64_t)(sizeof(double) * (size_t)(D + 1) * G.NS / sizeof(uint4));
    return A;
  }

  // The records that one call makes: those of accepted steps stay.
  size_t rec_base = 0;
  struct RecordScope {
    Solver& s;
    const size_t base;
    size_t kept = 0;
    explicit RecordScope(Solver& s_) : s(s_), base(s_.records.size()) { s.rec_base = base; }
    void accept(int n) {
      if (!s.recording) return;
      for (int i = 0; i < n; ++i) s.records[base + i].K = s.stats_h[i].iters;
      kept = n;
    }
    ~RecordScope() {
      if (s.records.size() > base + kept) {
        (void)hipStreamSynchronize(s.st);  // work that writes them
        s.records.resize(base + kept);
      }
      s.slab.reset();
      s.slab_at = s.slab_end = nullptr;
    }
  };

  void clear_records() {
    records.clear();
    slab.reset();
  }

  void free_adjoint_buffers() {
    for (void* p : adj_allocs) dfree(p);
    adj_allocs.clear();
    for (int i = 0; i < 2; ++i) adj_lam[i] = adj_L[i] = nullptr;
    adj_lh = adj_it = adj_dm = adj_y = adj_z = nullptr;
    adj_spec = nullptr;
    adj_it_cap = adj_dm_cap = adj_spec_cap = 0;
    adj_x = XformBufs<double, double>{};
  }

  // 2D: the transposed sweep with its row transforms (k_adj_rows), on the grids
  // whose forward sweeps do theirs
  bool adj_rows() const { return D == 2 && fuse_inv; }

  void ensure_adjoint_buffers(int K) {
    const int64_t NS = G.NS, FQ = (int64_t)Q * NS, FM = (int64_t)(D + 1) * NS;
    using C2 = cpx<double>;
    auto get = [&](size_t bytes) {
      void* p = dalloc(bytes);
      adj_allocs.push_back(p);
      return p;
    };
    const bool shadow = P.corrector == MSC_CORRECTOR_SHADOW;
    const size_t band = 3 * (size_t)Spec2<double>::field(G.N0, G.N2 / 4 + 1);
    if (!adj_lh) {
      for (int i = 0; i < 2; ++i) adj_lam[i] = (double*)get(sizeof(double) * state_size());
      for (int i = 0; i < 2; ++i) adj_L[i] = (double*)get(sizeof(double) * FQ);
      adj_y = (double*)get(sizeof(double) * FM);
      adj_z = (double*)get(sizeof(double) * FM);
      if (shadow) {
        adj_x.in = adj_y;
        adj_x.out = adj_z;
        if constexpr (std::is_same<CT, double>::value) {
          adj_x.spec1 = spec;
          adj_x.spec2 = spec2;
          for (int i = 0; i < 3; ++i) adj_x.tw[i] = tw[i];
        } else if (D == 2) {
          adj_x.spec1 = (C2*)get(sizeof(C2) * band);
          adj_x.tw[0] = adj_twiddles(G.N0);
          adj_x.tw[2] = adj_twiddles(G.N2);
        } else {
          const int NBz = G.n[2] / 4 + 1, NBy = 2 * (G.n[1] / 4) + 1;
          adj_x.spec1 = (C2*)get(sizeof(C2) * 4 * (size_t)Spec3<double>::field(G.n[0], G.n[1], NBz));
          adj_x.spec2 = (C2*)get(sizeof(C2) * 4 * (size_t)Spec3<double>::field(G.n[0], NBy, NBz));
          for (int a = 0; a < 3; ++a) adj_x.tw[a] = adj_twiddles(G.n[a]);
        }
      }
      adj_lh = (double*)get(sizeof(double) * FM);
    }
    if (K > adj_it_cap) {
      adj_it = (double*)get(sizeof(double) * FQ * (size_t)K);
      adj_it_cap = K;
    }
    if (shadow && adj_rows() && K > adj_spec_cap) {
      adj_spec = (C2*)get(sizeof(C2) * band * (size_t)(K + 1));
      adj_spec_cap = K;
    }
    if (shadow && !adj_rows() && K > adj_dm_cap) {
      adj_dm = (double*)get(sizeof(double) * FM * (size_t)K);
      adj_dm_cap = K;
    }
  }

  // FP64 dual-time sweep number ell of the step being reversed (diagnostic mode,
  // no control block), from the iterate that it lifts to its output f_T; P r
  // into adj_y, or its row spectrum into the correction's (adj_rows).
  void sweep64(int ell, const double* src, double* dst, const double* h64, double a) {
    const bool shadow = P.corrector == MSC_CORRECTOR_SHADOW, rows = shadow && adj_rows();
    SweepArgs<double, double> S{};
    const int mode = (!shadow || ell == 1) ? SW_DTS : (rows ? SW_DTS_LIFT_ROWS : SW_DTS_LIFT);
    S.N0 = G.N0;
    S.N1 = G.N1;
    S.N2 = G.N2;
    S.L = strip_L;
    const TileCfg tm = tile_of(mode);
    S.ntile1 = G.N1 / tm.T1;
    S.ntile2 = G.N2 / tm.T2;
    S.nstrip = G.N0 / strip_L;
    S.NS = G.NS;
    S.ctl = nullptr;
    S.src = src;
    S.dst = dst;
    S.h = const_cast<double*>(h64);  // read in these modes
    S.dm = (mode == SW_DTS_LIFT) ? adj_dm_of(ell - 1) : nullptr;
    S.Pr = adj_y;
    S.partials = partials;
    S.a = a;
    S.inv1pa2 = 1.0 / (1.0 + a / 2.0);
    S.wp = wp;
    S.wm = wm;
    if (rows) {
      S.fuse_rows = 1;
      S.NBr = G.N2 / 4 + 1;
      S.spec = adj_spec_of(ell);
      S.twr = adj_x.tw[2];
      if (mode == SW_DTS_LIFT_ROWS) S.spec_in = adj_spec_of(ell - 1);
    }
    if (D == 2)
      launch_sweep_d2<double, double>(tile_id, mode, S, sweep_grid(mode), st);
    else if (wide_mode(mode))
      launch_sweep_dual_wide<double, double>(mode, S, sweep_grid(mode), st);
    else
      launch_sweep_d3<double, double>(tile_id, mode, S, sweep_grid(mode), st);
    MSC_HIPCK(hipGetLastError());
  }

  // dm, or its solved band spectrum, of recomputed sweep ell = 1 .. K-1; spectra
  // of the transposed corrections in the two after sweep adj_spec_cap - 1
  double* adj_dm_of(int ell) const { return adj_dm + (size_t)(ell - 1) * (D + 1) * G.NS; }
  cpx<double>* adj_spec_of(int ell) const {
    return adj_spec + (size_t)(ell - 1) * 3 * Spec2<double>::field(G.N0, G.N2 / 4 + 1);
  }
  cpx<double>* adj_zspec_of(int ell) const { return adj_spec_of(adj_spec_cap + (ell & 1)); }

  // Reverse one recorded step: recompute its inner iterates from the record,
  // then run the transposed stages from the last sweep to the first and through
  // the history combination.  lin is the adjoint of the state after the step,
  // lout (another buffer) receives the adjoint of the state before it.
  //
  // A sweep and its correction take two launches each way on the grids of
  // adj_rows (sweep with row transforms, column pass), else a sweep and the
  // transform's passes.  N = 256, two inner iterations: 46 us of kernels in 6
  // launches per step, from 100 us in 15 when lift, E^T, P^T and the history
  // combination were launches of their own (each field written and read again
  // between them) and the row transforms too.
  void backward_step(const Record& R, const double* lin, double* lout) {
    const int64_t NS = G.NS, FQ = (int64_t)Q * NS, FM = (int64_t)(D + 1) * NS;
    const bool shadow = (P.corrector == MSC_CORRECTOR_SHADOW), rows = shadow && adj_rows();
    const int q = (R.bc == 0) ? 1 : 2;
    const int max_order = (P.extrap_states == 0) ? 2 : P.extrap_states - 1;
    const int order = (int)std::min<int64_t>(R.bc, max_order);
    const double a = (q == 1) ? 1.0 / P.dt : 3.0 / (2.0 * P.dt);
    const int K = R.K;
    auto it = [&](int ell) { return adj_it + (size_t)(ell - 1) * FQ; };
    const int eg = ew_grid();

    // forward recompute in FP64: it(1) the trial, it(ell + 1) = f_T of sweep ell
    hipLaunchKernelGGL((k_adj_trial<L, T>), dim3(eg), dim3(256), 0, st, NS, order, R.f[0], R.f[1], R.f[2], R.sig,
                       it(1));
    MSC_HIPCK(hipGetLastError());
    XformBufs<double, double> B = adj_x;
    for (int ell = 1; ell < K; ++ell) {
      sweep64(ell, it(ell), it(ell + 1), R.h, a);
      if (!shadow) continue;
      if (rows)
        B.spec1 = adj_spec_of(ell);
      else
        B.out = adj_dm_of(ell);
      enqueue_transform<double, double>(nullptr, 0, 0, a, nullptr, false, B, nullptr, rows, rows);
    }

    // backward through the inner iterations
    AdjArgs A{};
    A.g = AdjGeom{G.N0, G.N1, G.N2, NS};
    A.h = R.h;
    A.Lt = lin;
    A.zt = lin + 3 * FQ;
    A.zscale = 1.0 / (1.0 + a / 2.0);
    A.seed = 1;
    A.y = shadow ? adj_y : nullptr;
    A.lam_h = adj_lh;
    A.a = a;
    A.wp = wp;
    A.wm = wm;
    A.order = order;
    A.q = q;
    A.dt = P.dt;
    A.lf1n = lin + FQ;
    A.lf2n = lin + 2 * FQ;
    A.lm1n = lin + 3 * FQ + FM;
    A.of0 = lout;
    A.of1 = lout + FQ;
    A.of2 = lout + 2 * FQ;
    A.om0 = lout + 3 * FQ;
    A.om1 = lout + 3 * FQ + FM;
    A.twy = adj_x.tw[2];
    B = adj_x;
    for (int ell = K; ell >= 1; --ell) {
      A.fin = it(ell);
      A.LF = adj_L[ell & 1];
      A.last = (ell == 1) ? 1 : 0;
      if (rows) {
        A.dm_spec = (ell > 1) ? adj_spec_of(ell - 1) : nullptr;
        A.y_spec = adj_zspec_of(ell);
        if constexpr (D == 2)
          with_lg<2, 8>(ilog2(G.N2), [&](auto lg) {
            constexpr int T2 = 1 << lg.value;
            hipLaunchKernelGGL((k_adj_rows<T2>), dim3(G.N0), dim3(adj_rows_threads(T2)), 0, st, A);
          });
      } else {
        A.dm = (shadow && ell > 1) ? adj_dm_of(ell - 1) : nullptr;
        hipLaunchKernelGGL((k_adj_sweep<L>), dim3(eg), dim3(256), 0, st, A);
      }
      MSC_HIPCK(hipGetLastError());
      if (ell == 1) break;
      A.Lt = A.LF;
      A.zt = nullptr;
      A.zscale = 1.0;
      A.seed = 0;
      if (!shadow) continue;
      B.spec1 = rows ? adj_zspec_of(ell) : adj_x.spec1;
      enqueue_transform<double, double>(nullptr, 0, 0, a, nullptr, true, B, nullptr, rows, rows);
      if (rows)
        A.z_spec = B.spec1;
      else
        A.zt = adj_z;
    }
  }

  // ------------------------------------------------------ sweep config --
  int tile_id = 0, strip_L = 1;
  bool wide_dual = false;  // dual-time sweeps after the first of a step on kWideDualTile3
  int strip_setup = 1;     // planes per strip of the first sweep of a step
  int strip_explicit = 1;  // planes per strip of the tiled explicit sweep
  TileCfg tile{};
  // 2D with the shadow corrector and tiles spanning whole rows: the sweep
  // also does the forward row transform of P r
  bool fuse_rows = false;
  // ... and the inverse row transform before the lift (one-plane strips): the
  // correction's spectrum then alternates between spec and spec_alt
  bool fuse_inv = false;

  void choose_sweep() {
    const int n = TileSet<L>::count;
    int best = -1;
    if (tune.sweep_tile_index > 0 && tune.sweep_tile_index <= n) {
      const TileCfg t = TileSet<L>::get(tune.sweep_tile_index - 1);
      if (t.T1 <= G.N1 && t.T2 <= G.N2) best = tune.sweep_tile_index - 1;
    }
    if (best < 0 && tune.sweep_tile > 0) {
      for (int i = 0; i < n; ++i) {
        const TileCfg t = TileSet<L>::get(i);
        if (t.T1 * t.T2 == tune.sweep_tile && t.T1 <= G.N1 && t.T2 <= G.N2) best = i;
      }
    }
    if (best < 0) best = auto_sweep_tile<L>(G.N1, G.N2);
    tile_id = best;
    tile = TileSet<L>::get(best);
    wide_dual = D == 3 && tune.wide_dual && tile.T1 == 2 && tile.T2 == 128 && G.N2 == 128 && G.N1 >= 4;
    strip_L = wide_dual ? sweep_strip_for<L, T>(kWideDualTile3, G.N0, G.N1, G.N2, tune.sweep_strip, STRIP_DUAL_WIDE)
                        : sweep_strip_for<L, T>(tile, G.N0, G.N1, G.N2, tune.sweep_strip, STRIP_DUAL);
    strip_setup = sweep_strip_for<L, T>(tile, G.N0, G.N1, G.N2, tune.sweep_strip, STRIP_SETUP);
    strip_explicit = sweep_strip_for<L, T>(tile, G.N0, G.N1, G.N2, tune.sweep_strip, STRIP_EXPLICIT);
    fuse_rows = D == 2 && P.corrector == MSC_CORRECTOR_SHADOW && tile.T1 == 1 && tile.T2 == G.N2 &&
                tile.NT == tile.T2 && corrector_supported() && tune.fuse_rows != 0;
    fuse_inv = fuse_rows && strip_L == 1 && tune.fuse_rows >= 2;
  }

  int strip_of(int mode) const {
    return (mode == SW_DTS_SETUP) ? strip_setup : (mode == SW_EXPLICIT ? strip_explicit : strip_L);
  }
  bool wide_mode(int mode) const { return wide_dual && (mode == SW_DTS || mode == SW_DTS_LIFT); }
  TileCfg tile_of(int mode) const { return wide_mode(mode) ? kWideDualTile3 : tile; }
  int sweep_grid(int mode = SW_DTS) const {
    const TileCfg t = tile_of(mode);
    return (int)((int64_t)(G.N1 / t.T1) * (G.N2 / t.T2) * (G.N0 / strip_of(mode)));
  }
  int sweep_grid_max() const {
    return std::max({sweep_grid(), sweep_grid(SW_DTS_SETUP), sweep_grid(SW_EXPLICIT)});
  }

  SweepArgs<T, TM> sweep_args(double a) {
    SweepArgs<T, TM> S{};
    S.N0 = G.N0;
    S.N1 = G.N1;
    S.N2 = G.N2;
    S.L = strip_L;
    S.ntile1 = G.N1 / tile.T1;
    S.ntile2 = G.N2 / tile.T2;
    S.nstrip = G.N0 / strip_L;
    S.NS = G.NS;
    S.ctl = nullptr;
    S.fb = fb;
    S.h = h;
    S.dm = dm;
    S.Pr = Pr;
    S.partials = partials;
    S.a = a;
    S.inv1pa2 = 1.0 / (1.0 + a / 2.0);
    S.wp = wp;
    S.wm = wm;
    S.sig = sig;
    S.isig = 1.0f / sig;
    S.walls = walls() ? 1 : 0;
    S.ulid = P.u_lid;
    return S;
  }

  // algorithmic bytes per sweep launch (one read and one write of the
  // populations, plus h, dm in, P r out for the dual-time sweep)
  // algorithmic HBM bytes of one sweep launch: populations read once per
  // history state used and written once; h read (or, in setup mode, m^n and
  // m^{n-1} read and h written); the lift input and P r output
  double sweep_bytes(int mode, int order = 0, int q = 1) const {
    const double NS = (double)G.NS;
    const double fb1 = (double)pop_bytes(), mb1 = (double)(D + 1) * NS;
    if (mode == SW_EXPLICIT) return 2.0 * fb1;
    double b = 2.0 * fb1 + mb1 * sizeof(TM);  // f in, f_T out, P r out
    if (fullsym()) b += (double)(Q - D - 1) * NS * sizeof(TM);  // r of every field instead of P r
    if (fuse_rows && (lift_mode(mode) || mode == SW_DTS_SETUP))  // row spectrum out instead of P r
      b += (double)(D + 1) * G.N0 * (G.N2 / 4 + 1) * sizeof(cpx<TM>) - mb1 * sizeof(TM);
    if (mode == SW_DTS_SETUP)
      b += order * fb1 + mb1 * sizeof(double) * (q == 2 ? 3.0 : 2.0);
    else
      b += mb1 * sizeof(double);
    if (mode == SW_DTS_LIFT) b += mb1 * sizeof(TM);
    if (mode == SW_DTS_LIFT_ROWS)  // the band spectrum rows in instead of dm
      b += (double)(D + 1) * G.N0 * (G.N2 / 4 + 1) * sizeof(cpx<TM>);
    return b;
  }

  hipEvent_t get_event() {
    if (!ev_free.empty()) {
      hipEvent_t e = ev_free.back();
      ev_free.pop_back();
      return e;
    }
    hipEvent_t e;
    MSC_HIPCK(hipEventCreate(&e));
    return e;
  }

  void collect_timing() {
    if (ev_live.empty()) return;
    MSC_HIPCK(hipMemcpyAsync(run_flags_h, run_flags, sizeof(int) * ev_live.size(), hipMemcpyDeviceToHost, st));
    sync();
    for (auto& e : ev_live) {
      if (run_flags_h[e.flag]) {
        float ms = 0.f;
        MSC_HIPCK(hipEventElapsedTime(&ms, e.a, e.b));
        t_sum[e.kind] += 1e-3 * ms;
        t_count[e.kind] += 1;
        t_bytes[e.kind] += e.bytes;
      }
      ev_free.push_back(e.a);
      ev_free.push_back(e.b);
    }
    ev_live.clear();
    MSC_HIPCK(hipMemsetAsync(run_flags, 0, sizeof(int) * kFlagCap, st));
    sync();
  }

  // events and run flag of one timed launch (kind 0: dual-time sweep, 1:
  // explicit march)
  EvPair timed_pair(int kind, double bytes) {
    if (!run_flags) {
      run_flags = keep((int*)dalloc(sizeof(int) * kFlagCap));
      MSC_HIPCK(hipHostMalloc((void**)&run_flags_h, sizeof(int) * kFlagCap, hipHostMallocDefault));
      MSC_HIPCK(hipMemsetAsync(run_flags, 0, sizeof(int) * kFlagCap, st));
    }
    EvPair ep{};
    ep.a = get_event();
    ep.b = get_event();
    ep.kind = kind;
    ep.flag = (int)ev_live.size();
    ep.bytes = bytes;
    return ep;
  }

  void launch_sweep_timed(int mode, SweepArgs<T, TM> S, int kind) {
    EvPair ep{};
    (void)kind;
    if (timing) {
      ep = timed_pair((mode == SW_EXPLICIT) ? 1 : 0,
                      sweep_bytes(mode, S.order, S.q) - (S.skip_pr ? (double)(D + 1) * G.NS * sizeof(TM) : 0.0) +
                          ((mode == SW_DTS_SETUP && S.recon) ? (double)(D + 1) * G.NS * 8.0 : 0.0));
      S.did_run = run_flags + ep.flag;
    }
    S.L = strip_of(mode);
    S.nstrip = G.N0 / S.L;
    const TileCfg tm = tile_of(mode);
    S.ntile1 = G.N1 / tm.T1;
    S.ntile2 = G.N2 / tm.T2;
    if (D == 2)
      launch_sweep_d2<T, TM>(tile_id, mode, S, sweep_grid(mode), st, timing ? ep.a : nullptr, timing ? ep.b : nullptr);
    else if (wide_mode(mode))
      launch_sweep_dual_wide<T, TM>(mode, S, sweep_grid(mode), st, timing ? ep.a : nullptr, timing ? ep.b : nullptr);
    else
      launch_sweep_d3<T, TM>(tile_id, mode, S, sweep_grid(mode), st, timing ? ep.a : nullptr, timing ? ep.b : nullptr);
    MSC_HIPCK(hipGetLastError());
    if (timing) {
      ev_live.push_back(ep);
      if ((int)ev_live.size() >= kFlagCap) collect_timing();
    }
  }

  static void drop_graph(ExplicitGraph& g) {
    if (g.exec) (void)hipGraphExecDestroy(g.exec);
    if (g.graph) (void)hipGraphDestroy(g.graph);
    g = ExplicitGraph{};
  }

  hipGraphExec_t explicit_graph(T* A, T* B, int chunk, int kind) {
    const T* other = kind == EX_AA ? nullptr : B;
    for (int i = 0; i < 2; ++i) {
      const ExplicitGraph& g = graphs[i];
      if (g.exec && g.a == A && g.b == other && g.chunk == chunk && g.sig == sig && g.kind == kind) {
        graph_used = i;
        return g.exec;
      }
    }
    graph_used ^= 1;
    ExplicitGraph& g = graphs[graph_used];
    drop_graph(g);
    sync();
    MSC_HIPCK(hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal));
    SweepArgs<T, TM> S = sweep_args(0.0);
    S.L = strip_explicit;
    S.nstrip = G.N0 / strip_explicit;
    if (kind == EX_MULTI) {
      // an even number of launches: the chunk ends in A
      const int nl = chunk / march2_steps(march2_tile());
      for (int i = 0; i < nl; ++i) launch_march2((i & 1) ? B : A, (i & 1) ? A : B);
    }
    for (int i = 0; kind != EX_MULTI && i < chunk; ++i) {
      if (kind == EX_AA) {
        launch_aa(A, (i & 1) != 0);
        continue;
      }
      S.src = (i & 1) ? B : A;
      S.dst = (i & 1) ? A : B;
      if (D == 2)
        launch_sweep_d2<T, TM>(tile_id, SW_EXPLICIT, S, sweep_grid(SW_EXPLICIT), st);
      else
        launch_sweep_d3<T, TM>(tile_id, SW_EXPLICIT, S, sweep_grid(SW_EXPLICIT), st);
    }
    MSC_HIPCK(hipStreamEndCapture(st, &g.graph));
    MSC_HIPCK(hipGraphInstantiate(&g.exec, g.graph, nullptr, nullptr, 0));
    g.a = A;
    g.b = other;
    g.chunk = chunk;
    g.sig = sig;
    g.kind = kind;
    return g.exec;
  }

  // --------------------------------------------------- Algorithm 1 pieces --
  // One inner iteration of Algorithm 1 for (step n, sweep ell), guarded on the
  // device: the sweep (the first one of a step also forms h_q and the
  // extrapolated trial), then one grid whose blocks all take the acceptance
  // decision, and which goes on with the reconstruction of m^{n+1} (accepted) or
  // the correction's first pass, and the correction's other passes.
  // last: the final iteration enqueued for this step; its correction is left
  // out (it runs only if the step goes on, and then enqueue_correction_tail
  // supplies it before the next sweep).
  // recon: this step's setup sweep forms m^n (the previous step, coefficient
  // a_prev, left it); defer: this step's acceptance leaves m^{n+1} to the
  // next step's setup sweep.
  void enqueue_iteration(int n, int ell, int q, int order, double a, bool use_sched, int stat_base,
                         bool last = false, bool recon = false, double a_prev = 0.0, bool defer = false,
                         const CkptArgs<T>* rec = nullptr, bool hand_on = false) {
    SweepArgs<T, TM> S = sweep_args(a);
    S.ctl = ctl;
    S.h = h_of(n);
    S.recon = (ell == 1 && recon) ? 1 : 0;
    S.h_prev = h_of(n - 1);
    S.a_prev = a_prev;
    S.inv1pa2_prev = 1.0 / (1.0 + a_prev / 2.0);
    S.inv_dt = 1.0 / P.dt;
    S.inv_2dt = 1.0 / (2.0 * P.dt);
    S.n = n;
    S.ell = ell;
    for (int i = 0; i < 3; ++i) S.mb[i] = mb[i];
    S.q = q;
    S.order = order;
    S.dt = P.dt;
    FinishArgs F{};
    F.ctl = ctl;
    F.n = n;
    F.ell = ell;
    F.inv_count = 1.0 / ((double)Q * (double)G.NS);
    F.eps = P.eps;
    F.nmin = P.n_min;
    F.kmax = P.k_max;
    F.q = q;
    F.mcap = (D == 2) ? 10 : 8;
    F.sched = use_sched ? sched_d : nullptr;
    F.Rhist = Rhist;
    F.stats = stats_d;
    F.stat_base = stat_base;
    F.partials = S.partials = parts_of(n);
    int mode;
    if (ell == 1)
      mode = SW_DTS_SETUP;
    else if (P.corrector == MSC_CORRECTOR_SHADOW)
      mode = fuse_inv ? SW_DTS_LIFT_ROWS : SW_DTS_LIFT;
    else
      mode = SW_DTS;
    F.nparts = sweep_grid(mode);
    if (fullsym() || wallkin()) S.rout = rfs;
    const bool skip_pr = skip_pr_ok() && last && mode == SW_DTS_LIFT;
    S.skip_pr = skip_pr ? 1 : 0;
    if (fuse_rows) {
      S.fuse_rows = 1;
      S.NBr = G.N2 / 4 + 1;
      S.spec = spec_of(ell);
      S.twr = tw[2];
      if (mode == SW_DTS_LIFT_ROWS) S.spec_in = spec_of(ell - 1);
    }
    if (ell == 1 && handed_on.n == n - 1 && handed_on.ctl) {
      S.merge = 1;
      S.fin = handed_on;
    }
    handed_on.ctl = nullptr;
    launch_sweep_timed(mode, S, 0);
    if (rec && ell == 1) {
      hipLaunchKernelGGL((k_checkpoint<T>), dim3(ew_grid()), dim3(256), 0, st, *rec);
      MSC_HIPCK(hipGetLastError());
    }
    if (last && hand_on) {
      handed_on = F;
      return;
    }
    if (F.nparts > kFusedParts) {
      // many sweep blocks: fold the partials once instead of in every block
      hipLaunchKernelGGL(k_presum<0>, dim3(1), dim3(256), 0, st, F.partials, F.nparts, presum);
      MSC_HIPCK(hipGetLastError());
      F.partials = presum;
      F.nparts = 1;
    }

    AcceptArgs<L, T> Ac = accept_args(n, ell, a);
    Ac.defer = defer ? 1 : 0;
    if (P.corrector == MSC_CORRECTOR_SHADOW && !last) {
      XformBufs<CT, TM> B{Pr, dm, spec_of(ell), spec2, {tw[0], tw[1], tw[2]}};
      enqueue_transform<CT, TM>(ctl, n, ell, a, &Ac, false, B, &F, fuse_rows, fuse_inv);
    } else if (fullsym()) {
      enqueue_fullsym(ctl, n, ell, a, &Ac, &F, true, !last, nullptr);
    } else {
      // the decision alone (without the shadow corrector, and for the sweep
      // enqueued last for its step, which is predicted to end it); one block
      // unless an accepted step is to be reconstructed here
      hipLaunchKernelGGL((k_accept<L, T>), dim3(defer ? 1 : ew_grid()), dim3(256), 0, st, Ac, F);
      MSC_HIPCK(hipGetLastError());
    }
  }

  // The correction of (step n, sweep ell), the sweep enqueued last for its
  // step, guarded on the device (it runs only if that sweep was not accepted;
  // the decision was taken).
  void enqueue_correction_tail(int n, int ell, double a) {
    if (fullsym()) {
      enqueue_fullsym(ctl, n, ell, a, nullptr, nullptr, false, true, nullptr);
      return;
    }
    if (P.corrector != MSC_CORRECTOR_SHADOW) return;
    XformBufs<CT, TM> B{Pr, dm, spec_of(ell), spec2, {tw[0], tw[1], tw[2]}};
    if constexpr (!PopDev<T>::value) {
      // a lift sweep enqueued last left P r out: form it
      if (skip_pr_ok() && ell >= 2) {
        PrArgs<T, TM> R{ctl, n, ell, fb, dm, Pr, G.NS};
        hipLaunchKernelGGL((k_recompute_pr<L, T, TM>), dim3(ew_grid()), dim3(256), 0, st, R);
        MSC_HIPCK(hipGetLastError());
      }
    }
    enqueue_transform<CT, TM>(ctl, n, ell, a, nullptr, false, B, nullptr, fuse_rows, fuse_inv);
  }

  // The decision left to the next enqueued sweep (ctl null: none).  Each of its
  // blocks then sums the partials, so not on grids whose partials are folded
  // first (more than 4096 one-row blocks, which only key 1 asks for).
  FinishArgs handed_on{};
  bool merge_ok() const {
    return D == 2 && tile.T1 == 1 && tile.T2 == G.N2 && tile.T2 >= 64 && strip_setup == 1 &&
           sweep_grid_max() <= kFusedParts && !fullsym() && !wallkin();
  }

  // partial sums of r^2 of step n's sweeps: a step's first sweep writes its own
  // while its other blocks still fold those of the step before
  double* parts_of(int n) const { return partials + (n & 1) * (size_t)nparts_cap; }

  // band spectrum of the correction after sweep ell (alternating buffers
  // when the sweep inverts the previous correction's rows while writing its
  // own forward rows)
  cpx<CT>* spec_of(int ell) const { return (fuse_inv && (ell & 1)) ? spec_alt : spec; }

  // history term of physical step n (see h_alt); the wall corrector keeps one
  double* h_of(int n) const { return (!wallkin() && (n & 1)) ? h_alt : h; }

  AcceptArgs<L, T> accept_args(int n, int ell, double a) {
    AcceptArgs<L, T> Ac{};
    Ac.ctl = ctl;
    Ac.n = n;
    Ac.ell = ell;
    Ac.fb = fb;
    for (int i = 0; i < 3; ++i) Ac.mb[i] = mb[i];
    Ac.h = h_of(n);
    Ac.NS = G.NS;
    Ac.a = a;
    Ac.inv1pa2 = 1.0 / (1.0 + a / 2.0);
    return Ac;
  }

  // m^n of step n, the next to run, where step n - 1 (bc - 1 accepted before it)
  // left it to a step that is not enqueued.
  void reconstruct(int n, int64_t bc) {
    const Roles& ro = ctl_h->roles[n & 1];
    const double a = (bc - 1 == 0) ? 1.0 / P.dt : 3.0 / (2.0 * P.dt);
    hipLaunchKernelGGL((k_reconstruct<L, T>), dim3(ew_grid()), dim3(256), 0, st,
                       (const T*)fb.p[ro.slot_hist[0]], (const double*)h_of(n - 1), 1.0 / (1.0 + a / 2.0),
                       mb[ro.slot_m[0]], G.NS);
    MSC_HIPCK(hipGetLastError());
  }

  // Blocks of a kernel that the device holds at once (occupancy per CU times
  // the CU count) for a block size, cached: the grid of the grid-resident
  // passes (any grid size gives the same results).
  struct Resident {
    const void* k;
    int threads, blocks;
  };
  std::vector<Resident> resident_cache;
  int resident_blocks(const void* k, int threads) {
    for (const auto& e : resident_cache)
      if (e.k == k && e.threads == threads) return e.blocks;
    int dev = 0, cus = 0, per_cu = 0;
    MSC_HIPCK(hipGetDevice(&dev));
    MSC_HIPCK(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    MSC_HIPCK(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, threads, 0));
    const int n = std::max(1, per_cu) * std::max(1, cus);
    resident_cache.push_back({k, threads, n});
    return n;
  }

  // The full-symbol correction of Eq. (full-symbol) for (step n, sweep ell),
  // guarded on the device like the shadow passes.  head: the rows pass (with
  // Ac and Fin, it decides acceptance first); tail: the column pass and the
  // inverse rows pass, which leave f_{l+1} in the sweep's output buffer (out
  // when c is null).
  void enqueue_fullsym(const DevCtl* c, int n, int ell, double a, const AcceptArgs<L, T>* Ac,
                       const FinishArgs* Fin, bool head, bool tail, T* out) {
    if constexpr (D == 2 && !DV) {
      FsArgs<T, CT, TM> F{};
      F.g = CorrGuard{c, n, ell};
      F.do_accept = (Ac && Fin) ? 1 : 0;
      F.Nx = G.N0;
      F.Ny = G.N2;
      F.NH = G.N2 / 2 + 1;
      F.r = rfs;
      F.spec = spec_fs;
      F.twx = tw[0];
      F.twy = tw[2];
      F.a = a;
      F.wp = wp;
      F.wm = wm;
      F.inv_ns = 1.0 / (double)G.NS;
      F.fb = fb;
      F.out = out;
      constexpr int LX = LineMax<CT>::fs_cols, LY = LineMax<CT>::fs_rows;
      if (head) {
        const AcceptArgs<L, T> acc = Ac ? *Ac : AcceptArgs<L, T>{};
        const FinishArgs fin = Fin ? *Fin : FinishArgs{};
        with_lg<2, LY>(ilog2(G.N2), [&](auto lg) {
          using S = FsRows<CT, lg.value>;
          hipLaunchKernelGGL((k_fs_rows_fwd<L, T, CT, TM, lg.value>), dim3((G.N0 + S::R - 1) / S::R), dim3(S::NT), 0,
                             st, F, acc, fin);
        });
        MSC_HIPCK(hipGetLastError());
      }
      if (tail) {
        // split column pass where it is faster (measured: N_x = 512, 12% per
        // iteration; at N_x <= 256 the extra launches cost more than the
        // parallelism gains)
        const bool split = (tune.fs_split == 1) || (tune.fs_split == 0 && G.N0 >= 512);
        with_lg<2, LX>(ilog2(G.N0), [&](auto lg) {
          if (split) {
            constexpr int LPB = 256 / LineFft<CT, lg.value, line_le(lg.value)>::TPL;
            const int lgrid = pad8((Q * F.NH + LPB - 1) / LPB);  // XCD-aware order
            const int64_t nk = Spec2<CT>::field(G.N0, F.NH);
            hipLaunchKernelGGL((k_fs_cols_fft<L, T, CT, TM, lg.value, -1>), dim3(lgrid), dim3(256), 0, st, F);
            hipLaunchKernelGGL((k_fs_solve_k<L, T, CT, TM>), dim3((int)std::min<int64_t>((nk + 63) / 64, 4096)),
                               dim3(64), 0, st, F);
            hipLaunchKernelGGL((k_fs_cols_fft<L, T, CT, TM, lg.value, +1>), dim3(lgrid), dim3(256), 0, st, F);
          } else {
            hipLaunchKernelGGL((k_fs_cols_solve<L, T, CT, TM, lg.value>), dim3(pad8(F.NH)), dim3(320), 0, st, F);
          }
        });
        MSC_HIPCK(hipGetLastError());
        with_lg<2, LY>(ilog2(G.N2), [&](auto lg) {
          using S = FsRows<CT, lg.value>;
          hipLaunchKernelGGL((k_fs_rows_inv<L, T, CT, TM, lg.value>), dim3((G.N0 + S::R - 1) / S::R), dim3(S::NT), 0,
                             st, F);
        });
        MSC_HIPCK(hipGetLastError());
      }
    } else {
      (void)c, (void)n, (void)ell, (void)a, (void)Ac, (void)Fin, (void)head, (void)tail, (void)out;
    }
  }

  // The shadow correction of Eq. (shadow-update) for (step n, sweep ell):
  // transforms of P r, per-wavevector Schur solve, inverse transforms into dm
  // (the lift is fused into the next sweep).  With Ac the first pass instead
  // reconstructs m^{n+1} when the step was accepted at this sweep.
  void enqueue_correction(const DevCtl* c, int n, int ell, double a, const AcceptArgs<L, T>* Ac) {
    XformBufs<CT, TM> B{Pr, dm, spec, spec2, {tw[0], tw[1], tw[2]}};
    enqueue_transform<CT, TM>(c, n, ell, a, Ac, false, B);
  }

  // With Ac and Fin the first pass decides on the sweep.  rows_in_sweep: the
  // sweep wrote the row spectrum, so the column pass is the first;
  // inv_in_sweep: the next sweep inverts the rows.
  template <class CX, class TX>
  void enqueue_transform(const DevCtl* c, int n, int ell, double a, const AcceptArgs<L, T>* Ac, bool adjoint,
                         const XformBufs<CX, TX>& B, const FinishArgs* Fin = nullptr, bool rows_in_sweep = false,
                         bool inv_in_sweep = false) {
    const AcceptArgs<L, T> acc = Ac ? *Ac : AcceptArgs<L, T>{};
    const FinishArgs fin = Fin ? *Fin : FinishArgs{};
    if constexpr (D == 2) {
      Fft2Args<CX, TX> F{};
      F.g = CorrGuard{c, n, ell};
      F.do_accept = (Ac && !rows_in_sweep) ? 1 : 0;
      F.decide = (Ac && rows_in_sweep) ? 1 : 0;
      F.adjoint = adjoint ? 1 : 0;
      F.Nx = G.N0;
      F.Ny = G.N2;
      F.NBy = G.N2 / 4 + 1;
      F.Pr = B.in;
      F.spec = B.spec1;
      F.dm = B.out;
      F.twx = B.tw[0];
      F.twy = B.tw[2];
      F.a = a;
      F.nu = nu;
      F.inv_ns = 1.0 / (double)G.NS;
      constexpr int LX = LineMax<CX>::cols2, LY = LineMax<CX>::rows2;
      if (!rows_in_sweep)
        with_lg<2, LY>(ilog2(G.N2), [&](auto lg) {
          using S = RowsShape<CX, lg.value>;
          hipLaunchKernelGGL((k_fft2_rows_fwd<L, T, CX, TX, lg.value>), dim3((G.N0 + S::R - 1) / S::R), dim3(S::NT),
                             0, st, F, acc, fin);
        });
      MSC_HIPCK(hipGetLastError());
      with_lg<2, LX>(ilog2(G.N0), [&](auto lg) {
        // one column per block, in the XCD-aware order
        hipLaunchKernelGGL((k_fft2_cols_solve<L, T, CX, TX, lg.value>), dim3(pad8(F.NBy)),
                           dim3(ColsShape<CX, lg.value>::NT), 0, st, F, acc, fin);
      });
      MSC_HIPCK(hipGetLastError());
      if (!inv_in_sweep)
        with_lg<2, LY>(ilog2(G.N2), [&](auto lg) {
          using S = RowsShape<CX, lg.value>;
          hipLaunchKernelGGL((k_fft2_rows_inv<CX, TX, lg.value>), dim3((G.N0 + S::R - 1) / S::R), dim3(S::NT), 0, st,
                             F);
        });
      MSC_HIPCK(hipGetLastError());
    } else {
      Fft3Args<CX, TX> F{};
      F.g = CorrGuard{c, n, ell};
      F.do_accept = Ac ? 1 : 0;
      F.adjoint = adjoint ? 1 : 0;
      F.Nx = G.n[0];
      F.Ny = G.n[1];
      F.Nz = G.n[2];
      F.NBz = F.Nz / 4 + 1;
      F.NBy = 2 * (F.Ny / 4) + 1;
      F.Pr = B.in;
      F.dm = B.out;
      F.spec1 = B.spec1;
      F.spec2 = B.spec2;
      F.twx = B.tw[0];
      F.twy = B.tw[1];
      F.twz = B.tw[2];
      F.a = a;
      F.nu = nu;
      F.inv_ns = 1.0 / (double)G.NS;
      constexpr int LM = LineMax<CX>::line3;
      auto col_grid = [&](int planes, int cw) { return dim3(pad8(planes * ((F.NBz + cw - 1) / cw))); };
      // z passes: the forward one (which decides) at most one block per
      // resident slot, each looping over pencil groups
      with_lg<2, LM>(ilog2(F.Nz), [&](auto lg) {
        using S = ZShape<CX, lg.value>;
        const int gz = (F.Nx * F.Ny + S::PB - 1) / S::PB;
        const int gr = std::min(gz, resident_blocks((const void*)k_fft3_z_fwd<L, T, CX, TX, lg.value>, S::NT));
        hipLaunchKernelGGL((k_fft3_z_fwd<L, T, CX, TX, lg.value>), dim3(gr), dim3(S::NT), 0, st, F, acc, fin);
      });
      MSC_HIPCK(hipGetLastError());
      with_lg<2, LM>(ilog2(F.Ny), [&](auto lg) {
        using S = ColShape3<CX, lg.value>;
        hipLaunchKernelGGL((k_fft3_y_fwd<CX, TX, lg.value>), col_grid(F.Nx, S::CW), dim3(S::NT), 0, st, F);
      });
      MSC_HIPCK(hipGetLastError());
      with_lg<2, LM>(ilog2(F.Nx), [&](auto lg) {
        using S = ColShape3<CX, lg.value>;
        hipLaunchKernelGGL((k_fft3_x_solve<CX, TX, lg.value>), col_grid(F.NBy, S::CW), dim3(S::NT), 0, st, F);
      });
      MSC_HIPCK(hipGetLastError());
      with_lg<2, LM>(ilog2(F.Ny), [&](auto lg) {
        using S = ColShape3<CX, lg.value>;
        hipLaunchKernelGGL((k_fft3_y_inv<CX, TX, lg.value>), col_grid(F.Nx, S::CW), dim3(S::NT), 0, st, F);
      });
      MSC_HIPCK(hipGetLastError());
      with_lg<2, LM>(ilog2(F.Nz), [&](auto lg) {
        using S = ZShape<CX, lg.value>;
        hipLaunchKernelGGL((k_fft3_z_inv<CX, TX, lg.value>), dim3((F.Nx * F.Ny + S::PB - 1) / S::PB), dim3(S::NT), 0,
                           st, F);
      });
      MSC_HIPCK(hipGetLastError());
    }
  }
};

}  // namespace msc
