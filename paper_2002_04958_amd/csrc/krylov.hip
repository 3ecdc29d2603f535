// Restarted right-preconditioned (flexible) GMRES(m) on the block system of
// eq. 2.2.  Arnoldi uses classical Gram-Schmidt with selective
// reorthogonalisation: the projection coefficients and the norm come from one
// pass over the basis, the update is fused with the second projection, and a
// third pass (second update) runs only when the first projection removed more
// than half of the norm.  The small
// Hessenberg least-squares problem (Givens rotations) runs on the host from
// one readback of the new column per step.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <functional>
#include <mutex>
#include <vector>

#include "handles.hpp"
#include "kernels.hpp"

using namespace mgd;

struct EvPair {
  hipEvent_t a = nullptr, b = nullptr;
  EvPair() {
    MGD_HIP(hipEventCreate(&a));
    MGD_HIP(hipEventCreate(&b));
  }
  ~EvPair() {
    hipEventDestroy(a);
    hipEventDestroy(b);
  }
  float ms() {
    float t = 0;
    MGD_HIP(hipEventElapsedTime(&t, a, b));
    return t;
  }
};

void block_precond_apply_impl(block_precond* bp, const double* r, double* z);
void block_precond_apply_matvec(block_precond* bp, const double* r, double* z,
                                const BlockSysDev& S, double* y, bool first_done = false);
bool block_precond_has_first_stage(const block_precond* bp);
void block_precond_first_stage(block_precond* bp, const double* r);
void block_precond_side(block_precond* bp, hipStream_t* s, hipEvent_t* fork, hipEvent_t* join);
bool block_precond_steps_ahead(const block_precond* bp);

// Workspace of gmres_solve_noalloc: a static device array, one copy per
// device, shared by every such call on that device (the contents of the last
// call stay; the solve writes every buffer before it reads it).
constexpr size_t kNoAllocBytes = size_t(64) << 20;
static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

namespace {
// The basis, the preconditioned vectors and the scratch of one context,
// reallocated only when the problem size or the restart length grows.
struct GmresWork {
  size_t n = 0;
  int m = 0;
  DBuf<double> V, Z, t1, t2, hd, dd, dcoef;
  RedWork rw;
  hipEvent_t ev[2] = {nullptr, nullptr};  // readbacks of two steps in flight
  ~GmresWork() {
    for (auto e : ev)
      if (e) hipEventDestroy(e);
  }
};
GmresWork& gmres_work(Ctx* c, size_t n, int m, bool need_z, bool need_t) {
  auto* w = static_cast<GmresWork*>(c->gmres_ws.get());
  if (!w || w->n != n || w->m < m) {
    c->gmres_ws.reset();
    auto sp = std::make_shared<GmresWork>();
    w = sp.get();
    c->gmres_ws = sp;
    w->n = n;
    w->m = m;
    w->V.alloc(c, (size_t)(m + 1) * n);
    w->hd.alloc(c, 200);
    w->dd.alloc(c, 80);
    w->dcoef.alloc(c, kDcgsCoef);
  }
  if (!w->ev[0])
    for (auto& e : w->ev) MGD_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
  if (need_z && w->Z.n < (size_t)w->m * n) w->Z.alloc(c, (size_t)w->m * n);
  if (need_t && w->t1.n < n) {
    w->t1.alloc(c, n);
    w->t2.alloc(c, n);
  }
  return *w;
}

// ---------------------------------------------------------------------------
// workspace of the no-allocation entry point (the array `scratch` below)
// ---------------------------------------------------------------------------
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of this device's array (the host symbol is only a
// stand-in): looked up once per device, with that device current.
void* scratch_address(Ctx* c) {
  std::lock_guard<std::mutex> g(g_scratch_mu);
  MGD_REQUIRE(c->device >= 0 && c->device < kMaxDevices, "device ordinal out of range");
  if (!g_scratch_ptr[c->device]) {
    void* p = nullptr;
    MGD_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    MGD_REQUIRE(p != nullptr, "no device address for the scratch array");
    g_scratch_ptr[c->device] = p;
  }
  return g_scratch_ptr[c->device];
}

// Buffers of one solve laid out in the array, 256-byte aligned, in doubles.
struct ScratchLayout {
  size_t V = 0, Z = 0, t1 = 0, t2 = 0, hd = 0, dd = 0, dcoef = 0, part = 0, total = 0;
};
ScratchLayout scratch_layout(size_t n, int m, bool need_z, bool need_t) {
  ScratchLayout L;
  size_t at = 0;
  auto take = [&](size_t count) {
    const size_t o = at;
    at += (count + 31) / 32 * 32;  // 256 bytes
    return o;
  };
  L.V = take((size_t)(m + 1) * n);
  if (need_z) L.Z = take((size_t)m * n);
  if (need_t) {
    L.t1 = take(n);
    L.t2 = take(n);
  }
  L.hd = take(200);
  L.dd = take(80);
  L.dcoef = take(kDcgsCoef);
  L.part = take((size_t)kRedBlocks * 66);
  L.total = at * sizeof(double);
  return L;
}

// non-owning views of the array (a view has no context, so nothing frees it)
template <typename T>
void view(DBuf<T>& b, double* base, size_t off, size_t count) {
  b.ctx = nullptr;
  b.p = reinterpret_cast<T*>(base + off);
  b.n = count;
}
void scratch_work(Ctx* c, GmresWork& w, size_t n, int m, bool need_z, bool need_t) {
  const ScratchLayout L = scratch_layout(n, m, need_z, need_t);
  MGD_REQUIRE(L.total <= kNoAllocBytes, "the no-allocation workspace holds " +
                                            std::to_string(kNoAllocBytes) + " bytes; this solve needs " +
                                            std::to_string(L.total));
  double* base = static_cast<double*>(scratch_address(c));
  w.n = n;
  w.m = m;
  view(w.V, base, L.V, (size_t)(m + 1) * n);
  if (need_z) view(w.Z, base, L.Z, (size_t)m * n);
  if (need_t) {
    view(w.t1, base, L.t1, n);
    view(w.t2, base, L.t2, n);
  }
  view(w.hd, base, L.hd, 200);
  view(w.dd, base, L.dd, 80);
  view(w.dcoef, base, L.dcoef, kDcgsCoef);
  view(w.rw.partial, base, L.part, (size_t)kRedBlocks * 66);
}
}  // namespace

mgd_status gmres_impl(Ctx* c, const BlockSysDev& S, block_precond* M, const double* b, double* x,
                      const gmres_params& p, gmres_result& res) {
  res = gmres_result{};
  const size_t n = (size_t)(S.G + 2) * S.N;
  const int m = p.restart;
  MGD_REQUIRE(m >= 1 && m <= 31, "restart must be in [1, 31]");
  MGD_REQUIRE(p.max_iters >= 0, "max_iters must be >= 0");
  auto t_start = std::chrono::steady_clock::now();
  const bool flex = p.flexible != 0;
  GmresWork local;  // views of the static array in a no-allocation call
  if (c->no_alloc) scratch_work(c, local, n, m, flex && M, !flex && M);
  GmresWork& ws = c->no_alloc ? local : gmres_work(c, n, m, flex && M, !flex && M);
  DBuf<double>& V = ws.V;
  DBuf<double>& Z = ws.Z;
  DBuf<double>& t1 = ws.t1;
  DBuf<double>& t2 = ws.t2;
  DBuf<double>& hd = ws.hd;
  double* h1 = hd.get();
  double* h2 = hd.get() + 40;
  double* hc = hd.get() + 80;       // [0..J+2]: column, reorth flag, exact squared norm
  double* yd = hd.get() + 130;      // y (<= 31)
  double* bn = hd.get() + 125;
  RedWork& rw = ws.rw;
  std::unique_ptr<EvPair> evp, evm, evo;
  if (p.profile) {
    evp.reset(new EvPair);
    evm.reset(new EvPair);
    evo.reset(new EvPair);
  }
  double* hbuf = static_cast<double*>(c->host_stage(256 * sizeof(double)));
  // pinned slots for the coefficients of two steps in flight
  auto slot = [&](int jj) { return hbuf + 128 * (jj & 1); };

  dot_dev(c, rw, b, b, n, bn);
  const double bnorm = std::sqrt(read1(c, bn));
  if (bnorm == 0.0) {
    fill<double>(c, x, 0.0, n);
    c->sync();
    res.converged = 1;
    return MGD_OK;
  }
  const double tol = p.rtol * bnorm;
  double* V0 = V.get();
  block_matvec(c, S, x, b, V0);
  dot_dev(c, rw, V0, V0, n, bn);
  double beta = std::sqrt(read1(c, bn));
  res.relres_true = res.relres_est = beta / bnorm;
  if (beta <= tol) {
    res.converged = 1;
    res.t_total_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t_start).count();
    return MGD_OK;
  }
  std::vector<double> H((size_t)(m + 1) * m), cs(m), sn(m), g(m + 1), y(m);
  double r_last = 0.0, r_prev = 0.0;  // residual estimates of the last two steps
  int launched = -1;     // steps enqueued ahead in this cycle
  auto Hij = [&](int i, int j) -> double& { return H[(size_t)i * m + j]; };
  // Flexible GMRES with a preconditioner keeps the unrotated Hessenberg
  // matrix: the delayed reorthogonalisation completes each column one step
  // later, and the rotations are then recomputed.
  const bool delayed = M && flex;
  std::vector<double> Hunrot((size_t)(m + 1) * m);
  auto Hu = [&](int i, int j) -> double& { return Hunrot[(size_t)i * m + j]; };
  DBuf<double>& dd = ws.dd;
  DBuf<double>& dcoef = ws.dcoef;
  // Steps enqueued ahead of the host's look at their coefficients (no per-step
  // events then)
  const bool ahead = delayed && !p.profile && block_precond_steps_ahead(M);
  // Where the apply starts with w_E* = A_E^{-1} r_E, each such step ends by
  // computing it for the next basis vector beside the rest of its update
  // sweep (the E segment of the sweep first), and the next step skips it.
  const bool early_E = ahead && block_precond_has_first_stage(M);
  DcgsSplit split;
  if (early_E) {
    block_precond_side(M, &split.side, &split.fork, &split.join);
    split.lo = (size_t)S.G * S.N;
    split.hi = split.lo + S.N;
  }
  if (ahead) rw.ensure(c);
  // Enqueue step jj (z = M^{-1} v_jj, w = A z, the Gram-Schmidt
  // step) and the readback of its coefficients into pinned slot jj % 2.
  auto launch_step = [&](int jj) {
    double* vjj = V.get() + (size_t)jj * n;
    double* wj = V.get() + (size_t)(jj + 1) * n;
    double* zt = Z.get() + (size_t)jj * n;
    const bool prov = jj >= 1;
    const int F = prov ? jj : 1;
    // step jj-1 of this cycle computed w_E* for v_jj; step m-1 skips it for v_m
    const bool done = early_E && jj >= 1;
    const bool next = early_E && jj + 1 < m;
    block_precond_apply_matvec(M, vjj, zt, S, wj, done);
    if (next) split.beside = [&] { block_precond_first_stage(M, wj); };
    dcgs_step_dev(c, rw, V.get(), n, F, prov ? vjj : nullptr, wj, n, dd.get(), dcoef.get(),
                  next ? &split : nullptr);
    split.beside = nullptr;
    MGD_HIP(hipMemcpyAsync(slot(jj), dcoef.get(), kDcgsCoef * sizeof(double),
                           hipMemcpyDeviceToHost, c->stream));
    MGD_HIP(hipEventRecord(ws.ev[jj & 1], c->stream));
    res.precond_applies++;
    launched = jj;
  };
  while (res.iters < p.max_iters) {
    scale_copy(c, V0, V0, 1.0 / beta, n);
    std::fill(g.begin(), g.end(), 0.0);
    g[0] = beta;
    int k = 0;
    bool breakdown = false;
    double alpha_prev = 0.0;
    std::fill(Hunrot.begin(), Hunrot.end(), 0.0);
    launched = -1;
    r_last = beta;
    r_prev = 0.0;
    for (int j = 0; j < m; ++j) {
      double* vj = V.get() + (size_t)j * n;
      double* w = V.get() + (size_t)(j + 1) * n;
      const double* zj = vj;
      if (delayed && ahead) {
        if (launched < j) launch_step(j);
        // Enqueue step j+1 before waiting for this step's coefficients: it
        // needs only v_{j+1}, which this step writes, so the GPU works on it
        // while the host finishes column j.  Skipped at the end of a cycle,
        // at the iteration cap, and when the recent reduction rate says this
        // step is likely to converge.
        // residual estimates after j and j-1 steps: forecast the next one
        const double ratio = (j >= 2 && r_prev > 0.0) ? r_last / r_prev : 1.0;
        const bool likely_done = j >= 1 && r_last * ratio <= tol;
        if (j + 1 < m && res.iters + 1 < p.max_iters && !likely_done) launch_step(j + 1);
      } else if (M) {
        double* zt = flex ? Z.get() + (size_t)j * n : t1.get();
        if (evp) MGD_HIP(hipEventRecord(evp->a, c->stream));
        if (delayed && !p.profile)  // the launches a step enqueued ahead runs
          block_precond_apply_matvec(M, vj, zt, S, w);
        else
          block_precond_apply_impl(M, vj, zt);
        if (evp) MGD_HIP(hipEventRecord(evp->b, c->stream));
        res.precond_applies++;
        zj = zt;
      }
      if (!(delayed && (ahead || !p.profile))) {
        if (evm) MGD_HIP(hipEventRecord(evm->a, c->stream));
        block_matvec(c, S, zj, nullptr, w);
        if (evm) MGD_HIP(hipEventRecord(evm->b, c->stream));
      }
      const int J = j + 1;
      if (delayed) {
        // Classical Gram-Schmidt with the reorthogonalisation of v_j delayed
        // into this step: two sweeps over the basis.  The previous column is
        // completed here (v_j = V a + beta v_j_new), then this column.
        const bool prov = j >= 1;
        const int F = prov ? j : 1;
        if (!ahead) {
          if (evo) MGD_HIP(hipEventRecord(evo->a, c->stream));
          dcgs_step_dev(c, rw, V.get(), n, F, prov ? vj : nullptr, w, n, dd.get(), dcoef.get());
          if (evo) MGD_HIP(hipEventRecord(evo->b, c->stream));
        }
        const double* hb = hbuf;
        if (ahead) {
          hb = slot(j);
          MGD_HIP(hipEventSynchronize(ws.ev[j & 1]));
        } else {
          MGD_HIP(hipMemcpyAsync(hbuf, dcoef.get(), kDcgsCoef * sizeof(double),
                                 hipMemcpyDeviceToHost, c->stream));
          c->sync();
          if (evp) res.t_precond_ms += evp->ms();
          if (evm) res.t_matvec_ms += evm->ms();
          if (evo) res.t_orth_ms += evo->ms();
        }
        double hF = prov ? hb[32 + F] : 0.0;
        if (prov) {
          res.reorths++;
          for (int i = 0; i < j; ++i) Hu(i, j - 1) += alpha_prev * hb[i];
          Hu(j, j - 1) = alpha_prev * hb[64];
          // v_j_new came out of Pythagoras' beta; where its exact norm is off
          // unit length, rescale it and the two coefficients that multiply it
          // (not when the next step is already under way with it: that step's
          // dots use its actual norm, and the relation stays exact)
          const double nv = std::sqrt(hb[66]);
          if (!ahead && !(std::fabs(nv - 1.0) <= 1e-6) && nv > 0.0) {
            scale_dev(c, 1.0 / nv, vj, n);
            Hu(j, j - 1) *= nv;
            hF *= nv;
          }
        }
        for (int i = 0; i < F; ++i) Hu(i, j) = hb[32 + i];
        if (prov) Hu(j, j) = hF;
        double al = hb[65];
        const double ex = std::sqrt(hb[67]);
        if (!ahead && !(std::fabs(ex - al) <= 1e-6 * ex)) {
          if (ex > 0.0) scale_dev(c, al / ex, w, n);
          al = ex;
        }
        if (ahead && !(ex > 0.0)) al = 0.0;  // w' vanished: breakdown
        Hu(j + 1, j) = al;
        alpha_prev = al;
        breakdown = al == 0.0;
        // Givens QR of the columns so far (the last two changed this step)
        for (int q = 0; q <= j; ++q)
          for (int i = 0; i <= q + 1; ++i) Hij(i, q) = Hu(i, q);
        std::fill(g.begin(), g.end(), 0.0);
        g[0] = beta;
        for (int q = 0; q <= j; ++q) {
          for (int i = 0; i < q; ++i) {
            const double tt = cs[i] * Hij(i, q) + sn[i] * Hij(i + 1, q);
            Hij(i + 1, q) = -sn[i] * Hij(i, q) + cs[i] * Hij(i + 1, q);
            Hij(i, q) = tt;
          }
          const double den = std::sqrt(Hij(q, q) * Hij(q, q) + Hij(q + 1, q) * Hij(q + 1, q));
          if (den == 0.0) fail(MGD_EBREAKDOWN, "GMRES breakdown: singular Hessenberg matrix");
          cs[q] = Hij(q, q) / den;
          sn[q] = Hij(q + 1, q) / den;
          Hij(q, q) = den;
          Hij(q + 1, q) = 0.0;
          g[q + 1] = -sn[q] * g[q];
          g[q] = cs[q] * g[q];
        }
        res.iters++;
        k = j + 1;
        r_prev = r_last;
        r_last = std::fabs(g[j + 1]);
        res.relres_est = std::fabs(g[j + 1]) / bnorm;
        if (std::fabs(g[j + 1]) <= tol || res.iters >= p.max_iters || breakdown) break;
        continue;
      }
      if (evo) MGD_HIP(hipEventRecord(evo->a, c->stream));
      mdot_dev(c, rw, V.get(), n, J, w, n, h1);
      update_mdot_dev(c, rw, V.get(), n, J, h1, w, n, h2);
      orth_finish_dev(c, rw, V.get(), n, J, h1, h2, hc, w, n);
      if (evo) MGD_HIP(hipEventRecord(evo->b, c->stream));
      MGD_HIP(hipMemcpyAsync(hbuf, hc, (J + 3) * sizeof(double), hipMemcpyDeviceToHost, c->stream));
      c->sync();
      if (evp && M) res.t_precond_ms += evp->ms();
      if (evm) res.t_matvec_ms += evm->ms();
      if (evo) res.t_orth_ms += evo->ms();
      for (int i = 0; i <= J; ++i) Hij(i, j) = hbuf[i];
      if (hbuf[J + 1] != 0.0) {
        res.reorths++;
        // The new basis vector is w''/s with s = hbuf[J] from Pythagoras, and
        // H(J, j) = s keeps the Arnoldi relation exact.  Where s is off the
        // exact norm (a severe cancellation, or the fallback s = 1), rescale
        // the vector to unit length and record the exact norm instead.
        const double ex = std::sqrt(hbuf[J + 2]);
        const double s = hbuf[J];
        if (!(std::fabs(ex - s) <= 1e-6 * ex)) {
          if (ex > 0.0) scale_dev(c, s / ex, w, n);
          Hij(J, j) = ex;
        }
      }
      breakdown = Hij(j + 1, j) == 0.0;
      for (int i = 0; i < j; ++i) {
        const double tt = cs[i] * Hij(i, j) + sn[i] * Hij(i + 1, j);
        Hij(i + 1, j) = -sn[i] * Hij(i, j) + cs[i] * Hij(i + 1, j);
        Hij(i, j) = tt;
      }
      const double den = std::sqrt(Hij(j, j) * Hij(j, j) + Hij(j + 1, j) * Hij(j + 1, j));
      if (den == 0.0) fail(MGD_EBREAKDOWN, "GMRES breakdown: singular Hessenberg matrix");
      cs[j] = Hij(j, j) / den;
      sn[j] = Hij(j + 1, j) / den;
      Hij(j, j) = den;
      Hij(j + 1, j) = 0.0;
      g[j + 1] = -sn[j] * g[j];
      g[j] = cs[j] * g[j];
      res.iters++;
      k = j + 1;
      res.relres_est = std::fabs(g[j + 1]) / bnorm;
      if (std::fabs(g[j + 1]) <= tol || res.iters >= p.max_iters || breakdown) break;
    }
    // back substitution H y = g
    for (int i = k - 1; i >= 0; --i) {
      double s = g[i];
      for (int q = i + 1; q < k; ++q) s -= Hij(i, q) * y[q];
      y[i] = s / Hij(i, i);
    }
    std::copy(y.begin(), y.begin() + k, hbuf + 80);  // pinned staging (k <= 31)
    MGD_HIP(hipMemcpyAsync(yd, hbuf + 80, k * sizeof(double), hipMemcpyHostToDevice, c->stream));
    if (!M) {
      combine_dev(c, V.get(), n, k, yd, x, n);
    } else if (flex) {
      combine_dev(c, Z.get(), n, k, yd, x, n);
    } else {
      fill<double>(c, t1.get(), 0.0, n);
      combine_dev(c, V.get(), n, k, yd, t1.get(), n);
      block_precond_apply_impl(M, t1.get(), t2.get());
      res.precond_applies++;
      axpy(c, x, t2.get(), 1.0, n);
    }
    res.restarts++;
    block_matvec(c, S, x, b, V0);
    dot_dev(c, rw, V0, V0, n, bn);
    beta = std::sqrt(read1(c, bn));
    res.relres_true = beta / bnorm;
    if (beta <= tol) {
      res.converged = 1;
      break;
    }
    if (beta == 0.0) break;
  }
  c->sync();
  res.t_total_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t_start).count();
  return res.converged ? MGD_OK : MGD_ENOTCONV;
}
