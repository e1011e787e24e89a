// Alg. momentum_verification end to end for the verifiers of p pipeline stages with d workers each
// (worker r of every stage belongs to data-parallel pipe r).  The device work -- the statistics of every
// worker's signal against the stage's EMA, the gradient replacement, the EMA update over the clean set --
// goes through the library's own entry points (the checks of a call through one pass over the signals, check_signals, where
// the shape allows it) on the caller's stream; the decisions in between are the
// host-side policy (sv_policy_*).  Each forward / backward call therefore waits once for its checks: the
// few scalars per worker have to reach the host before the policy can decide who enters the EMA.  (For the stream, or, where work that
// is likely to stand is queued behind the checks already, for an event between the two.)
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <limits>
#include <utility>
#include <vector>

#include <hip/hip_runtime.h>

#include "common.h"

struct sv_sentinel {
  sv_ctx* ctx = nullptr;
  sv_sentinel_cfg cfg;
  int n_metrics = 0;
  int metric_bit[5];                       // mask bit of column i of Gamma
  std::vector<float*> m[2];                // [kind][stage] device fp32 [T, D]; kind 0 = activations, 1 = gradients
  std::vector<sv_policy*> pol[2];
  std::vector<uint8_t> tainted;            // [stage * d + r] of the current iteration
  bool warm = true;
  uint8_t* mask_dev = nullptr;             // two rows of d bytes: replacement mask, EMA exclusion mask
  float* sum_dev = nullptr;                // [T, D]: sum over the signals not excluded beforehand, written by the score pass; where one
                                           // pass has updated the EMA as well: what it was before
  // sliced Wasserstein against the EMA without projecting the EMA: its projections follow from the signals' (linearity)
  std::vector<float*> pm[2];               // [kind][stage] device fp32 [n_dirs, Tpad]: <u_l, m_t>, kept up to date with m
  // their rows sorted, for the next call's one pass; sorted_ok: they are those of pm as it is.  Both are made behind the checks, for the
  // verdicts that are to be expected (nobody excluded who was not beforehand), before the host has them: it waits for the checks
  // alone, and the GPU has work while the verdicts are made and the next call is on its way.  The update goes to pm_next, which takes
  // pm's place when the verdicts stand (else it is made again from pm).  4 x 16 workers of 8192 x 4096: behind the verdicts the GPU
  // stood still 33 us a call: 3635 us an iteration, 3485 so
  std::vector<float*> ps[2];
  std::vector<uint8_t> sorted_ok[2];
  float* pm_next = nullptr;
  hipEvent_t checked = nullptr;            // the checks of the call under way have run; releases to the system: the host reads what they wrote
  float* cproj = nullptr;                  // [d, n_dirs, Tpad]: the current signals' projections
  int64_t n_calls = 0, n_from_sum = 0, n_from_signals = 0, n_sw_carried = 0;
  // pinned host memory; the statistics' last kernels write their few scalars straight into the first two, and the call waits for
  // the checks before it reads them (as copies they were two launches more in every call's chain)
  sv_result* res_host = nullptr;
  float* sw_host = nullptr;
  uint8_t* mask_host = nullptr;
  char err[256] = "";
};

namespace {

void set_err(sv_sentinel* s, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(s->err, sizeof(s->err), fmt, ap);
  va_end(ap);
}

#define SN_HIP(s, call)                                                         \
  do {                                                                          \
    hipError_t e_ = (call);                                                     \
    if (e_ != hipSuccess) { set_err(s, "%s failed: %s", #call, hipGetErrorString(e_)); return SV_EHIP; } \
  } while (0)
#define SN_SV(s, call)                                                          \
  do {                                                                          \
    sv_status st_ = (call);                                                     \
    if (st_ != SV_OK) { set_err(s, "%s: %s", #call, sv_last_error((s)->ctx)); return st_; } \
  } while (0)

// A stage call's EMA while the call is under way.  Where one pass did the checks it has updated m already, over the signals not
// excluded beforehand, and left what it was in sum_dev.  A call that ends before its verdicts stand leaves m as it was.
struct CallEma {
  sv_sentinel* s;
  int kind, stage;
  float beta;
  hipStream_t st;
  float* m = s->m[kind][stage];
  float* pm = s->pm[kind].empty() ? nullptr : s->pm[kind][stage];       // its projections, or none
  bool one_pass = false, updated = false;
  bool ahead = false;                      // pm_next and the sorted rows are those of pm with the signals not excluded beforehand
  const float* now() const { return updated ? s->sum_dev : m; }
  ~CallEma() {
    if (updated) (void)hipMemcpyAsync(m, s->sum_dev, (size_t)s->cfg.T * s->cfg.D * sizeof(float), hipMemcpyDeviceToDevice, st);
  }
};

// Gamma [d, n_metrics] of the d signals against the reference point ema.m, on the host (waits for the checks).
// `skip` [d]: the signals known to be excluded from the EMA before they are scored.  Where the score pass can do it,
// it also leaves the sum over the others in sum_dev, or updates the EMA with it (*summed = true), which saves the EMA update its own
// pass over the signals whenever the verdicts exclude nobody else.
sv_status gamma_of(sv_sentinel* s, const void* signals, int dtype, CallEma& ema, const uint8_t* skip, bool* summed,
                   std::vector<double>& gamma, hipStream_t st) {
  const sv_sentinel_cfg& c = s->cfg;
  const int d = c.n_workers;
  const int64_t stride = c.T * c.D;
  const float inf = std::numeric_limits<float>::infinity();
  const float tau[4] = {inf, inf, inf, inf};      // nothing is decided on the device here: the fences live in the policy
  float* m = ema.m;
  const float* pm = ema.pm;
  // statistics, EMA update and projections in one pass over the signals where the shape allows it
  sv_status one = SV_EUNSUPPORTED;
  if ((c.metric_mask & SV_M_SW) && pm && s->sum_dev) {
    one = sv::check_signals(s->ctx, signals, stride, d, dtype, m, s->sum_dev, ema.beta, c.T, c.D, c.metric_mask & 15u, tau, s->res_host, skip, c.directions,
                            c.n_dirs, pm, s->sorted_ok[ema.kind][ema.stage] ? s->ps[ema.kind][ema.stage] : nullptr, s->cproj, s->sw_host, &ema.updated, st);
    ema.one_pass = ema.updated;
    if (one != SV_OK && one != SV_EUNSUPPORTED) { set_err(s, "the loop's pass: %s", sv_last_error(s->ctx)); return one; }
  }
  sv_status sum_st = one == SV_OK ? SV_OK : s->sum_dev ? sv_score_and_sum(s->ctx, signals, stride, d, m, dtype, SV_F32, c.T, c.D, c.metric_mask & 15u, tau,
                                                   SV_REDUCE_GLOBAL, nullptr, s->res_host, skip, s->sum_dev, st)
                                : SV_EUNSUPPORTED;
  *summed = sum_st == SV_OK;
  if (sum_st == SV_EUNSUPPORTED)                  // shapes the summing pass does not take: the plain one
    SN_SV(s, sv_score_and_flag(s->ctx, signals, stride, d, m, 0, dtype, SV_F32, c.T, c.D, c.metric_mask & 15u, tau, SV_REDUCE_GLOBAL, nullptr,
                               s->res_host, st));
  else if (sum_st != SV_OK) { set_err(s, "sv_score_and_sum: %s", sv_last_error(s->ctx)); return sum_st; }
  if (c.metric_mask & SV_M_SW) {
    if (pm) ++s->n_sw_carried;
    if (one == SV_OK) {
    } else if (pm)
      SN_SV(s, sv_sw_against_projection(s->ctx, signals, stride, d, dtype, c.T, c.D, c.directions, c.n_dirs, pm, s->cproj, inf, s->sw_host,
                                        nullptr, st));
    else
      SN_SV(s, sv_sliced_wasserstein(s->ctx, signals, stride, d, m, 0, dtype, SV_F32, c.T, c.D, c.directions, c.n_dirs, inf, s->sw_host,
                                     nullptr, st));
  }
  uint32_t mask = 0;
  int taken = 0;
  for (int r = 0; r < d; ++r) { if (skip[r]) mask |= 1u << (r & 31); else ++taken; }
  if (ema.one_pass && s->pm_next && taken > 0) {
    const int64_t row = sv_sw_row_len(c.T);
    float* sorted = s->ps[ema.kind][ema.stage];
    SN_HIP(s, hipEventRecord(s->checked, st));
    s->sorted_ok[ema.kind][ema.stage] = 0;         // until the verdicts say so
    SN_HIP(s, sv::launch_sw_proj_ema(s->pm_next, pm, s->cproj, d, mask, c.n_dirs, c.T, row, ema.beta, (1.0f - ema.beta) / (float)taken, st));
    SN_HIP(s, sv::launch_sw_sort(sorted, c.n_dirs, c.T, row, nullptr, 0, c.n_dirs, nullptr, 0, st, s->pm_next));
    ema.ahead = true;
    SN_HIP(s, hipEventSynchronize(s->checked));
  } else {
    SN_HIP(s, hipStreamSynchronize(st));
  }
  gamma.assign((size_t)d * s->n_metrics, 0.0);
  for (int r = 0; r < d; ++r)
    for (int i = 0; i < s->n_metrics; ++i) {
      const int bit = s->metric_bit[i];
      double v;
      if (bit == SV_M_SW) v = s->sw_host[r];
      else v = s->res_host[r].score[bit == SV_M_RELL2 ? SV_IDX_RELL2 : bit == SV_M_L1 ? SV_IDX_L1 : bit == SV_M_ZL2 ? SV_IDX_ZL2 : SV_IDX_SFR];
      gamma[(size_t)r * s->n_metrics + i] = v;
    }
  return SV_OK;
}

// Eq. momentum_def over the signals with excl[r] == 0.  If the score pass has left the sum over the signals with
// skip[r] == 0 and the verdicts excluded nobody beyond those, the update is one pass over m and that sum, or done already; otherwise
// the update reads the signals itself.
sv_status update_ema(sv_sentinel* s, CallEma& ema, const void* signals, int dtype, const uint8_t* excl, const uint8_t* skip,
                     bool summed, bool mask_uploaded = false) {
  const int d = s->cfg.n_workers;
  const hipStream_t hs = ema.st;
  bool same = summed;
  int n = 0;
  for (int r = 0; r < d; ++r) { same = same && (excl[r] != 0) == (skip[r] != 0); n += excl[r] == 0; }
  if (ema.pm && ema.ahead && same) {
    std::swap(s->pm[ema.kind][ema.stage], s->pm_next);
    s->sorted_ok[ema.kind][ema.stage] = 1;
  } else if (ema.pm) {
    uint8_t& ok = s->sorted_ok[ema.kind][ema.stage];
    if (n > 0) ok = 0;                             // with nobody to take the projections stay as they are
    SN_SV(s, sv_sw_projection_ema(s->ctx, ema.pm, s->cproj, d, excl, s->cfg.T, s->cfg.n_dirs, ema.beta, hs));
    if (ema.one_pass && !ok) {
      SN_HIP(s, sv::launch_sw_sort(s->ps[ema.kind][ema.stage], s->cfg.n_dirs, s->cfg.T, sv_sw_row_len(s->cfg.T), nullptr, 0, s->cfg.n_dirs, nullptr, 0, hs, ema.pm));
      ok = 1;
    }
  }
  ++s->n_calls;
  if (same) {
    ++s->n_from_sum;
    if (!ema.updated) SN_SV(s, sv_ema_from_sum(s->ctx, ema.m, s->sum_dev, n, s->cfg.T, s->cfg.D, ema.beta, hs));
    ema.updated = false;
    return SV_OK;
  }
  ++s->n_from_signals;
  if (!mask_uploaded) SN_HIP(s, hipMemcpyAsync(s->mask_dev + d, excl, (size_t)d, hipMemcpyHostToDevice, hs));
  if (ema.updated) SN_HIP(s, sv::launch_ema(ema.m, signals, s->cfg.T * s->cfg.D, d, dtype, s->mask_dev + d, s->cfg.T, s->cfg.D, ema.beta, hs, s->sum_dev));
  else SN_SV(s, sv_ema_update(s->ctx, ema.m, signals, s->cfg.T * s->cfg.D, d, dtype, s->mask_dev + d, s->cfg.T, s->cfg.D, ema.beta, hs));
  ema.updated = false;
  return SV_OK;
}

sv_status check_stage(sv_sentinel* s, int stage, const void* sig, int dtype, uint8_t* tainted_out) {
  if (stage < 0 || stage >= s->cfg.n_stages) { set_err(s, "stage %d out of range", stage); return SV_EINVAL; }
  if (!sig || !tainted_out) { set_err(s, "signals and tainted_out must be non-NULL"); return SV_EINVAL; }
  if (dtype != SV_F32 && dtype != SV_BF16) { set_err(s, "unknown dtype"); return SV_EINVAL; }
  return SV_OK;
}

}  // namespace

extern "C" {

sv_status sv_sentinel_create(sv_ctx* ctx, const sv_sentinel_cfg* cfg, sv_sentinel** out) {
  if (!out) return SV_EINVAL;
  *out = nullptr;
  if (!ctx || !cfg || cfg->n_stages < 1 || cfg->n_workers < 1 || cfg->n_workers > 1024 || cfg->T < 1 || cfg->D < 1 || cfg->D % 8) return SV_EINVAL;
  if (!(cfg->metric_mask & 31u) || (cfg->metric_mask & ~31u)) return SV_EINVAL;
  if ((cfg->metric_mask & SV_M_SW) && (!cfg->directions || cfg->n_dirs < 1)) return SV_EINVAL;
  if (!(cfg->beta_h >= 0.0f && cfg->beta_h < 1.0f && cfg->beta_g >= 0.0f && cfg->beta_g < 1.0f)) return SV_EINVAL;
  sv_sentinel* s = new sv_sentinel();
  s->ctx = ctx; s->cfg = *cfg;
  for (int bit = 1; bit <= 16; bit <<= 1)
    if (cfg->metric_mask & (uint32_t)bit) s->metric_bit[s->n_metrics++] = bit;
  const int d = cfg->n_workers;
  sv_status st = SV_OK;
  for (int kind = 0; kind < 2 && st == SV_OK; ++kind)
    for (int i = 0; i < cfg->n_stages && st == SV_OK; ++i) {
      sv_policy* p = nullptr;
      st = sv_policy_create(d, s->n_metrics, kind == 0 ? &cfg->policy_h : &cfg->policy_g, &p);
      if (st == SV_OK) s->pol[kind].push_back(p);
    }
  const size_t m_bytes = (size_t)cfg->T * cfg->D * sizeof(float);
  hipError_t e = hipSuccess;
  for (int kind = 0; kind < 2 && st == SV_OK && e == hipSuccess; ++kind)
    for (int i = 0; i < cfg->n_stages && e == hipSuccess; ++i) {
      float* p = nullptr;
      e = hipMalloc(&p, m_bytes);
      if (e == hipSuccess) { s->m[kind].push_back(p); e = hipMemset(p, 0, m_bytes); }     // m_0 = 0
    }
  if (st == SV_OK && e == hipSuccess) e = hipMalloc(&s->mask_dev, 2 * (size_t)d);
  if (st == SV_OK && e == hipSuccess && (cfg->metric_mask & SV_M_SW) && d <= 32 && cfg->n_dirs % 32 == 0 && cfg->D % 64 == 0 &&
      sv_sw_row_len(cfg->T) <= 16384) {               // optional: without them the EMA itself is projected in every check
    const size_t p_bytes = (size_t)cfg->n_dirs * (size_t)sv_sw_row_len(cfg->T) * sizeof(float);
    bool ok = hipMalloc(&s->cproj, p_bytes * d) == hipSuccess;
    for (int kind = 0; kind < 2 && ok; ++kind)
      for (int i = 0; i < cfg->n_stages && ok; ++i) {
        float* p = nullptr;
        ok = hipMalloc(&p, p_bytes) == hipSuccess;
        if (ok) { s->pm[kind].push_back(p); ok = hipMemset(p, 0, p_bytes) == hipSuccess; }     // projections of m_0 = 0
        float* q = nullptr;
        ok = ok && hipMalloc(&q, p_bytes) == hipSuccess;
        if (ok) { s->ps[kind].push_back(q); s->sorted_ok[kind].push_back(0); }
      }
    if (ok && (hipMalloc(&s->pm_next, p_bytes) != hipSuccess || hipMemset(s->pm_next, 0, p_bytes) != hipSuccess ||
               hipEventCreateWithFlags(&s->checked, hipEventDisableTiming | hipEventReleaseToSystem) != hipSuccess)) {       // optional: without it behind the verdicts
      if (s->pm_next) (void)hipFree(s->pm_next);
      s->pm_next = nullptr;
      (void)hipGetLastError();
    }
    if (!ok) {
      (void)hipGetLastError();
      for (int kind = 0; kind < 2; ++kind)
        for (std::vector<float*>* v : {&s->pm[kind], &s->ps[kind]}) { for (float* p : *v) (void)hipFree(p); v->clear(); }
      if (s->cproj) { (void)hipFree(s->cproj); s->cproj = nullptr; }
    }
  }
  if (st == SV_OK && e == hipSuccess && d <= 32) {  // optional: without it the EMA update reads the signals itself
    if (hipMalloc(&s->sum_dev, m_bytes) != hipSuccess) { s->sum_dev = nullptr; (void)hipGetLastError(); }
  }
  if (st == SV_OK && e == hipSuccess) e = hipHostMalloc((void**)&s->res_host, sizeof(sv_result) * d, hipHostMallocDefault);
  if (st == SV_OK && e == hipSuccess) e = hipHostMalloc((void**)&s->sw_host, sizeof(float) * d, hipHostMallocDefault);
  if (st == SV_OK && e == hipSuccess) e = hipHostMalloc((void**)&s->mask_host, 2 * (size_t)d, hipHostMallocDefault);
  if (st != SV_OK || e != hipSuccess) {
    sv_sentinel_destroy(s);
    return st != SV_OK ? st : (e == hipErrorOutOfMemory ? SV_ENOMEM : SV_EHIP);
  }
  s->tainted.assign((size_t)cfg->n_stages * d, 0);
  *out = s;
  return SV_OK;
}

void sv_sentinel_destroy(sv_sentinel* s) {
  if (!s) return;
  for (int kind = 0; kind < 2; ++kind) {
    for (float* p : s->m[kind]) (void)hipFree(p);
    for (sv_policy* p : s->pol[kind]) sv_policy_destroy(p);
  }
  if (s->mask_dev) (void)hipFree(s->mask_dev);
  if (s->sum_dev) (void)hipFree(s->sum_dev);
  for (int kind = 0; kind < 2; ++kind)
    for (const std::vector<float*>* v : {&s->pm[kind], &s->ps[kind]})
      for (float* p : *v) (void)hipFree(p);
  if (s->cproj) (void)hipFree(s->cproj);
  if (s->pm_next) (void)hipFree(s->pm_next);
  if (s->checked) (void)hipEventDestroy(s->checked);
  if (s->res_host) (void)hipHostFree(s->res_host);
  if (s->sw_host) (void)hipHostFree(s->sw_host);
  if (s->mask_host) (void)hipHostFree(s->mask_host);
  delete s;
}

const char* sv_sentinel_last_error(const sv_sentinel* s) { return s ? s->err : "sentinel is NULL"; }

sv_status sv_sentinel_begin_iteration(sv_sentinel* s, int32_t warmup) {
  if (!s) return SV_EINVAL;
  std::fill(s->tainted.begin(), s->tainted.end(), (uint8_t)0);
  s->warm = warmup != 0;
  return SV_OK;
}

sv_status sv_sentinel_forward(sv_sentinel* s, int32_t stage, const void* h, int32_t dtype, uint8_t* tainted_out, double* gamma_out,
                              void* stream) {
  if (!s) return SV_EINVAL;
  sv_status st = check_stage(s, stage, h, dtype, tainted_out);
  if (st != SV_OK) return st;
  hipStream_t hs = (hipStream_t)stream;
  const int d = s->cfg.n_workers, p = s->cfg.n_stages;
  std::vector<double> gamma;
  sv_policy* pol = s->pol[0][stage];
  std::vector<uint8_t> upstream(d, 0), banned(d, 0), skip(d, 0);
  if (!s->warm) {                                  // excluded whatever this check says: banned or tainted upstream
    for (int r = 0; r < d; ++r)
      for (int s2 = 0; s2 < p; ++s2) upstream[r] |= s->tainted[(size_t)s2 * d + r];
    SN_SV(s, sv_policy_state(pol, nullptr, banned.data(), nullptr, nullptr, nullptr, nullptr));
    for (int r = 0; r < d; ++r) skip[r] = banned[r] | upstream[r];
  }
  bool summed = false;
  CallEma ema{s, 0, stage, s->cfg.beta_h, hs};
  st = gamma_of(s, h, dtype, ema, skip.data(), &summed, gamma, hs);
  if (st != SV_OK) return st;
  if (gamma_out) memcpy(gamma_out, gamma.data(), gamma.size() * sizeof(double));
  uint8_t* excl = s->mask_host + d;
  if (s->warm) {
    SN_SV(s, sv_policy_warmup(pol, gamma.data()));
    for (int r = 0; r < d; ++r) { tainted_out[r] = 0; excl[r] = 0; }
  } else {
    SN_SV(s, sv_policy_step(pol, gamma.data(), upstream.data(), nullptr, tainted_out));
    SN_SV(s, sv_policy_state(pol, nullptr, banned.data(), nullptr, nullptr, nullptr, nullptr));
    for (int r = 0; r < d; ++r) {
      if (tainted_out[r]) s->tainted[(size_t)stage * d + r] = 1;
      excl[r] = banned[r] | upstream[r] | tainted_out[r];
    }
  }
  return update_ema(s, ema, h, dtype, excl, skip.data(), summed);
}

sv_status sv_sentinel_backward(sv_sentinel* s, int32_t stage, void* g, int32_t dtype, uint8_t* tainted_out, double* gamma_out, void* stream) {
  if (!s) return SV_EINVAL;
  sv_status st = check_stage(s, stage, g, dtype, tainted_out);
  if (st != SV_OK) return st;
  hipStream_t hs = (hipStream_t)stream;
  const int d = s->cfg.n_workers, p = s->cfg.n_stages;
  std::vector<double> gamma;
  sv_policy* pol = s->pol[1][stage];
  std::vector<uint8_t> down(d, 0), banned(d, 0), skip(d, 0);
  if (!s->warm) {                                  // excluded whatever this check says (short of a majority reset): banned,
                                                   // tainted here on the way forward, or tainted at a later stage
    for (int r = 0; r < d; ++r)
      for (int s2 = stage + 1; s2 < p; ++s2) down[r] |= s->tainted[(size_t)s2 * d + r];
    SN_SV(s, sv_policy_state(pol, nullptr, banned.data(), nullptr, nullptr, nullptr, nullptr));
    for (int r = 0; r < d; ++r) skip[r] = banned[r] | s->tainted[(size_t)stage * d + r] | down[r];
  }
  bool summed = false;
  CallEma ema{s, 1, stage, s->cfg.beta_g, hs};
  st = gamma_of(s, g, dtype, ema, skip.data(), &summed, gamma, hs);
  if (st != SV_OK) return st;
  if (gamma_out) memcpy(gamma_out, gamma.data(), gamma.size() * sizeof(double));
  uint8_t* repl = s->mask_host;
  uint8_t* excl = s->mask_host + d;
  if (s->warm) {
    SN_SV(s, sv_policy_warmup(pol, gamma.data()));
    for (int r = 0; r < d; ++r) { tainted_out[r] = 0; repl[r] = 0; excl[r] = 0; }
  } else {
    SN_SV(s, sv_policy_step(pol, gamma.data(), nullptr, down.data(), tainted_out));
    SN_SV(s, sv_policy_state(pol, nullptr, banned.data(), nullptr, nullptr, nullptr, nullptr));
    for (int r = 0; r < d; ++r) {
      if (tainted_out[r]) s->tainted[(size_t)stage * d + r] = 1;
      repl[r] = s->tainted[(size_t)stage * d + r];           // includes a forward-pass taint at this very stage
      excl[r] = banned[r] | repl[r];
    }
  }
  // the EMA reads only signals that are not replaced, and the replacement reads what m was before it is updated
  bool any_repl = false;
  for (int r = 0; r < d; ++r) any_repl |= repl[r] != 0;
  if (any_repl) SN_HIP(s, hipMemcpyAsync(s->mask_dev, s->mask_host, 2 * (size_t)d, hipMemcpyHostToDevice, hs));
  if (any_repl) SN_SV(s, sv_replace_with_ema(s->ctx, g, s->cfg.T * s->cfg.D, d, dtype, s->mask_dev, ema.now(), s->cfg.T, s->cfg.D, hs));
  // (the sum the score pass left was taken before the replacement, over signals that are not replaced)
  return update_ema(s, ema, g, dtype, excl, skip.data(), summed, /*mask_uploaded=*/any_repl);
}

sv_status sv_sentinel_state(const sv_sentinel* s, int32_t stage, int32_t kind, const float** ema_dev, int32_t* violations, uint8_t* banned,
                            double* lower, double* upper, double* k) {
  if (!s || stage < 0 || stage >= s->cfg.n_stages || (kind != 0 && kind != 1)) return SV_EINVAL;
  if (ema_dev) *ema_dev = s->m[kind][stage];
  return sv_policy_state(s->pol[kind][stage], violations, banned, lower, upper, k, nullptr);
}

sv_status sv_sentinel_counters(const sv_sentinel* s, int64_t* counts) {
  if (!s || !counts) return SV_EINVAL;
  counts[0] = s->n_calls; counts[1] = s->n_from_sum; counts[2] = s->n_from_signals; counts[3] = s->n_sw_carried;
  return SV_OK;
}

sv_status sv_sentinel_read_ema(sv_sentinel* s, int32_t stage, int32_t kind, float* out_host, void* stream) {
  if (!s || stage < 0 || stage >= s->cfg.n_stages || (kind != 0 && kind != 1) || !out_host) return SV_EINVAL;
  hipStream_t hs = (hipStream_t)stream;
  SN_HIP(s, hipMemcpyAsync(out_host, s->m[kind][stage], (size_t)s->cfg.T * s->cfg.D * sizeof(float), hipMemcpyDeviceToHost, hs));
  SN_HIP(s, hipStreamSynchronize(hs));
  return SV_OK;
}

}  // extern "C"
