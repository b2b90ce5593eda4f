// C ABI of the adjoint lattice-Boltzmann library (lbm_adj.h): argument and state
// checks, context lifetime, the static device workspace.  The work behind each
// call is in ops.hpp, reached through dispatch().
#include <mutex>

#include "context.hpp"

using namespace lbmh;

namespace {

// ------------------------------------------------- static device workspace
// For callers that cannot allocate device memory (code under HIP graph
// capture, allocation-free serving loops): lbm_create_static carves the
// context from this file-scope array instead of a caller's workspace.  Each
// device holds its own copy until the process ends; host code reaches it only
// through the address hipGetSymbolAddress returns for the current device (the
// array's name in host code is a host-side stand-in, not a device address).
constexpr uint64_t kStaticWorkspaceBytes = 128ull << 20;
constexpr int kMaxDevices = 64;
static __device__ __align__(256) unsigned char scratch[kStaticWorkspaceBytes];

struct StaticSlot {
  void* ptr = nullptr;  // device address of scratch on this device
  bool busy = false;    // a static context is alive on this device
};
std::mutex g_static_mu;
StaticSlot g_static[kMaxDevices];

// Runs a checked batch, one kernel variant after the other.
template <template <class> class F, class... A>
lbm_status dispatch_batch(lbm_ctx* const* cs, int n, A... a) {
  for (int k = 0; k < n; ++k) {
    lbm_ctx* part[kBatchMax];
    const int m = batch_part(cs, n, k, part);
    if (m == 0) continue;
    const lbm_status s = dispatch<F>(part[0], (lbm_ctx* const*)part, m, a...);
    if (s != LBM_OK) {
      cs[0]->err = part[0]->err;
      return s;
    }
  }
  return LBM_OK;
}

}  // namespace

// ================================================================= C ABI
extern "C" {

lbm_status lbm_required_bytes(const lbm_config* cfg, uint64_t* bytes_out) {
  if (!bytes_out) return LBM_EINVAL;
  Plan p;
  lbm_status s = make_plan(cfg, &p, nullptr);
  if (s != LBM_OK) return s;
  *bytes_out = p.total;
  return LBM_OK;
}

lbm_status lbm_create(const lbm_config* cfg, void* hip_stream, void* workspace_dev, uint64_t workspace_bytes,
                      lbm_ctx** ctx_out) {
  if (!ctx_out) return LBM_EINVAL;
  *ctx_out = nullptr;
  Plan p;
  std::string why;
  lbm_status s = make_plan(cfg, &p, &why);
  if (s != LBM_OK) {
    fprintf(stderr, "lbm_create: %s\n", why.c_str());
    return s;
  }
  if (!workspace_dev || ((uintptr_t)workspace_dev % kAlign) != 0) return LBM_EINVAL;
  if (workspace_bytes < p.total) return LBM_ENOMEM;
  lbm_ctx* c = new lbm_ctx();
  c->cfg = *cfg;
  c->plan = p;
  c->stream = (hipStream_t)hip_stream;
  c->ws = (char*)workspace_dev;
  c->ws_bytes = workspace_bytes;
  char* q = c->ws;
  c->w = q;
  q += p.node_bytes;
  c->grad = q;
  q += p.node_bytes;
  c->glob = (double*)q;
  q += align_up(kGlobBytes);
  c->desc = q;
  q += align_up(kDescBytes);
  if (p.inplace) {
    c->lam[0] = c->lam[1] = q;  // one adjoint buffer, rewritten in place
    q += p.state_bytes;
    c->pp[0] = c->pp[1] = nullptr;
    if (cfg->nsteps > 0 && p.C < cfg->nsteps) {  // checkpointed: a working buffer of its own
      c->work = q;
      q += p.state_bytes;
    }
  } else {
    for (int i = 0; i < 2; ++i) {
      c->lam[i] = q;
      q += p.state_bytes;
    }
    for (int i = 0; i < 2; ++i) {
      c->pp[i] = q;
      q += p.state_bytes;
    }
  }
  c->ckpt = q;
  q += (uint64_t)p.S * p.state_bytes;
  c->mom = q;
  q += (uint64_t)p.C * p.mom_bytes;
  if (p.W > 1) {
    c->win = q;
    q += p.win_bytes;
  }
  if (p.inplace && !c->work) c->work = c->ckpt;  // store-all / unrecorded: the state lives in ckpt[0]
  reset_times(c);
  s = dispatch<RunReset>(c);
  if (s == LBM_OK) s = dispatch<RunWriteStatic>(c);
  if (s != LBM_OK) {
    delete c;
    return s;
  }
  *ctx_out = c;
  return LBM_OK;
}

lbm_status lbm_create_static(const lbm_config* cfg, void* hip_stream, lbm_ctx** ctx_out) {
  if (!ctx_out) return LBM_EINVAL;
  *ctx_out = nullptr;
  uint64_t need = 0;
  lbm_status s = lbm_required_bytes(cfg, &need);
  if (s != LBM_OK) return s;
  if (need > kStaticWorkspaceBytes) {
    fprintf(stderr, "lbm_create_static: the configuration needs %llu bytes, the static workspace holds %llu\n",
            (unsigned long long)need, (unsigned long long)kStaticWorkspaceBytes);
    return LBM_ENOMEM;
  }
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return LBM_EHIP;
  std::lock_guard<std::mutex> lock(g_static_mu);
  StaticSlot& slot = g_static[dev];
  if (!slot.ptr) {
    void* ptr = nullptr;
    hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr) {
      fprintf(stderr, "lbm_create_static: hipGetSymbolAddress: %s\n", hipGetErrorString(e));
      return LBM_EHIP;
    }
    slot.ptr = ptr;
  }
  if (slot.busy) {
    fprintf(stderr, "lbm_create_static: another static context is alive on device %d\n", dev);
    return LBM_ESTATE;
  }
  s = lbm_create(cfg, hip_stream, slot.ptr, kStaticWorkspaceBytes, ctx_out);
  if (s != LBM_OK) return s;
  slot.busy = true;
  (*ctx_out)->static_dev = dev;
  return LBM_OK;
}

uint64_t lbm_static_workspace_bytes(void) { return kStaticWorkspaceBytes; }

lbm_status lbm_destroy(lbm_ctx* ctx) {
  if (!ctx) return LBM_EINVAL;
  if (ctx->static_dev >= 0) {
    // the next static context on this device reuses the array: let this
    // context's queued work finish first (unless its stream is being captured)
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(ctx->stream, &cs) == hipSuccess && cs == hipStreamCaptureStatusNone)
      (void)hipStreamSynchronize(ctx->stream);
    std::lock_guard<std::mutex> lock(g_static_mu);
    g_static[ctx->static_dev].busy = false;
  }
  delete ctx;
  return LBM_OK;
}

lbm_status lbm_set_design(lbm_ctx* c, const void* w_dev) {
  if (!c) return LBM_EINVAL;
  if (!w_dev) return fail(c, LBM_EINVAL, "set_design: NULL design field");
  lbm_status s = dispatch<RunSetDesign>(c, w_dev);
  if (s != LBM_OK) return s;
  c->design_set = true;
  // a recorded trajectory or adjoint of another design is no longer valid; once an
  // adjoint has run, recomputed segments may have overwritten the buffer that held
  // the primal state, so calls that read it wait for lbm_reset / lbm_set_state
  if (c->adj_started) c->state_lost = true;
  if (c->rec_len > 0 || c->adj_started) {
    c->rec_len = 0;
    c->rec_open = false;
    c->adj_started = false;
    c->t_adj = -1;
  }
  return LBM_OK;
}

lbm_status lbm_reset(lbm_ctx* c) {
  if (!c) return LBM_EINVAL;
  reset_times(c);
  return dispatch<RunReset>(c);
}

lbm_status lbm_set_state(lbm_ctx* c, const double* f_dev, const double* g_dev) {
  if (!c) return LBM_EINVAL;
  if (!f_dev) return fail(c, LBM_EINVAL, "set_state: NULL f");
  reset_times(c);
  return dispatch<RunSetState>(c, f_dev, g_dev);
}

lbm_status lbm_primal_steps(lbm_ctx* c, int64_t nsteps, int32_t record) {
  if (!c) return LBM_EINVAL;
  if (nsteps < 0) return fail(c, LBM_EINVAL, "primal_steps: negative count");
  if (!c->design_set) return fail(c, LBM_ESTATE, "primal_steps: no design field set");
  if (c->adj_started) return fail(c, LBM_ESTATE, "primal_steps: adjoint started; call lbm_reset first");
  if (c->state_lost) return fail(c, LBM_ESTATE, "primal_steps: primal state consumed by an adjoint; call lbm_reset");
  if (record && c->os_active) return fail(c, LBM_ESTATE, "primal_steps: one-shot running; call lbm_reset first");
  if (record && c->plan.inplace && c->cfg.nsteps == 0)
    return fail(c, LBM_ESTATE, "primal_steps: an in-place context with no horizon does not record");
  if (record) {
    if (!(c->rec_open && c->t == c->rec_len))
      return fail(c, LBM_ESTATE, "primal_steps: recording must start at t = 0 or continue a recorded run");
    if (c->t + nsteps > c->cfg.nsteps)
      return fail(c, LBM_EINVAL, "primal_steps: recorded run of %lld steps exceeds the horizon %lld",
                  (long long)(c->t + nsteps), (long long)c->cfg.nsteps);
  }
  if (nsteps == 0) return LBM_OK;
  Range r(record ? "lbm_primal_steps (recorded)" : "lbm_primal_steps");
  lbm_status s = dispatch<RunPrimal>(c, nsteps, (int)(record != 0));
  if (record) {
    c->rec_len = c->t;
  } else {
    c->rec_open = false;
  }
  return s;
}

lbm_status lbm_objective_async(lbm_ctx* c, double* J_dev) {
  if (!c) return LBM_EINVAL;
  if (c->adj_started || c->state_lost) return fail(c, LBM_ESTATE, "objective: primal state consumed by the adjoint");
  return dispatch<RunObjective>(c, J_dev);
}

lbm_status lbm_objective(lbm_ctx* c, double* J_host, double* globals_host) {
  if (!c) return LBM_EINVAL;
  if (c->adj_started || c->state_lost) return fail(c, LBM_ESTATE, "objective: primal state consumed by the adjoint");
  lbm_status s = dispatch<RunObjective>(c, (double*)nullptr);
  if (s != LBM_OK) return s;
  double h[kNG + 1];
  hipError_t e = hipMemcpyAsync(h, c->glob, sizeof h, hipMemcpyDeviceToHost, c->stream);
  if (e != hipSuccess) return fail(c, LBM_EHIP, "objective: %s", hipGetErrorString(e));
  s = sync_check(c, "objective");
  if (s != LBM_OK) return s;
  if (J_host) *J_host = h[kNG];
  if (globals_host) std::memcpy(globals_host, h, kNG * sizeof(double));
  if (!std::isfinite(h[kNG])) return fail(c, LBM_ENONFINITE, "objective is not finite");
  return LBM_OK;
}

lbm_status lbm_adjoint_steps(lbm_ctx* c, int64_t nsteps) {
  if (!c) return LBM_EINVAL;
  if (nsteps < 0) return fail(c, LBM_EINVAL, "adjoint_steps: negative count");
  if (c->os_active) return fail(c, LBM_ESTATE, "adjoint_steps: one-shot running; call lbm_reset first");
  if (c->plan.inplace && c->cfg.nsteps == 0)
    return fail(c, LBM_ESTATE, "adjoint_steps: an in-place context with no horizon keeps no trajectory");
  if (!c->adj_started) {
    if (!c->design_set) return fail(c, LBM_ESTATE, "adjoint_steps: no design field set");
    if (!(c->rec_open && c->t == c->rec_len))
      return fail(c, LBM_ESTATE, "adjoint_steps: needs a recorded run ending at the current time");
    if (nsteps > c->rec_len) return fail(c, LBM_EINVAL, "adjoint_steps: more steps than recorded");
    if (c->plan.W > 1 && !window_complete(c))
      return fail(c, LBM_ESTATE, "adjoint_steps: the time-averaged objective needs a recorded run to the horizon");
  } else if (nsteps > c->t_adj) {
    return fail(c, LBM_EINVAL, "adjoint_steps: only %lld steps remain", (long long)c->t_adj);
  }
  Range r("lbm_adjoint_steps");
  return dispatch<RunAdjoint>(c, nsteps);
}

lbm_status lbm_gradient(lbm_ctx* c, void* grad_dev) {
  if (!c) return LBM_EINVAL;
  if (!grad_dev) return fail(c, LBM_EINVAL, "gradient: NULL output");
  if (!(c->adj_started && c->t_adj == 0) && !c->os_active)
    return fail(c, LBM_ESTATE, "gradient: adjoint has not reached t = 0 and no one-shot iteration ran");
  return dispatch<RunGradient>(c, grad_dev);
}

lbm_status lbm_gradient_penalty(lbm_ctx* c, double penalty, void* grad_dev) {
  if (!c) return LBM_EINVAL;
  if (!grad_dev) return fail(c, LBM_EINVAL, "gradient_penalty: NULL output");
  if (!std::isfinite(penalty)) return fail(c, LBM_EINVAL, "gradient_penalty: non-finite weight");
  if (!(c->adj_started && c->t_adj == 0) && !c->os_active)
    return fail(c, LBM_ESTATE, "gradient_penalty: adjoint has not reached t = 0 and no one-shot iteration ran");
  return dispatch<RunGradientPenalty>(c, penalty, grad_dev);
}

lbm_status lbm_fields(lbm_ctx* c, double* rho_dev, double* u_dev, double* s_dev) {
  if (!c) return LBM_EINVAL;
  if (!rho_dev || !u_dev) return fail(c, LBM_EINVAL, "fields: NULL output");
  if (c->adj_started || c->state_lost) return fail(c, LBM_ESTATE, "fields: primal state consumed by the adjoint");
  return dispatch<RunFields>(c, rho_dev, u_dev, s_dev);
}

lbm_status lbm_get_state(lbm_ctx* c, double* f_dev, double* g_dev) {
  if (!c) return LBM_EINVAL;
  if (!f_dev) return fail(c, LBM_EINVAL, "get_state: NULL output");
  if (c->adj_started || c->state_lost)
    return fail(c, LBM_ESTATE, "get_state: primal state consumed by the adjoint");
  return dispatch<RunGetState>(c, f_dev, g_dev);
}

lbm_status lbm_get_adjoint(lbm_ctx* c, double* lf_dev, double* lg_dev) {
  if (!c) return LBM_EINVAL;
  if (!lf_dev) return fail(c, LBM_EINVAL, "get_adjoint: NULL output");
  if (!c->adj_started && !c->os_active) return fail(c, LBM_ESTATE, "get_adjoint: no adjoint state");
  return dispatch<RunGetAdjoint>(c, lf_dev, lg_dev);
}

lbm_status lbm_export_maps(lbm_ctx* c, uint8_t* mask_dev, int64_t* src_dev) {
  if (!c) return LBM_EINVAL;
  return dispatch<RunMaps>(c, mask_dev, src_dev);
}

lbm_status lbm_oneshot_steps(lbm_ctx* c, int64_t nsteps, double zeta, double penalty) {
  if (!c) return LBM_EINVAL;
  if (nsteps < 0) return fail(c, LBM_EINVAL, "oneshot_steps: negative count");
  if (!std::isfinite(zeta) || !std::isfinite(penalty)) return fail(c, LBM_EINVAL, "oneshot_steps: non-finite step");
  if (!c->design_set) return fail(c, LBM_ESTATE, "oneshot_steps: no design field set");
  if (c->adj_started || c->state_lost)
    return fail(c, LBM_ESTATE, "oneshot_steps: unsteady adjoint started; call lbm_reset first");
  Range r("lbm_oneshot_steps");
  return dispatch<RunOneshot>(c, nsteps, zeta, penalty);
}

lbm_status lbm_get_design(lbm_ctx* c, void* w_dev) {
  if (!c) return LBM_EINVAL;
  if (!w_dev) return fail(c, LBM_EINVAL, "get_design: NULL output");
  if (!c->design_set) return fail(c, LBM_ESTATE, "get_design: no design field set");
  return dispatch<RunGetDesign>(c, w_dev);
}

lbm_status lbm_times(const lbm_ctx* c, int64_t* t, int64_t* recorded, int64_t* t_adj) {
  if (!c) return LBM_EINVAL;
  if (t) *t = c->t;
  if (recorded) *recorded = c->rec_len;
  if (t_adj) *t_adj = c->adj_started ? c->t_adj : -1;
  return LBM_OK;
}

lbm_status lbm_plan(const lbm_ctx* c, int64_t* interval, int64_t* n_checkpoints, int64_t* n_moment_sets,
                    uint64_t* state_bytes) {
  if (!c) return LBM_EINVAL;
  if (interval) *interval = c->plan.C;
  if (n_checkpoints) *n_checkpoints = c->plan.S;
  if (n_moment_sets) *n_moment_sets = c->plan.C;
  if (state_bytes) *state_bytes = c->plan.state_bytes;
  return LBM_OK;
}

lbm_status lbm_primal_steps_batch(lbm_ctx* const* ctxs, int32_t n, int64_t nsteps, int32_t record) {
  lbm_status s = check_batch(ctxs, n);
  if (s != LBM_OK) return s;
  lbm_ctx* c0 = ctxs[0];
  if (nsteps < 0) return fail(c0, LBM_EINVAL, "primal_steps_batch: negative count");
  for (int k = 0; k < n; ++k) {
    lbm_ctx* c = ctxs[k];
    if (!c->design_set) return fail(c0, LBM_ESTATE, "primal_steps_batch: context %d has no design", k);
    if (c->adj_started || c->state_lost)
      return fail(c0, LBM_ESTATE, "primal_steps_batch: context %d is in its adjoint", k);
    if (record && !(c->rec_open && c->t == c->rec_len))
      return fail(c0, LBM_ESTATE, "primal_steps_batch: context %d cannot continue recording", k);
    if (record && c->t + nsteps > c->cfg.nsteps)
      return fail(c0, LBM_EINVAL, "primal_steps_batch: context %d would exceed its horizon", k);
  }
  if (nsteps == 0) return LBM_OK;
  Range r("lbm_primal_steps_batch");
  s = dispatch_batch<RunPrimalBatch>(ctxs, (int)n, nsteps, (int)(record != 0));
  for (int k = 0; k < n; ++k) {
    if (record) ctxs[k]->rec_len = ctxs[k]->t;
    else ctxs[k]->rec_open = false;
  }
  return s;
}

lbm_status lbm_adjoint_steps_batch(lbm_ctx* const* ctxs, int32_t n, int64_t nsteps) {
  lbm_status s = check_batch(ctxs, n);
  if (s != LBM_OK) return s;
  lbm_ctx* c0 = ctxs[0];
  if (nsteps < 0) return fail(c0, LBM_EINVAL, "adjoint_steps_batch: negative count");
  for (int k = 0; k < n; ++k) {
    lbm_ctx* c = ctxs[k];
    if (!c->adj_started) {
      if (!c->design_set) return fail(c0, LBM_ESTATE, "adjoint_steps_batch: context %d has no design", k);
      if (!(c->rec_open && c->t == c->rec_len))
        return fail(c0, LBM_ESTATE, "adjoint_steps_batch: context %d has no complete recorded run", k);
      if (nsteps > c->rec_len) return fail(c0, LBM_EINVAL, "adjoint_steps_batch: context %d: too many steps", k);
    } else if (nsteps > c->t_adj) {
      return fail(c0, LBM_EINVAL, "adjoint_steps_batch: context %d: only %lld steps remain", k,
                  (long long)c->t_adj);
    }
  }
  if (nsteps == 0) {
    // still seed, so that a zero-step call behaves like the single-context form
    return dispatch_batch<RunAdjointBatch>(ctxs, (int)n, (int64_t)0);
  }
  Range r("lbm_adjoint_steps_batch");
  return dispatch_batch<RunAdjointBatch>(ctxs, (int)n, nsteps);
}

const char* lbm_last_error(const lbm_ctx* c) { return c ? c->err.c_str() : "NULL context"; }

const char* lbm_status_string(lbm_status s) {
  switch (s) {
    case LBM_OK: return "ok";
    case LBM_EINVAL: return "invalid argument";
    case LBM_ENOMEM: return "workspace too small";
    case LBM_EHIP: return "HIP error";
    case LBM_ESTATE: return "invalid state";
    case LBM_ENONFINITE: return "non-finite objective";
  }
  return "unknown status";
}

}  // extern "C"
