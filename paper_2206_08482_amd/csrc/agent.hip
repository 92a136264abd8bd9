// The agent kernel for bf16 models: which rows per workgroup.
#include "agent_kernel.h"

namespace {
using namespace gmi_agent;

void fill_model(const gmi_model* m, const float* obs, int n, float* value, AgentArgs* a) {
  const ModelLayout& L = m->L;
  for (int net = 0; net < 2; ++net)
    for (int l = 0; l < L.n_layers; ++l) {
      const LayerInfo& li = L.net[net][l];
      a->l[net][l] = {reinterpret_cast<const uint4*>(m->shadow + li.sh_wf), reinterpret_cast<const float*>(m->shadow + li.sh_b),
                      nullptr, li.in_pad, li.out_pad};
    }
  a->nl = L.n_layers;
  a->n = n; a->O = L.obs_dim; a->A = L.act_dim;
  a->log_std = reinterpret_cast<const float*>(m->shadow + L.sh_logstd);
  a->obs = obs; a->value = value;
  a->vec_obs = ((uintptr_t)obs & 15) == 0 ? 1 : 0;
}

// units: nets or, for values_kernel, slots per row tile.
int launch_rows(gmi_instance* g, AgentArgs& a, int64_t units, bool sample, int64_t weight_bytes) {
  // Rows per workgroup, us for 32 / 64 / 128 rows:
  //   32 while all workgroups are resident at once (two per compute unit): 5000 rows of 108:400:200:100:21 16 / 18;
  //   128 where two such tiles fit a compute unit and there are enough of them: 32768 rows of 45:128:128:12 31 / 20 / 15
  //   (16384 rows: 17 / 11 / 12);
  //   64 where two of those fit (262144 rows of 60:256:128:64:8: 286 / 164; with 8 weight blocks in flight instead of 4,
  //   which takes 128 registers instead of 96, 185), or where the weights are so many that fetching them half as often
  //   counts (65536 rows of 200:512:512:300:20: 258 / 228, 20000: 85 / 88);
  //   else 32 (20000 rows of 108:400:200:100:21: 40 / 47).
  const int64_t slots = 2 * (int64_t)g->cu_count;
  auto groups = [&](int rt) { return (int64_t)((a.n + 32 * rt - 1) / (32 * rt)) * units; };
  auto per_cu = [&](int rt) { return (int)(kLdsMax / agent_lds<Bf16>(a, rt, sample)); };
  if (per_cu(1) < 1) return GMI_ERR_UNSUPPORTED;
  const bool values = a.T > 0;
  if (groups(1) > slots && per_cu(4) >= 2 && groups(4) >= slots)
    return values ? launch_slots<Bf16, 4, 4, 2, 4>(g, a) : launch<Bf16, 4, 4, 2, 4>(g, a, (int)units, sample);
  if (groups(1) > slots && (per_cu(2) >= 2 || (per_cu(2) == 1 && weight_bytes > (1 << 20) && groups(1) >= 8 * slots)))
    return values ? launch_slots<Bf16, 2, 4, 2, 4>(g, a) : launch<Bf16, 2, 4, 2, 4>(g, a, (int)units, sample);
  return values ? launch_slots<Bf16, 1, 8, 1, 4>(g, a) : launch<Bf16, 1, 8, 1, 4>(g, a, (int)units, sample);
}

}  // namespace

namespace gmi {

// act NULL: the policy's means (mu_out) and the values only.  Returns GMI_ERR_UNSUPPORTED (no error message) where the per-layer
// path or the row-tile kernel has to be used instead.
int launch_agent(gmi_instance* g, gmi_model* m, const float* obs, int n, uint64_t seed, uint32_t step, uint32_t env_offset,
                 float* act, float* logp, float* value, float* mu_out, bool do_policy) {
  const ModelLayout& L = m->L;
  if (L.dtype != GMI_DTYPE_BF16) return GMI_ERR_UNSUPPORTED;
  if (use_tile_forward(g, m, n)) return GMI_ERR_UNSUPPORTED;
  AgentArgs a = {};
  fill_model(m, obs, n, value, &a);
  a.net0 = do_policy ? 0 : 1;
  a.lp_blocks = has_tile_forward(L) ? 0 : 1;      // the order in which this model's rollout_collect sums
  a.k0 = (uint32_t)seed; a.k1 = (uint32_t)(seed >> 32); a.step = step; a.env_offset = env_offset;
  a.act = act; a.logp = logp; a.mu_out = mu_out;
  return launch_rows(g, a, do_policy ? 2 : 1, act != nullptr, L.weight_bytes);
}

int launch_values(gmi_instance* g, gmi_model* m, const float* obs, int T, int n, int64_t ld, float* value, const float* obs_last,
                  float* value_last) {
  const int tile = launch_forward_values(g, m, obs, T, n, ld, value, obs_last, value_last);
  if (tile != GMI_ERR_UNSUPPORTED) return tile;
  const int per = std::max(1, (1 << 30) / ((n + 31) / 32) - 1);      // slots of a launch: its items are a 32-bit count
  for (int t0 = 0; t0 < T; t0 += per) {
    AgentArgs a = {};
    a.obs_step = ld * m->L.obs_dim; a.val_step = ld;
    fill_model(m, obs + t0 * a.obs_step, n, value + t0 * a.val_step, &a);
    a.net0 = 1;
    a.T = std::min(T - t0, per);
    if (a.T > 1 && (a.obs_step & 3) != 0) a.vec_obs = 0;
    if (t0 + a.T == T) {
      a.obs_last = obs_last; a.value_last = value_last;
      if (((uintptr_t)obs_last & 15) != 0) a.vec_obs = 0;
    }
    const int rc = launch_rows(g, a, a.T + (a.value_last ? 1 : 0), false, m->L.weight_bytes);
    if (rc != GMI_OK) return rc;
  }
  return GMI_OK;
}

}  // namespace gmi
