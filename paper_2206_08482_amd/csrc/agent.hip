// The agent kernel for bf16 models: which rows per workgroup.
#include "agent_kernel.h"

namespace gmi {
using namespace gmi_agent;

// act NULL: the policy's means (mu_out) and the values only.  Returns GMI_ERR_UNSUPPORTED (no error message) where the per-layer
// path or the row-tile kernel has to be used instead.
int launch_agent(gmi_instance* g, gmi_model* m, const float* obs, int n, uint64_t seed, uint32_t step, uint32_t env_offset,
                 float* act, float* logp, float* value, float* mu_out, bool do_policy) {
  const ModelLayout& L = m->L;
  if (L.dtype != GMI_DTYPE_BF16) return GMI_ERR_UNSUPPORTED;
  if (use_tile_forward(m, n)) return GMI_ERR_UNSUPPORTED;
  AgentArgs a;
  const int nets = do_policy ? 2 : 1;
  for (int net = 0; net < 2; ++net)
    for (int l = 0; l < L.n_layers; ++l) {
      const LayerInfo& li = L.net[net][l];
      a.l[net][l] = {reinterpret_cast<const uint4*>(m->shadow + li.sh_wf), reinterpret_cast<const float*>(m->shadow + li.sh_b),
                     nullptr, li.in_pad, li.out_pad};
    }
  a.nl = L.n_layers; a.net0 = do_policy ? 0 : 1;
  a.n = n; a.O = L.obs_dim; a.A = L.act_dim;
  a.vec_obs = ((uintptr_t)obs & 15) == 0 ? 1 : 0;
  a.lp_blocks = has_tile_forward(L) ? 0 : 1;      // the order in which this model's rollout_collect sums
  a.k0 = (uint32_t)seed; a.k1 = (uint32_t)(seed >> 32); a.step = step; a.env_offset = env_offset;
  a.log_std = reinterpret_cast<const float*>(m->shadow + L.sh_logstd);
  a.obs = obs; a.act = act; a.logp = logp; a.value = value; a.mu_out = mu_out;
  // Rows per workgroup, us for 32 / 64 / 128 rows:
  //   32 while all workgroups are resident at once (two per compute unit): 5000 rows of 108:400:200:100:21 16 / 18;
  //   128 where two such tiles fit a compute unit and there are enough of them: 32768 rows of 45:128:128:12 31 / 20 / 15
  //   (16384 rows: 17 / 11 / 12);
  //   64 where two of those fit (262144 rows of 60:256:128:64:8: 286 / 164; with 8 weight blocks in flight instead of 4,
  //   which takes 128 registers instead of 96, 185), or where the weights are so many that fetching them half as often
  //   counts (65536 rows of 200:512:512:300:20: 258 / 228, 20000: 85 / 88);
  //   else 32 (20000 rows of 108:400:200:100:21: 40 / 47).
  const bool sample = act != nullptr;
  const int64_t slots = 2 * (int64_t)g->cu_count;
  auto groups = [&](int rt) { return (int64_t)((n + 32 * rt - 1) / (32 * rt)) * nets; };
  auto per_cu = [&](int rt) { return (int)(kLdsMax / agent_lds<Bf16>(a, rt, sample)); };
  if (per_cu(1) < 1) return GMI_ERR_UNSUPPORTED;
  if (groups(1) > slots && per_cu(4) >= 2 && groups(4) >= slots) return launch<Bf16, 4, 4, 2, 4>(g, a, nets, sample);
  if (groups(1) > slots && (per_cu(2) >= 2 || (per_cu(2) == 1 && L.weight_bytes > (1 << 20) && groups(1) >= 8 * slots)))
    return launch<Bf16, 2, 4, 2, 4>(g, a, nets, sample);
  return launch<Bf16, 1, 8, 1, 4>(g, a, nets, sample);
}

}  // namespace gmi
