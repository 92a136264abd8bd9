// Parts of the one-launch experience collection that do not depend on how the networks are evaluated: what the
// kernel knows about the simulator and the experience arrays, the simulator step of a tile of envs, and the random
// draws of a step (fused.hip: bf16 networks; f32.hip: fp32 networks).
#pragma once
#include "internal.h"
#include "rng.h"

namespace {

struct RolloutEnv {
  const float* log_std;
  float* obs_state;                 // [n, O]: in = state before the first step, out = state after the last
  const float* m_r;                 // [o4, ms] rows of [A B], zero padded
  uint32_t* episode_step;           // [n]
  int n, obs_dim, act_dim, o4, ms, T, ld_envs;
  int rows_per_wg;                  // envs owned by a workgroup: 16, 32 or 64
  int row_shift;                    // log2 of the threads that share an env outside the products: 512 / rows_per_wg
  int n_tiles;                      // ceil(n / rows_per_wg); the grid may be smaller (workgroups loop)
  int obs_vec;                      // 1 = observation rows are whole 16-byte pieces in the buffer
  uint32_t npr_magic;               // of the random blocks per env and step
  float noise_std, reward_scale;
  uint32_t done_period, done_threshold;
  uint32_t ak0, ak1, a_env_offset;  // agent's Philox key and env offset
  uint32_t ek0, ek1, e_env_offset;  // simulator's
  uint32_t step0;
  float* b_obs; float* b_act; float* b_logp; float* b_val; float* b_rew; uint8_t* b_done;
  float* last_value;
};

typedef float simx4 __attribute__((ext_vector_type(4)));

// Value of lane q of each group of four lanes.
template <int Q>
__device__ __forceinline__ float quad_lane(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), Q * 0x55, 0xF, 0xF, true));
}

// The tile's states into rows OS floats apart, by row_shift threads per env; rows past the last env and the floats beyond the
// state are zero.
__device__ __forceinline__ void load_states(const RolloutEnv& a, int r0, float* s_in, int OS, int tid) {
  const int r = tid >> a.row_shift, c = tid & ((1 << a.row_shift) - 1), nc = 1 << a.row_shift, O = a.obs_dim;
  const bool ok = r0 + r < a.n;
  const float* src = a.obs_state + (int64_t)min(r0 + r, a.n - 1) * O;
  for (int k = c; k < OS; k += nc) s_in[r * OS + k] = ok && k < O ? src[k] : 0.f;
}

// Decides the actions of a step -- action = mu + exp(log_std) * eps, an element per lane, beside the state in s_in; s_lp gets the
// log-density per block of 4 elements, its terms in index order -- and stores actions and observations.  s_ls: [A] log_std,
// [A] exp(log_std).
__device__ __forceinline__ void sample_and_store(const RolloutEnv& a, int r0, int64_t slot0, float* s_in, int OS, const float* s_mu,
                                                 int mu_stride, const float4* s_noise, int npr, int nba, const float* s_ls,
                                                 float* s_lp, int tid) {
  const int r = tid >> a.row_shift, c = tid & ((1 << a.row_shift) - 1), nc = 1 << a.row_shift;
  const int O = a.obs_dim, A = a.act_dim;
  const bool ok = r0 + r < a.n;
  const float* zp = reinterpret_cast<const float*>(s_noise + r * npr);
  float* row = s_in + r * OS;
  for (int j = c; j < 4 * nba; j += nc) {
    float term = 0.f;
    if (j < A) {
      const float z = zp[j], ls = s_ls[j];
      const float act = ok ? fmaf(s_ls[A + j], z, s_mu[r * mu_stride + j]) : 0.f;
      term = -0.5f * z * z - ls - 0.918938533204672742f;
      row[O + j] = act;
      if (ok) a.b_act[(slot0 + r) * A + j] = act;
    }
    const float lp = ((term + quad_lane<1>(term)) + quad_lane<2>(term)) + quad_lane<3>(term);
    if ((c & 3) == 0) s_lp[r * nba + (j >> 2)] = lp;
  }
  if (!ok) return;
  float* dst = a.b_obs + (slot0 + r) * O;
  if (a.obs_vec) {
    for (int k = 4 * c; k < O; k += 4 * nc) *reinterpret_cast<float4*>(dst + k) = *reinterpret_cast<const float4*>(row + k);
  } else {
    for (int k = c; k < O; k += nc) dst[k] = row[k];
  }
}

// Simulator step of a tile: next = A s + B act + noise_std * eps (or a fresh N(0,1) state after a done), rows of s_in -> put(row,
// first element, 4 elements), and the reward's partial sums per block of 4 elements (s_part).
// The products run on the 4x4x1 matrix instruction: 16 independent blocks, one k per instruction, whose result is the fmaf of
// its operands bit for bit (denormals included; checked on the device), so the sums are env_step's, k after k.  An item -- 16
// state elements (lane / 4 % 4: block of 4) of 16 envs (lane / 16: four of them) -- leaves every lane 4 consecutive elements of
// one env; four k cost two 16-byte LDS reads and four products.  On the vector unit a thread read 16 bytes of the matrix per
// 4 multiply-adds and env: a step's simulator phase took 4900 cycles for 16 envs of 60 + 8 elements and 10500 for 108 + 21; now
// 2800 and 4700 beside the draws.
// What a lane's part of an item is does not change from step to step: of a wave's first item it is worked out once.
struct SimLane {
  int r, blk, m_off, x_off;      // env of the tile, block of 4 elements (may lie beyond the last), floats into m_r / the state rows
};
__device__ __forceinline__ SimLane sim_lane(const RolloutEnv& a, int item, int OS, int lane) {
  const int nbo = a.o4 >> 2, n_ot = (nbo + 3) >> 2;
  int ot = item, eg = 0;
  while (ot >= n_ot) { ot -= n_ot; ++eg; }
  SimLane s;
  s.blk = 4 * ot + ((lane >> 2) & 3);
  s.r = 16 * eg + 4 * (lane >> 4) + (lane & 3);
  s.m_off = (4 * min(s.blk, nbo - 1) + (lane & 3)) * a.ms;
  s.x_off = min(s.r, a.rows_per_wg - 1) * OS;
  return s;
}
template <class Put>
__device__ __forceinline__ void sim_items(const RolloutEnv& a, int r0, uint32_t step, SimLane sl, const float* s_in, int OS, const float* mr,
                                          float* s_part, const int* s_done, const float4* s_noise, int npr, int nba, int wave, int lane,
                                          Put put) {
  const int O = a.obs_dim, A = a.act_dim, OA = O + A, nbo = a.o4 >> 2;
  const int n_items = ((nbo + 3) >> 2) * (a.rows_per_wg >> 4), ng = OA >> 2, rem = OA & 3;
  for (int item = wave; item < n_items; ) {
    const int blk = sl.blk, r = sl.r, bc = min(blk, nbo - 1);
    const float* mp = mr + sl.m_off;
    const float* xp = s_in + sl.x_off;
    float4 m[4], x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int gu = max(min(u, ng - 1), 0);
      m[u] = *reinterpret_cast<const float4*>(mp + 4 * gu);
      x[u] = *reinterpret_cast<const float4*>(xp + 4 * gu);
    }
    const int done = s_done[r];
    const float4 zn = s_noise[r * npr + nba + bc];        // drawn ahead
    const float4 xs = *reinterpret_cast<const float4*>(xp + 4 * bc);
    const float xa = xp[O + min(blk, A - 1)];
    const int gt = rem ? ng : 0;
    const float4 mt = *reinterpret_cast<const float4*>(mp + 4 * gt), xt = *reinterpret_cast<const float4*>(xp + 4 * gt);
    simx4 acc = {0.f, 0.f, 0.f, 0.f};
    auto step4 = [&](const float4& mv, const float4& xv) {
      acc = __builtin_amdgcn_mfma_f32_4x4x1f32(mv.x, xv.x, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_4x4x1f32(mv.y, xv.y, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_4x4x1f32(mv.z, xv.z, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_4x4x1f32(mv.w, xv.w, acc, 0, 0, 0);
    };
    int g = 0;
    for (; g + 4 < ng; g += 4)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        step4(m[u], x[u]);
        const int gn = min(g + 4 + u, ng - 1);      // past the end: read again, not used (no load behind a branch)
        m[u] = *reinterpret_cast<const float4*>(mp + 4 * gn);
        x[u] = *reinterpret_cast<const float4*>(xp + 4 * gn);
      }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (g + u < ng) step4(m[u], x[u]);
    if (rem) {
      acc = __builtin_amdgcn_mfma_f32_4x4x1f32(mt.x, xt.x, acc, 0, 0, 0);
      if (rem > 1) acc = __builtin_amdgcn_mfma_f32_4x4x1f32(mt.y, xt.y, acc, 0, 0, 0);
      if (rem > 2) acc = __builtin_amdgcn_mfma_f32_4x4x1f32(mt.z, xt.z, acc, 0, 0, 0);
    }
    if (blk < nbo) {
      const float xv[4] = {xs.x, xs.y, xs.z, xs.w}, zv[4] = {zn.x, zn.y, zn.z, zn.w};
      float ps = 0.f, pa = 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (4 * blk + j < O) ps = fmaf(xv[j], xv[j], ps);
      if (blk < A) pa = fmaf(xa, xa, pa);
      for (int q = blk + nbo; q < A; q += nbo) { const float v = xp[O + q]; pa = fmaf(v, v, pa); }
      s_part[r * nbo + blk] = gmi::reward_part(ps, pa);
      float out[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) out[j] = fmaf(a.noise_std, zv[j], acc[j]);
      if (done) {
        float z[4] = {0.f, 0.f, 0.f, 0.f};
        if (r0 + r < a.n) gmi::normal_block(a.e_env_offset + (uint32_t)(r0 + r), step, gmi::kStreamReset, (uint32_t)blk, a.ek0, a.ek1, z);
#pragma unroll
        for (int j = 0; j < 4; ++j) out[j] = z[j];
      }
      put(r, 4 * blk, out);
    }
    item += 8;
    if (item < n_items) sl = sim_lane(a, item, OS, lane);
  }
}

// Words of random block q of env r of the tile: its npr blocks are nba action-noise blocks, the env-noise blocks, then the done draw.
// (Left as kernel arguments the keys are chosen between by address: loads of their own in front of every draw.)
__device__ __forceinline__ gmi::Words4 draw_words(const RolloutEnv& a, uint32_t stp, int r0, int r, bool is_act, bool is_done, uint32_t blk) {
  auto uniform = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); };
  const uint32_t ak0 = uniform(a.ak0), ak1 = uniform(a.ak1), ao = uniform(a.a_env_offset);
  const uint32_t ek0 = uniform(a.ek0), ek1 = uniform(a.ek1), eo = uniform(a.e_env_offset);
  const uint32_t e = (uint32_t)(r0 + r < a.n ? r0 + r : a.n - 1);
  const uint32_t strm = is_act ? gmi::kStreamAction : (is_done ? gmi::kStreamDone : gmi::kStreamEnv);
  return gmi::philox4x32_10((is_act ? ao : eo) + e, stp, strm, blk, is_act ? ak0 : ek0, is_act ? ak1 : ek1);
}
// One random block of a step (the done draw: raw word in .x).
__device__ __forceinline__ void draw_item(const RolloutEnv& a, float4* dst, uint32_t stp, int r0, int npr, int nba, int item) {
  const int r = (int)__umulhi((uint32_t)item, a.npr_magic), q = item - r * npr;
  const bool is_act = q < nba, is_done = q == npr - 1;
  const gmi::Words4 w = draw_words(a, stp, r0, r, is_act, is_done, is_act ? (uint32_t)q : (is_done ? 0u : (uint32_t)(q - nba)));
  float z0, z1, z2, z3;
  gmi::normal_pair(w.w[0], w.w[1], z0, z1);
  gmi::normal_pair(w.w[2], w.w[3], z2, z3);
  dst[item] = is_done ? make_float4(__uint_as_float(w.w[0]), 0.f, 0.f, 0.f) : make_float4(z0, z1, z2, z3);
}
// All random blocks of a step, by all 512 threads.
__device__ __forceinline__ void draw_all(const RolloutEnv& a, float4* dst, uint32_t stp, int r0, int npr, int nba, int tid) {
  for (int item = tid; item < a.rows_per_wg * npr; item += 512) draw_item(a, dst, stp, r0, npr, nba, item);
}
// The same beside the simulator, whose items go to the first waves: last threads first.  (Handed out 64 at a time through a
// counter in LDS, the collection of 17:64:64:6 took 196 us instead of 185.)
__device__ __forceinline__ void draw_rest(const RolloutEnv& a, float4* dst, uint32_t stp, int r0, int npr, int nba, int tid, int top) {
  for (int item = top - tid; item >= 0 && item < a.rows_per_wg * npr; item += 512) draw_item(a, dst, stp, r0, npr, nba, item);
}
// The thread with the first of them: the last one, or the last of the wave before where the waves beside the simulator's are enough
// without the last, which writes the step's sums first.
__device__ __forceinline__ int draw_thread(const RolloutEnv& a, int npr) {
  const int sim = (((a.o4 >> 2) + 3) >> 2) * (a.rows_per_wg >> 4), draws = (a.rows_per_wg * npr + 63) >> 6;
  return sim + draws <= 7 ? 447 : 511;
}

// Thread e < rows_per_wg: env r0 + e's done flag, and its episode counter.
__device__ __forceinline__ void finish_env(const RolloutEnv& a, int r0, int64_t slot0, int e, const float4* s_noise, int npr, uint32_t& ep,
                                           int* s_done) {
  int d = 0;
  if (r0 + e < a.n) {
    if (a.done_period > 0) d = ((ep + 1u) % a.done_period) == 0u;
    else d = __float_as_uint(s_noise[e * npr + npr - 1].x) < a.done_threshold;
    ep = d ? 0u : ep + 1u;
    a.b_done[slot0 + e] = (uint8_t)d;
  }
  s_done[e] = d;
}
// Its log-density and its reward: sums over the blocks, in order.
__device__ __forceinline__ float block_sum(const float* q, int n) {
  float sum = 0.f;
  int j = 0;
  for (; j + 8 <= n; j += 8) {      // eight LDS reads in flight
    float t8[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) t8[u] = q[j + u];
#pragma unroll
    for (int u = 0; u < 8; ++u) sum += t8[u];
  }
  for (; j < n; ++j) sum += q[j];
  return sum;
}

// Whether a model, a simulator and an experience buffer fit together.
int check_rollout(const char* fn, const gmi_model* m, const gmi_env* env, const gmi_buffer* b) {
  const ModelLayout& L = m->L;
  if (env->d.obs_dim != L.obs_dim || env->d.act_dim != L.act_dim || b->d.obs_dim != L.obs_dim || b->d.act_dim != L.act_dim)
    GMI_FAIL(GMI_ERR_BAD_SHAPE, "%s: model, env and buffer disagree on obs_dim / act_dim", fn);
  if (env->d.n_envs != b->d.n_envs)
    GMI_FAIL(GMI_ERR_BAD_SHAPE, "%s: env has %d envs, buffer %d", fn, env->d.n_envs, b->d.n_envs);
  return GMI_OK;
}

// Envs per workgroup and what follows from it.
void set_rows(RolloutEnv* a, int rows) {
  a->rows_per_wg = rows;
  a->row_shift = rows == 16 ? 5 : rows == 32 ? 4 : 3;
  a->n_tiles = (a->n + rows - 1) / rows;
}

// Everything of a RolloutEnv but log_std and the tiling.
void fill_rollout_env(const gmi_model* m, const gmi_env* env, const gmi_buffer* b, float* obs, uint64_t seed, uint32_t step0,
                      uint32_t env_offset, float* last_value, RolloutEnv* a) {
  const gmi_env_desc& ed = env->d;
  const gmi_buffer_desc& bd = b->d;
  a->obs_state = obs;
  a->m_r = env->m_r;
  a->episode_step = env->episode_step;
  a->n = bd.n_envs; a->obs_dim = m->L.obs_dim; a->act_dim = m->L.act_dim; a->o4 = (m->L.obs_dim + 3) & ~3;
  a->ms = gmi::env_row_stride(a->obs_dim, a->act_dim);
  a->T = bd.horizon; a->ld_envs = bd.ld_envs;
  a->obs_vec = (a->obs_dim % 4 == 0 && ((uintptr_t)bd.obs & 15) == 0) ? 1 : 0;
  a->npr_magic = 0xFFFFFFFFu / (uint32_t)((a->act_dim + 3) / 4 + a->o4 / 4 + 1) + 1u;
  a->noise_std = ed.noise_std; a->reward_scale = ed.reward_scale;
  a->done_period = ed.done_period; a->done_threshold = ed.done_threshold;
  a->ak0 = (uint32_t)seed; a->ak1 = (uint32_t)(seed >> 32); a->a_env_offset = env_offset;
  a->ek0 = (uint32_t)ed.seed; a->ek1 = (uint32_t)(ed.seed >> 32); a->e_env_offset = ed.env_offset;
  a->step0 = step0;
  a->b_obs = bd.obs; a->b_act = bd.act; a->b_logp = bd.logp; a->b_val = bd.val; a->b_rew = bd.rew; a->b_done = bd.done;
  a->last_value = last_value;
}

}  // namespace
