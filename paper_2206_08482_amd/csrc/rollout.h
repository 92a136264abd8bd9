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
  const float* m_t;                 // [(O + A), o4] transposed env matrices
  uint32_t* episode_step;           // [n]
  int n, obs_dim, act_dim, o4, T, ld_envs;
  int rows_per_wg;                  // envs owned by a workgroup: the tile height, or half of it
  int n_tiles;                      // ceil(n / rows_per_wg); the grid may be smaller (workgroups loop)
  float noise_std, reward_scale;
  uint32_t done_period, done_threshold;
  uint32_t ak0, ak1, a_env_offset;  // agent's Philox key and env offset
  uint32_t ek0, ek1, e_env_offset;  // simulator's
  uint32_t step0;
  float* b_obs; float* b_act; float* b_logp; float* b_val; float* b_rew; uint8_t* b_done;
  float* last_value;
};

// Envs per simulator item, and the threads that get an item.  An item reads 16 bytes of the matrix and 4 bytes per env for
// its 4 EPT products of a k, so the LDS bounds many items of one env: 16 envs of 108 + 21 elements (432 items) take 18.0 us
// a step with one, 15.7 with two and the next draws beside them.  Up to one wave per SIMD the chain of a wave's own reads
// is the bound and items of one env are the faster ones (16 envs of 60 + 8: 7.4 against 8.5 us a step).
__host__ __device__ __forceinline__ int sim_ept(int R, int nbo) { return (R / 4) * nbo >= 192 ? 4 : R * nbo > 256 ? 2 : 1; }
__host__ __device__ __forceinline__ int sim_threads(int R, int nbo) { return ((R / sim_ept(R, nbo)) * nbo + 63) & ~63; }

// Simulator step for the tile: items (group of EPT envs, block of 4 state elements).  mt points at the
// transposed matrices (LDS copy or global), row stride nbo float4; ld: floats between the rows of s_in, VEC: a multiple of 4.
template <int EPT, bool VEC>
__device__ __forceinline__ void sim_items(const RolloutEnv& a, int R, int r0, uint32_t step, const float* s_in, int ld,
                                          const float4* mt, float* s_part, float* s_next, const int* s_done,
                                          const float4* s_noise, int npr, int nba) {
  const int O = a.obs_dim, A = a.act_dim, OA = O + A, o4 = a.o4, nbo = o4 >> 2;
  for (int item = threadIdx.x; item < (R / EPT) * nbo; item += blockDim.x) {
    const int g = item / nbo, b = item - g * nbo;
    const float* xin = s_in + (g * EPT) * ld;
    const float4* mrow = mt + b;
    float acc[EPT][4];
#pragma unroll
    for (int i = 0; i < EPT; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;
    // eight matrix rows (and state elements) are fetched before the first of their products: left to the
    // compiler under this kernel's register pressure, every k waited a full LDS round trip for its row
    int k = 0;
    for (; k + 8 <= OA; k += 8) {
      float4 m[8];
      float xv[EPT][8];
#pragma unroll
      for (int u = 0; u < 8; ++u) m[u] = mrow[(k + u) * nbo];
      if constexpr (VEC) {
#pragma unroll
        for (int i = 0; i < EPT; ++i)
#pragma unroll
          for (int u = 0; u < 8; u += 4) {
            const float4 v = *reinterpret_cast<const float4*>(xin + i * ld + k + u);
            xv[i][u] = v.x; xv[i][u + 1] = v.y; xv[i][u + 2] = v.z; xv[i][u + 3] = v.w;
          }
      } else {
#pragma unroll
        for (int i = 0; i < EPT; ++i)
#pragma unroll
          for (int u = 0; u < 8; ++u) xv[i][u] = xin[i * ld + k + u];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int i = 0; i < EPT; ++i) {
          acc[i][0] = fmaf(xv[i][u], m[u].x, acc[i][0]);
          acc[i][1] = fmaf(xv[i][u], m[u].y, acc[i][1]);
          acc[i][2] = fmaf(xv[i][u], m[u].z, acc[i][2]);
          acc[i][3] = fmaf(xv[i][u], m[u].w, acc[i][3]);
        }
    }
    for (; k < OA; ++k) {
      const float4 m = mrow[k * nbo];
#pragma unroll
      for (int i = 0; i < EPT; ++i) {
        const float x = xin[i * ld + k];
        acc[i][0] = fmaf(x, m.x, acc[i][0]);
        acc[i][1] = fmaf(x, m.y, acc[i][1]);
        acc[i][2] = fmaf(x, m.z, acc[i][2]);
        acc[i][3] = fmaf(x, m.w, acc[i][3]);
      }
    }
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      const int r = g * EPT + i;
      float ps = 0.f, pa = 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int o = 4 * b + j;
        if (o < O) { const float x = xin[i * ld + o]; ps = fmaf(x, x, ps); }
      }
      for (int q = b; q < A; q += nbo) { const float x = xin[i * ld + O + q]; pa = fmaf(x, x, pa); }
      s_part[r * nbo + b] = ps + 0.01f * pa;
      const int e = r0 + r;
      float z[4] = {0.f, 0.f, 0.f, 0.f};
      float outv[4];
      if (s_done[r]) {
        if (e < a.n) gmi::normal_block(a.e_env_offset + (uint32_t)e, step, gmi::kStreamReset, (uint32_t)b, a.ek0, a.ek1, z);
#pragma unroll
        for (int j = 0; j < 4; ++j) outv[j] = z[j];
      } else {
        const float4 zn = s_noise[r * npr + nba + b];       // drawn at the top of the step
        z[0] = zn.x; z[1] = zn.y; z[2] = zn.z; z[3] = zn.w;
#pragma unroll
        for (int j = 0; j < 4; ++j) outv[j] = fmaf(a.noise_std, z[j], acc[i][j]);
      }
      *reinterpret_cast<float4*>(&s_next[r * o4 + 4 * b]) = make_float4(outv[0], outv[1], outv[2], outv[3]);
    }
  }
}

template <bool VEC, typename... Args>
__device__ __forceinline__ void sim_step(int R, int nbo, const RolloutEnv& a, Args... args) {
  const int ept = sim_ept(R, nbo);
  if (ept == 4) sim_items<4, VEC>(a, R, args...);
  else if (ept == 2) sim_items<2, VEC>(a, R, args...);
  else sim_items<1, VEC>(a, R, args...);
}

// Random blocks first, first + stride, ... of one step of a tile, one float4 per (env, block): nba action-noise
// blocks, nbo env-noise blocks, then the done draw (raw word in .x).
__device__ __forceinline__ void draw_items(const RolloutEnv& a, float4* dst, uint32_t stp, int Rv, int r0, int npr, int nba,
                                           int nbo, int first, int stride) {
  for (int item = first; item < Rv * npr; item += stride) {
    const int r = item / npr, q = item - r * npr;
    const uint32_t e = (uint32_t)(r0 + r < a.n ? r0 + r : a.n - 1);
    const bool is_act = q < nba, is_env = q >= nba && q < nba + nbo;
    const uint32_t strm = is_act ? gmi::kStreamAction : (is_env ? gmi::kStreamEnv : gmi::kStreamDone);
    const uint32_t blk = is_act ? (uint32_t)q : (is_env ? (uint32_t)(q - nba) : 0u);
    const gmi::Words4 w = gmi::philox4x32_10((is_act ? a.a_env_offset : a.e_env_offset) + e, stp, strm, blk,
                                             is_act ? a.ak0 : a.ek0, is_act ? a.ak1 : a.ek1);
    float z0, z1, z2, z3;
    gmi::normal_pair(w.w[0], w.w[1], z0, z1);
    gmi::normal_pair(w.w[2], w.w[3], z2, z3);
    dst[item] = (is_act || is_env) ? make_float4(z0, z1, z2, z3) : make_float4(__uint_as_float(w.w[0]), 0.f, 0.f, 0.f);
  }
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

// Everything of a RolloutEnv but log_std and the tiling.
void fill_rollout_env(const gmi_model* m, const gmi_env* env, const gmi_buffer* b, float* obs, uint64_t seed, uint32_t step0,
                      uint32_t env_offset, float* last_value, RolloutEnv* a) {
  const gmi_env_desc& ed = env->d;
  const gmi_buffer_desc& bd = b->d;
  a->obs_state = obs;
  a->m_t = env->m_t;
  a->episode_step = env->episode_step;
  a->n = bd.n_envs; a->obs_dim = m->L.obs_dim; a->act_dim = m->L.act_dim; a->o4 = (m->L.obs_dim + 3) & ~3;
  a->T = bd.horizon; a->ld_envs = bd.ld_envs;
  a->noise_std = ed.noise_std; a->reward_scale = ed.reward_scale;
  a->done_period = ed.done_period; a->done_threshold = ed.done_threshold;
  a->ak0 = (uint32_t)seed; a->ak1 = (uint32_t)(seed >> 32); a->a_env_offset = env_offset;
  a->ek0 = (uint32_t)ed.seed; a->ek1 = (uint32_t)(ed.seed >> 32); a->e_env_offset = ed.env_offset;
  a->step0 = step0;
  a->b_obs = bd.obs; a->b_act = bd.act; a->b_logp = bd.logp; a->b_val = bd.val; a->b_rew = bd.rew; a->b_done = bd.done;
  a->last_value = last_value;
}

}  // namespace
