// Environment simulator role: the seeded linear-Gaussian stand-in (Section 3 of the paper describes
// the role: receive actions, return new states and rewards for hundreds or thousands of envs).
#include "internal.h"
#include "rng.h"

namespace {

// m_t[k, o] (row stride o4) and m_r[o, k] (row stride ms) = A[o, k] for k < O, B[o, k-O] for O <= k < O+A; zero padded.
__global__ void build_env_matrix(const float* __restrict__ a_mat, const float* __restrict__ b_mat, int O,
                                 int A, int o4, int ms, float* __restrict__ m_t, float* __restrict__ m_r) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= ms * o4) return;
  const int k = idx / o4, o = idx % o4;
  float v = 0.f;
  if (o < O && k < O + A) v = k < O ? a_mat[o * O + k] : b_mat[o * A + (k - O)];
  if (k < O + A) m_t[idx] = v;
  m_r[o * ms + k] = v;
}

// FUSED (gmi::StepFuse, internal.h): what the collection stage of a model too large for the one-launch rollout kernel
// adds to an env step -- the action decision from the policy means that the forward kernel left (the arithmetic of
// sample_kernel: same draws, same operations in the same order), the experience store of the step (copies), and the
// bf16 copy of the next state that the next step's forward kernel reads.
__device__ __forceinline__ uint32_t bf16_pair(float lo, float hi) {      // round to nearest even, as gather_kernel converts
  uint32_t a = __float_as_uint(lo), b = __float_as_uint(hi);
  a += 0x7FFFu + ((a >> 16) & 1u);
  b += 0x7FFFu + ((b >> 16) & 1u);
  return (a >> 16) | (b & 0xFFFF0000u);
}

// State (ACT: and action) of the envs env0 .. env0 + EB - 1 into LDS rows OS floats apart (zeros past the
// last env), eight loads at a time; the state also into copy [N, O] if given.
template <bool ACT>
__device__ __forceinline__ void stage_inputs(const float* __restrict__ obs, const float* __restrict__ act, float* __restrict__ copy,
                                             int env0, int EB, int N, int O, int A, float* dst, int OS, int tid) {
  const int W = ACT ? O + A : O, n = EB * W;
  const int dk = 256 % W, de = 256 / W;
  int e = tid / W, k = tid - e * W;
  for (int i0 = tid; i0 < n; i0 += 8 * 256) {
    float v[8];
    int es = e, ks = k;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int64_t env = min(env0 + e, N - 1);
      if constexpr (ACT) v[u] = *(k < O ? obs + env * O + k : act + env * A + (k - O));
      else v[u] = obs[env * O + k];
      e += de; k += dk;
      if (k >= W) { k -= W; ++e; }
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (es < EB) {
        const bool ok = env0 + es < N;
        dst[es * OS + ks] = ok ? v[u] : 0.f;
        if (copy && ok) copy[(int64_t)(env0 + es) * O + ks] = v[u];
      }
      es += de; ks += dk;
      if (ks >= W) { ks -= W; ++es; }
    }
  }
}

// One workgroup owns EB = G*EPT envs.  Thread (g, b): output block b (4 consecutive next-state
// elements) of envs g*EPT .. g*EPT+EPT-1.  Inputs of the workgroup's envs are staged in LDS once, rows OS floats apart.
// The phases before the product are round trips to memory: loads of a phase are issued together, and every element has a
// thread (one element after the other, the staging of 16 envs of 211 + 20 and their actions cost 33 round trips).
// MF: the product on the 4x4x1 fp32 matrix instruction, whose chain over k is the vector form's sequence of fused multiply-adds, bit for
// bit, in half its cycles and beside the vector unit's work for other waves.  A wave owns 16 of up to 64 output blocks (lane L: block
// L / 4) of all 4 EPT envs, a thread's env i = 4 i + L % 4 of them; a matrix row is one load of 64 consecutive floats per wave.
template <int EPT, bool FUSED, bool MF>
__global__ __launch_bounds__(256) void env_step_kernel(
    const float* __restrict__ obs, const float* __restrict__ act, const float* __restrict__ m_t,
    uint32_t* __restrict__ episode_step, float* __restrict__ next_obs, float* __restrict__ reward,
    uint8_t* __restrict__ done, int N, int O, int A, int OS, int o4, int nb, int G, float noise_std,
    float reward_scale, uint32_t done_period, uint32_t done_threshold, uint32_t k0, uint32_t k1,
    uint32_t env_offset, uint32_t step, int vec_store, gmi::StepFuse fu) {
  extern __shared__ float smem[];
  const int OA = O + A;
  const int EB = G * EPT;
  float* s_in = smem;                          // [EB][OS] state | action
  float* s_part = s_in + EB * OS;              // [EB][nb]
  int* s_done = (int*)(s_part + EB * nb);      // [EB]
  const int env0 = blockIdx.x * EB;
  const int tid = threadIdx.x;

  if constexpr (FUSED) {
    float* s_z = (float*)(s_done + EB);        // [EB][4 * nba] standard-normal draws of the step's actions
    const int nba = (A + 3) / 4;
    stage_inputs<false>(obs, nullptr, fu.b_obs, env0, EB, N, O, A, s_in, OS, tid);
    for (int p = tid; p < EB * nba; p += 256) {
      const int e = p / nba, b = p % nba;
      const int env = env0 + e;
      float z[4] = {0.f, 0.f, 0.f, 0.f};
      if (env < N) gmi::normal_block(fu.a_env_offset + (uint32_t)env, step, gmi::kStreamAction, (uint32_t)b, fu.ak0, fu.ak1, z);
#pragma unroll
      for (int i = 0; i < 4; ++i) s_z[(e * nba + b) * 4 + i] = z[i];
    }
    __syncthreads();
    for (int p = tid; p < EB * A; p += 256) {
      const int e = p / A, j = p - e * A;
      const int env = env0 + e;
      float* zp = s_z + e * nba * 4 + j;
      float a_j = 0.f;
      if (env < N) {
        const float zj = *zp, ls = fu.log_std[j];
        a_j = fmaf(expf(ls), zj, fu.mu[(int64_t)env * A + j]);
        fu.b_act[(int64_t)env * A + j] = a_j;
        *zp = -0.5f * zj * zj - ls - 0.918938533204672742f;
      }
      s_in[e * OS + O + j] = a_j;
    }
    __syncthreads();
    for (int e = tid; e < EB; e += 256) {      // the log-density is summed in action order
      if (env0 + e >= N) continue;
      float lp = 0.f;
      for (int j = 0; j < A; ++j) lp += s_z[e * nba * 4 + j];
      fu.b_logp[env0 + e] = lp;
    }
  } else {
    stage_inputs<true>(obs, act, nullptr, env0, EB, N, O, A, s_in, OS, tid);
  }
  // done flags (integer decisions): periodic counter or Bernoulli by an integer threshold
  for (int el = tid; el < EB; el += 256) {
    const int env = env0 + el;
    int d = 0;
    if (env < N) {
      const uint32_t ep = episode_step[env];
      if (done_period > 0) {
        d = ((ep + 1u) % done_period) == 0u;
      } else {
        const gmi::Words4 w = gmi::philox4x32_10(env_offset + (uint32_t)env, step, gmi::kStreamDone, 0u, k0, k1);
        d = w.w[0] < done_threshold;
      }
      episode_step[env] = d ? 0u : ep + 1u;
      done[env] = (uint8_t)d;
    }
    s_done[el] = d;
  }
  __syncthreads();

  const int b = MF ? tid >> 2 : tid % nb;
  const int e0 = MF ? tid & 3 : tid / nb * EPT;      // the thread's envs: e0 + ES i
  constexpr int ES = MF ? 4 : 1;
  const bool active = MF ? b < nb : tid / nb < G;
  float acc[EPT][4];
#pragma unroll
  for (int i = 0; i < EPT; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;
  const float* xin = s_in + e0 * OS;

  if constexpr (MF) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    f4 c[EPT];
#pragma unroll
    for (int i = 0; i < EPT; ++i) c[i] = f4{0.f, 0.f, 0.f, 0.f};
    const float* mcol = m_t + min(tid, o4 - 1);
    float m[2][4];
    auto fetch = [&](int buf, int k) {
#pragma unroll
      for (int u = 0; u < 4; ++u) m[buf][u] = mcol[min(k + u, OA - 1) * o4];
    };
    auto multiply = [&](int buf, int k) {      // OS is a multiple of 4
      float4 x[EPT];
#pragma unroll
      for (int i = 0; i < EPT; ++i) x[i] = *reinterpret_cast<const float4*>(xin + 4 * i * OS + k);
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < EPT; ++i)
          c[i] = __builtin_amdgcn_mfma_f32_4x4x1f32(m[buf][u], u == 0 ? x[i].x : u == 1 ? x[i].y : u == 2 ? x[i].z : x[i].w, c[i], 0, 0, 0);
    };
    fetch(0, 0);
    int k = 0;
    for (; k + 8 <= OA; k += 8) {
      fetch(1, k + 4);
      multiply(0, k);
      fetch(0, k + 8);
      multiply(1, k + 4);
    }
    if (k + 4 <= OA) {
      multiply(0, k);
      k += 4;
    }
    for (; k < OA; ++k) {
      const float mk = mcol[k * o4];
#pragma unroll
      for (int i = 0; i < EPT; ++i) c[i] = __builtin_amdgcn_mfma_f32_4x4x1f32(mk, xin[4 * i * OS + k], c[i], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < EPT; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = c[i][j];
  }
  if (!MF && active) {
    const float4* mrow = reinterpret_cast<const float4*>(m_t) + b;
    const int stride4 = o4 / 4;
    // four matrix rows are fetched while the four before them are multiplied
    float4 m[2][4];
    auto fetch = [&](int buf, int k) {
#pragma unroll
      for (int u = 0; u < 4; ++u) m[buf][u] = mrow[(int64_t)min(k + u, OA - 1) * stride4];
    };
    auto multiply = [&](int buf, int k) {
      float x[EPT][4];
      if ((OS & 3) == 0) {
#pragma unroll
        for (int i = 0; i < EPT; ++i) {
          const float4 v = *reinterpret_cast<const float4*>(xin + i * OS + k);
          x[i][0] = v.x; x[i][1] = v.y; x[i][2] = v.z; x[i][3] = v.w;
        }
      } else {
#pragma unroll
        for (int i = 0; i < EPT; ++i)
#pragma unroll
          for (int u = 0; u < 4; ++u) x[i][u] = xin[i * OS + k + u];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < EPT; ++i) {
          acc[i][0] = fmaf(x[i][u], m[buf][u].x, acc[i][0]);
          acc[i][1] = fmaf(x[i][u], m[buf][u].y, acc[i][1]);
          acc[i][2] = fmaf(x[i][u], m[buf][u].z, acc[i][2]);
          acc[i][3] = fmaf(x[i][u], m[buf][u].w, acc[i][3]);
        }
    };
    fetch(0, 0);
    int k = 0;
    for (; k + 8 <= OA; k += 8) {
      fetch(1, k + 4);
      multiply(0, k);
      fetch(0, k + 8);
      multiply(1, k + 4);
    }
    if (k + 4 <= OA) {
      multiply(0, k);
      k += 4;
    }
    for (; k < OA; ++k) {
      const float4 mk = mrow[(int64_t)k * stride4];
#pragma unroll
      for (int i = 0; i < EPT; ++i) {
        const float x = xin[i * OS + k];
        acc[i][0] = fmaf(x, mk.x, acc[i][0]);
        acc[i][1] = fmaf(x, mk.y, acc[i][1]);
        acc[i][2] = fmaf(x, mk.z, acc[i][2]);
        acc[i][3] = fmaf(x, mk.w, acc[i][3]);
      }
    }
  }
  if (active) {
    // partial squared norms for the reward: this thread's 4 state elements, and its share of the action
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      float ps = 0.f, pa = 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int o = 4 * b + j;
        if (o < O) { const float x = xin[ES * i * OS + o]; ps = fmaf(x, x, ps); }
      }
      for (int a = b; a < A; a += nb) { const float x = xin[ES * i * OS + O + a]; pa = fmaf(x, x, pa); }
      s_part[(e0 + ES * i) * nb + b] = gmi::reward_part(ps, pa);
    }
  }
  __syncthreads();
  for (int el = tid; el < EB; el += 256) {
    if (env0 + el >= N) break;
    float s = 0.f;
    for (int j = 0; j < nb; ++j) s += s_part[el * nb + j];
    reward[env0 + el] = -reward_scale * s;
  }
  if (!active) return;
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const int e = e0 + ES * i;
    const int env = env0 + e;
    if (env >= N) continue;
    float z[4];
    float outv[4];
    if (s_done[e]) {
      gmi::normal_block(env_offset + (uint32_t)env, step, gmi::kStreamReset, (uint32_t)b, k0, k1, z);
#pragma unroll
      for (int j = 0; j < 4; ++j) outv[j] = z[j];
    } else {
      gmi::normal_block(env_offset + (uint32_t)env, step, gmi::kStreamEnv, (uint32_t)b, k0, k1, z);
#pragma unroll
      for (int j = 0; j < 4; ++j) outv[j] = fmaf(noise_std, z[j], acc[i][j]);
    }
    float* dst = next_obs + (int64_t)env * O + 4 * b;
    if (vec_store) {
      *reinterpret_cast<float4*>(dst) = make_float4(outv[0], outv[1], outv[2], outv[3]);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (4 * b + j < O) dst[j] = outv[j];
    }
    if constexpr (FUSED) {
      if (fu.x16_next) {      // rows of o_pad >= o4 two-byte elements, zero beyond O (as gather_kernel leaves them)
        const uint32_t lo = bf16_pair(4 * b + 0 < O ? outv[0] : 0.f, 4 * b + 1 < O ? outv[1] : 0.f);
        const uint32_t hi = bf16_pair(4 * b + 2 < O ? outv[2] : 0.f, 4 * b + 3 < O ? outv[3] : 0.f);
        *reinterpret_cast<uint2*>(fu.x16_next + (int64_t)env * fu.o_pad + 4 * b) = make_uint2(lo, hi);
      }
    }
  }
}

}  // namespace

extern "C" int gmi_env_bind(gmi_t g, const gmi_env_desc* d, const float* a_mat, const float* b_mat,
                            uint32_t* episode_step, gmi_env_t* out) {
  if (!out) GMI_FAIL(GMI_ERR_INVALID_ARG, "gmi_env_bind: out is NULL");
  *out = nullptr;
  if (!valid(g)) GMI_FAIL(GMI_ERR_BAD_HANDLE, "gmi_env_bind: bad instance");
  if (!d || !a_mat || !b_mat || !episode_step) GMI_FAIL(GMI_ERR_INVALID_ARG, "gmi_env_bind: NULL argument");
  if (d->n_envs < 0 || d->obs_dim < 1 || d->act_dim < 1 || d->obs_dim > 1024 || d->act_dim > 1024)
    GMI_FAIL(GMI_ERR_BAD_SHAPE, "gmi_env_bind: need n_envs >= 0, 1 <= obs_dim, act_dim <= 1024");
  const int O = d->obs_dim, A = d->act_dim;
  const int o4 = (O + 3) & ~3;
  const int ms = gmi::env_row_stride(O, A);
  float* m_t = nullptr;
  GMI_HIP(hipMalloc(&m_t, sizeof(float) * (size_t)(O + A + ms) * o4));
  float* m_r = m_t + (size_t)(O + A) * o4;      // o4 is a multiple of 4: 16-byte aligned
  const int total = ms * o4;
  build_env_matrix<<<(total + 255) / 256, 256, 0, g->stream>>>(a_mat, b_mat, O, A, o4, ms, m_t, m_r);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = hipStreamSynchronize(g->stream);
  if (e != hipSuccess) {
    (void)hipFree(m_t);
    GMI_FAIL(GMI_ERR_HIP, "gmi_env_bind: building the transposed matrix failed: %s", hipGetErrorString(e));
  }
  gmi_env* env = new gmi_env();
  env->magic = gmi::kMagicEnv;
  env->d = *d;
  env->m_t = m_t;
  env->m_r = m_r;
  env->episode_step = episode_step;
  *out = env;
  return GMI_OK;
}

extern "C" int gmi_env_destroy(gmi_env_t env) {
  if (!valid(env)) GMI_FAIL(GMI_ERR_BAD_HANDLE, "gmi_env_destroy: bad handle");
  (void)hipFree(env->m_t);
  env->magic = 0;
  delete env;
  return GMI_OK;
}

namespace gmi {
int launch_env_step(gmi_instance* g, gmi_env* env, const float* obs, const float* act, uint32_t step, float* next_obs,
                    float* reward, uint8_t* done, const StepFuse* fuse) {
  const gmi_env_desc& d = env->d;
  const int N = d.n_envs, O = d.obs_dim, A = d.act_dim;
  const int o4 = (O + 3) & ~3, nb = o4 / 4;
  const int G = 256 / nb;
  // more envs per thread once there is enough work to fill the device several times over
  int ept = 1;
  const int64_t wg1 = ((int64_t)N + G - 1) / G;
  if (wg1 >= 4096) ept = 4; else if (wg1 >= 2048) ept = 2;
  // LDS: [EB][O+A] inputs + [EB][nb] partials + [EB] flags (+ [EB][4 ceil(A/4)] action draws in the fused form)
  const int zw = fuse ? 4 * ((A + 3) / 4) : 0;
  auto lds_bytes = [&](int e) { return (size_t)(G * e) * (O + A + nb + 1 + zw) * sizeof(float); };
  while (ept > 1 && lds_bytes(ept) > 64 * 1024) ept >>= 1;
  if (lds_bytes(ept) > 64 * 1024) GMI_FAIL(GMI_ERR_UNSUPPORTED, "env_step: obs_dim + act_dim too large for the staging buffer");
  const int EB = G * ept;
  int OS = (O + A + 3) & ~3;      // rows of 16-byte pieces where the padding fits
  if (lds_bytes(ept) + (size_t)EB * (OS - O - A) * sizeof(float) > 64 * 1024) OS = O + A;
  const size_t lds = lds_bytes(ept) + (size_t)EB * (OS - O - A) * sizeof(float);
  // Four waves of 16 output blocks are the 4 envs' workgroup of 52 to 64 blocks.  Vector form / matrix instruction, us: 211 + 20, 512 envs
  // 13.8 / 11.2, 4096 32.6 / 19.4, 12288 49.1 / 36.2, 16384 43.3 / 41.5, 65536 149 / 135, 262144 629 / 566; 256 + 32, 4096 38.5 / 22.3,
  // 65536 185 / 165; a step of the collection of 16384 envs of 211 + 20 53.6 / 51.8.  Two or four groups of envs beside fewer blocks lose at large numbers:
  // 108 + 21, 524288 envs 423 / 435, 60 + 8, 1048576 envs 344 / 372.
  const bool mf = G == 4 && (OS & 3) == 0;
  const unsigned grid = (unsigned)((N + EB - 1) / EB);
  const int vec_store = ((O & 3) == 0) && (((uintptr_t)next_obs & 15) == 0);
  const uint32_t k0 = (uint32_t)d.seed, k1 = (uint32_t)(d.seed >> 32);
  const StepFuse fu = fuse ? *fuse : StepFuse{};
  gmi::ProfScope ps(g, gmi::kClsEnvStep);
#define GMI_ENV_LAUNCH(E, F)                                                                       \
  ps.launch(mf ? env_step_kernel<E, F, true> : env_step_kernel<E, F, false>, dim3(grid), dim3(256), lds,  \
      obs, act, env->m_t, env->episode_step, next_obs, reward, done, N, O, A, OS, o4, nb, G,          \
      d.noise_std, d.reward_scale, d.done_period, d.done_threshold, k0, k1, d.env_offset, step, vec_store, fu)
  if (fuse) {
    if (ept == 4) GMI_ENV_LAUNCH(4, true); else if (ept == 2) GMI_ENV_LAUNCH(2, true); else GMI_ENV_LAUNCH(1, true);
  } else {
    if (ept == 4) GMI_ENV_LAUNCH(4, false); else if (ept == 2) GMI_ENV_LAUNCH(2, false); else GMI_ENV_LAUNCH(1, false);
  }
#undef GMI_ENV_LAUNCH
  GMI_LAUNCH_CHECK();
  return GMI_OK;
}
}  // namespace gmi

extern "C" int env_step(gmi_t g, gmi_env_t env, const float* obs, const float* act, uint32_t step,
                        float* next_obs, float* reward, uint8_t* done) {
  if (!valid(g)) GMI_FAIL(GMI_ERR_BAD_HANDLE, "env_step: bad instance");
  if (!valid(env)) GMI_FAIL(GMI_ERR_BAD_HANDLE, "env_step: bad env");
  if (env->d.n_envs == 0) return GMI_OK;
  if (!obs || !act || !next_obs || !reward || !done) GMI_FAIL(GMI_ERR_INVALID_ARG, "env_step: NULL pointer");
  if (obs == next_obs) GMI_FAIL(GMI_ERR_INVALID_ARG, "env_step: next_obs must not alias obs");
  return gmi::launch_env_step(g, env, obs, act, step, next_obs, reward, done, nullptr);
}
