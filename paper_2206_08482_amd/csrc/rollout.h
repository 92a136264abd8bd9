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
  for (int j = 0; j < n; j += 8) {      // eight LDS reads in flight
    float t8[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) t8[u] = q[min(j + u, n - 1)];
#pragma unroll
    for (int u = 0; u < 8; ++u) sum = j + u < n ? sum + t8[u] : sum;
  }
  return sum;
}

// ------------------------------------------------------------------------------------------------
// The collection of 16 envs per workgroup with the roles of a step on waves of their own: 8 waves carry the networks (the wave with a
// tile of the policy's head decides its actions from the products in its registers), 4 the simulator, 4 the draws and sums.  A step has
// an interval per layer and one of the simulator's, each with a barrier at its end.  What the actions do not decide is done beside the
// policy's layers: the state's part of the simulator's product, whose sums stay in registers, the next step's draws, done flags,
// observations on their way to memory, the sums of the step before; behind the head's barrier only the actions' part of the product
// is left.  The value net is an interval behind the policy, its head beside the simulator.
// A step is a chain of dependent latencies, 16 envs being a fraction of what a compute unit could work on; but waves on one SIMD
// take its vector unit (4 cycles an instruction) and its matrix unit (32 a product of 16x16x4) in turn, so what runs beside the
// policy's layers is kept small, spread over the SIMDs (wave % 4), and yields to them.  With every phase on 8 waves in turn a step of
// 8:32:32:2 took 10100 cycles, of 17:64:64:6 11100; now 4900 and 7000, of which the policy's layers 850, 1000 and 1450 and the rest of
// the simulator 850.
constexpr int kNetWaves = 8, kSimWaves = 4, kDrawWaves = 4, kSplitThreads = 64 * (kNetWaves + kSimWaves + kDrawWaves);
// floats of a row of state | action: whole blocks of four actions
__host__ __device__ __forceinline__ int split_stride(int O, int A) { return (O + ((A + 3) & ~3) + 3) & ~3; }

// Where the waves find a tile's arrays in LDS.
struct SplitArrays {
  float* in2;                 // [2][16][OS] state | action, of this and the next step
  float4* noise2;             // [2][16][npr]
  float* lp;                  // [16][nba]
  float* part;                // [16][nbo]
  int* done;                  // [16]
  const float* val;           // [16] values of the step; NULL: not computed here
  const float* ls;            // [act_dim] log_std
};

// A step's draws in two passes with a barrier between them: the random words of every block, then -- a thread per half of a block, in
// place -- their normals (the done draw stays a raw word).  Blocks whole, a wave's 64 take longer than a small net's layer.
// Both: 64 items from i0 on.
__device__ __forceinline__ void draw_word_items(const RolloutEnv& a, float4* dst, uint32_t stp, int r0, int npr, int nba, int i0, int lane) {
  const int item = i0 + lane;
  if (item >= 16 * npr) return;
  const int r = (int)__umulhi((uint32_t)item, a.npr_magic), q = item - r * npr;
  const bool is_act = q < nba, is_done = q == npr - 1;
  const gmi::Words4 w = draw_words(a, stp, r0, r, is_act, is_done, is_act ? (uint32_t)q : (is_done ? 0u : (uint32_t)(q - nba)));
  reinterpret_cast<uint4*>(dst)[item] = make_uint4(w.w[0], w.w[1], w.w[2], w.w[3]);
}
__device__ __forceinline__ void draw_normal_items(const RolloutEnv& a, float4* dst, int npr, int i0, int lane) {
  const int half = i0 + lane, item = half >> 1;
  if (half >= 2 * 16 * npr) return;
  const int r = (int)__umulhi((uint32_t)item, a.npr_magic);
  if (item - r * npr == npr - 1) return;
  const uint2 w = reinterpret_cast<const uint2*>(dst)[half];
  float z0, z1;
  gmi::normal_pair(w.x, w.y, z0, z1);
  reinterpret_cast<float2*>(dst)[half] = make_float2(z0, z1);
}
// The first step's, by all waves; ends with a barrier.
__device__ __forceinline__ void first_draws(const RolloutEnv& a, float4* dst, int r0, int npr, int nba, int wave, int lane) {
#pragma unroll 1
  for (int i = 64 * wave; i < 16 * npr; i += kSplitThreads) draw_word_items(a, dst, a.step0, r0, npr, nba, i, lane);
  __syncthreads();
#pragma unroll 1
  for (int i = 64 * wave; i < 32 * npr; i += kSplitThreads) draw_normal_items(a, dst, npr, i, lane);
  __syncthreads();
}
// Items of a place of `places`, 64 at a time, for draw wave d of kDrawWaves: as few as possible in each.
template <class Draw>
__device__ __forceinline__ void place_items(int place, int places, int n, int d, Draw draw) {
#pragma unroll 1
  for (int u = place + places * d; 64 * u < n; u += places * kDrawWaves) draw(64 * u);
}

// The decision of four actions, block b of env r of the tile, from the policy's means, into the state row.  std: exp(log_std).
__device__ __forceinline__ void decide_actions(float* s_in, int OS, int O, const float4& z, const float4& std, int r, int b, const float (&mu)[4]) {
  float* row = s_in + r * OS + O + 4 * b;
  row[0] = fmaf(std.x, z.x, mu[0]);
  row[1] = fmaf(std.y, z.y, mu[1]);
  row[2] = fmaf(std.z, z.z, mu[2]);
  row[3] = fmaf(std.w, z.w, mu[3]);
}

// The simulator's product over the k groups g0 .. g1 - 1 of four, in order (see sim_items).
__device__ __forceinline__ void sim_groups(simx4& acc, const float* mp, const float* xp, int g0, int g1) {
  if (g0 >= g1) return;
  float4 m[4], x[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int gu = min(g0 + u, g1 - 1);      // past the end: read again, not used (no load behind a branch)
    m[u] = *reinterpret_cast<const float4*>(mp + 4 * gu);
    x[u] = *reinterpret_cast<const float4*>(xp + 4 * gu);
  }
  auto step4 = [&](const float4& mv, const float4& xv) {
    acc = __builtin_amdgcn_mfma_f32_4x4x1f32(mv.x, xv.x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_4x4x1f32(mv.y, xv.y, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_4x4x1f32(mv.z, xv.z, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_4x4x1f32(mv.w, xv.w, acc, 0, 0, 0);
  };
  int g = g0;
#pragma unroll 1
  for (; g + 4 < g1; g += 4)
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      step4(m[u], x[u]);
      const int gn = min(g + 4 + u, g1 - 1);
      m[u] = *reinterpret_cast<const float4*>(mp + 4 * gn);
      x[u] = *reinterpret_cast<const float4*>(xp + 4 * gn);
    }
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (g + u < g1) step4(m[u], x[u]);
}

// A uniform value that is not known to be the one of the step before: what follows from it is worked out where it is used.  (Kept over
// the steps, every condition of a lane takes two scalar registers; 200 of them were spilled and read back one by one.)
__device__ __forceinline__ int fresh(int v) {
  asm volatile("" : "+s"(v));
  return v;
}

// Groups of four k that a simulator wave reads before the actions are there: the two behind the state's part, and the ragged one
// (0 where there is none).  A row has a group behind its whole ones only where O + A is ragged: past the last one that one is read
// again, not used.
struct SimGroups { int g0, g1, gt; };
__host__ __device__ __forceinline__ SimGroups sim_groups_ahead(int O, int A) {
  const int gs = O >> 2, ng = (O + A) >> 2, rem = (O + A) & 3, last = rem ? ng : ng - 1;
  return {gs < last ? gs : last, gs + 1 < last ? gs + 1 : last, rem ? ng : 0};
}

// What a simulator wave has of an item before the actions are there: the state's part of the sums and the other operands.
struct SimItem {
  SimLane sl;
  simx4 acc;
  float4 m0, m1, mt, zn;      // the matrix behind the state's part: two groups of k and the ragged one; the noise
  int done;
};

// All steps of a tile for simulator wave w: an interval per layer and the simulator's own, each with a barrier at its end, and once
// more those after the last step, for the value net.  mr: the simulator's matrix, LDS or global.  put(t, row, first element, 4
// elements): the next state.
template <int NL, class Put>
__device__ __forceinline__ void sim_wave_steps(const RolloutEnv& a, const SplitArrays& s, const float* mr, int r0, int w, int lane, Put put) {
  typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));
  const int OS = split_stride(a.obs_dim, a.act_dim), w_items = ((a.o4 >> 2) + 3) >> 2;
  const int mine = (w_items - w + kSimWaves - 1) / kSimWaves;      // (0 or less: none)
  auto item_lane = [&](int u) { return sim_lane(a, min(w + kSimWaves * u, w_items - 1), OS, lane); };
  SimItem i0, i1;      // (rows of up to 128 elements have no more)
  i0.sl = item_lane(0);
  i1.sl = item_lane(1);
  int64_t slot0 = r0;
#pragma unroll 1
  for (int t = 0; t <= a.T; ++t, slot0 += a.ld_envs) {
    const int O = fresh(a.obs_dim), A = fresh(a.act_dim), OA = O + A, nbo = (O + 3) >> 2, nba = (A + 3) >> 2, npr = nba + nbo + 1;
    const int gs = O >> 2, ng = OA >> 2, rem = OA & 3, left = fresh(a.n - r0);
    const SimGroups ahead = sim_groups_ahead(O, A);
    const float* s_in = s.in2 + (t & 1) * 16 * OS;
    const float4* s_noise = s.noise2 + (t & 1) * 16 * npr;
    const bool step = t < a.T;
    auto observe = [&](const SimLane& sl) {      // the item's part of the observations goes out
      if (sl.blk >= nbo || sl.r >= left) return;
      const float4 x = *reinterpret_cast<const float4*>(s_in + sl.x_off + 4 * sl.blk);
      float* dst = a.b_obs + (slot0 + sl.r) * O + 4 * sl.blk;
      if (4 * sl.blk + 4 <= O) {
        *reinterpret_cast<float4u*>(dst) = float4u{x.x, x.y, x.z, x.w};
      } else {
        dst[0] = x.x;
        if (4 * sl.blk + 1 < O) dst[1] = x.y;
        if (4 * sl.blk + 2 < O) dst[2] = x.z;
      }
    };
    auto operands = [&](SimItem& it) {      // what does not wait for the actions
      const float* mp = mr + it.sl.m_off;
      it.m0 = *reinterpret_cast<const float4*>(mp + 4 * ahead.g0);
      it.m1 = *reinterpret_cast<const float4*>(mp + 4 * ahead.g1);
      it.mt = *reinterpret_cast<const float4*>(mp + 4 * ahead.gt);
      it.zn = s_noise[it.sl.r * npr + nba + min(it.sl.blk, nbo - 1)];
      it.done = s.done[it.sl.r];
    };
    i0.acc = i1.acc = simx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      if (mine > 0) {
        if (step) {      // a share of the state's part per interval
          const int g0 = gs * l / NL, g1 = gs * (l + 1) / NL;
          sim_groups(i0.acc, mr + i0.sl.m_off, s_in + i0.sl.x_off, g0, g1);
          if (mine > 1) sim_groups(i1.acc, mr + i1.sl.m_off, s_in + i1.sl.x_off, g0, g1);
          if (l == NL - 1) {
            operands(i0);
            if (mine > 1) operands(i1);
          }
        }
        if (l == 0 && step) {
          observe(i0.sl);
          if (mine > 1) observe(i1.sl);
#pragma unroll 1
          for (int u = 2; u < mine; ++u) observe(item_lane(u));
        }
      }
      __syncthreads();
    }
    if (step && mine > 0) {
      __builtin_amdgcn_s_setprio(3);
      int dones = 0;
      auto finish = [&](SimItem& it) {
        const float* xp = s_in + it.sl.x_off;
        const float4 x0 = *reinterpret_cast<const float4*>(xp + 4 * ahead.g0), x1 = *reinterpret_cast<const float4*>(xp + 4 * ahead.g1);
        const float4 xt = *reinterpret_cast<const float4*>(xp + 4 * ahead.gt);
        auto step4 = [&](const float4& mv, const float4& xv) {
          it.acc = __builtin_amdgcn_mfma_f32_4x4x1f32(mv.x, xv.x, it.acc, 0, 0, 0);
          it.acc = __builtin_amdgcn_mfma_f32_4x4x1f32(mv.y, xv.y, it.acc, 0, 0, 0);
          it.acc = __builtin_amdgcn_mfma_f32_4x4x1f32(mv.z, xv.z, it.acc, 0, 0, 0);
          it.acc = __builtin_amdgcn_mfma_f32_4x4x1f32(mv.w, xv.w, it.acc, 0, 0, 0);
        };
        if (gs < ng) step4(it.m0, x0);
        if (gs + 1 < ng) step4(it.m1, x1);
        if (gs + 2 < ng) sim_groups(it.acc, mr + it.sl.m_off, xp, gs + 2, ng);
        if (rem) {
          it.acc = __builtin_amdgcn_mfma_f32_4x4x1f32(it.mt.x, xt.x, it.acc, 0, 0, 0);
          if (rem > 1) it.acc = __builtin_amdgcn_mfma_f32_4x4x1f32(it.mt.y, xt.y, it.acc, 0, 0, 0);
          if (rem > 2) it.acc = __builtin_amdgcn_mfma_f32_4x4x1f32(it.mt.z, xt.z, it.acc, 0, 0, 0);
        }
        dones |= it.done;
        const float out[4] = {fmaf(a.noise_std, it.zn.x, it.acc[0]), fmaf(a.noise_std, it.zn.y, it.acc[1]),
                              fmaf(a.noise_std, it.zn.z, it.acc[2]), fmaf(a.noise_std, it.zn.w, it.acc[3])};
        if (it.sl.blk < nbo) put(t, it.sl.r, 4 * it.sl.blk, out);
      };
      finish(i0);
      if (mine > 1) finish(i1);
#pragma unroll 1
      for (int u = 2; u < mine; ++u) {
        SimItem it;
        it.sl = item_lane(u);
        it.acc = simx4{0.f, 0.f, 0.f, 0.f};
        operands(it);
        sim_groups(it.acc, mr + it.sl.m_off, s_in + it.sl.x_off, 0, gs);
        finish(it);
      }
      if (__ballot(dones != 0))      // a fresh state for the envs that ended
#pragma unroll 1
        for (int u = 0; u < mine; ++u) {
          const SimLane sl = u == 0 ? i0.sl : u == 1 ? i1.sl : item_lane(u);
          if (sl.blk >= nbo || !s.done[sl.r]) continue;
          float z[4] = {0.f, 0.f, 0.f, 0.f};
          if (r0 + sl.r < a.n)
            gmi::normal_block(a.e_env_offset + (uint32_t)(r0 + sl.r), a.step0 + (uint32_t)t, gmi::kStreamReset, (uint32_t)sl.blk, a.ek0, a.ek1, z);
          put(t, sl.r, 4 * sl.blk, z);
        }
      __builtin_amdgcn_s_setprio(0);
    }
    __syncthreads();
  }
}

// The same for draw wave m; waves 0 and 1 have the sums.  Lane e of wave 0 carries env e's episode counter.
template <int NL>
__device__ __forceinline__ void draw_wave_steps(const RolloutEnv& a, const SplitArrays& s, int r0, int m, int lane, uint32_t& ep) {
  const int OS = split_stride(a.obs_dim, a.act_dim);
  const uint32_t a_magic = 0xFFFFFFFFu / (uint32_t)a.act_dim + 1u;      // (A = 1: 0, see below)
  int64_t slot0 = r0;
#pragma unroll 1
  for (int t = 0; t <= a.T; ++t, slot0 += a.ld_envs) {
    const int O = fresh(a.obs_dim), A = fresh(a.act_dim), nbo = (O + 3) >> 2, nba = (A + 3) >> 2, npr = nba + nbo + 1;
    const int left = fresh(a.n - r0), n_act = min(16, left) * A, d = kDrawWaves - 1 - m;
    const bool env = lane < 16, env_ok = lane < min(16, left);
    const float* s_in = s.in2 + (t & 1) * 16 * OS;
    const float* s_prev = s.in2 + (~t & 1) * 16 * OS;
    float4* s_noise = s.noise2 + (t & 1) * 16 * npr;
    float4* next = s.noise2 + (~t & 1) * 16 * npr;
    const bool step = t < a.T;
#pragma unroll
    for (int l = 0; l <= NL; ++l) {      // l = NL: the simulator's
      // the next step's words, then their normals
      if (l < NL && t + 1 < a.T) {
        if (l == 0) place_items(0, 1, 16 * npr, d, [&](int i) { draw_word_items(a, next, a.step0 + (uint32_t)t + 1u, r0, npr, nba, i, lane); });
        else place_items(l - 1, NL - 1, 32 * npr, d, [&](int i) { draw_normal_items(a, next, npr, i, lane); });
      }
      if (l == NL - 2 && t > 0)      // the parts of the last step's rewards
#pragma unroll 1
        for (int i = 64 * m + lane; i < 16 * nbo; i += 64 * kDrawWaves) {
          const int r = i & 15, blk = i >> 4;
          const float* xp = s_prev + r * OS;
          const float4 y = *reinterpret_cast<const float4*>(xp + 4 * blk);
          const float v0 = xp[O + min(blk, A - 1)], v1 = xp[O + min(blk + nbo, A - 1)];
          float ps = y.x * y.x;
          ps = 4 * blk + 1 < O ? fmaf(y.y, y.y, ps) : ps;
          ps = 4 * blk + 2 < O ? fmaf(y.z, y.z, ps) : ps;
          ps = 4 * blk + 3 < O ? fmaf(y.w, y.w, ps) : ps;
          float pa = blk < A ? v0 * v0 : 0.f;
          pa = blk + nbo < A ? fmaf(v1, v1, pa) : pa;
          if (A > 2 * nbo)
#pragma unroll 1
            for (int q = blk + 2 * nbo; q < A; q += nbo) { const float v = xp[O + q]; pa = fmaf(v, v, pa); }
          s.part[r * nbo + blk] = gmi::reward_part(ps, pa);
        }
      if (m == 0) {
        if (l == 0) {
          if (step && env) finish_env(a, r0, slot0, lane, s_noise, npr, ep, s.done);
          if (s.val && t > 0 && env_ok) a.b_val[slot0 - a.ld_envs + lane] = s.val[lane];
        } else if (l == NL - 1) {
          if (t > 0 && env_ok) a.b_rew[slot0 - a.ld_envs + lane] = -a.reward_scale * block_sum(s.part + lane * nbo, nbo);
        }
      } else if (m == 1 && step) {
        if (l == 0) {      // the step's log-densities per block of four actions, its terms in index order
#pragma unroll 1
          for (int i = lane; i < 16 * nba; i += 64) {
            const int r = i & 15, b = i >> 4;
            const float4 z4 = s_noise[r * npr + b];
            const float z[4] = {z4.x, z4.y, z4.z, z4.w};
            float lp = 0.f;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              const float ls = s.ls[min(4 * b + j, A - 1)], term = -0.5f * z[j] * z[j] - ls - 0.918938533204672742f;
              lp = j == 0 ? term : lp + (4 * b + j < A ? term : 0.f);
            }
            s.lp[r * nba + b] = lp;
          }
        } else if (l == NL) {
          if (env_ok) a.b_logp[slot0 + lane] = block_sum(s.lp + lane * nba, nba);
        }
      }
      if (l == NL && step)      // the actions
#pragma unroll 1
        for (int i = 64 * m + lane; i < n_act; i += 64 * kDrawWaves) {
          const int r = A == 1 ? i : (int)__umulhi((uint32_t)i, a_magic);
          a.b_act[slot0 * A + i] = s_in[r * OS + O + i - r * A];
        }
      __syncthreads();
    }
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
