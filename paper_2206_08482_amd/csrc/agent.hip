// The agent's action decision in one launch (Section 3 of the paper, "DRL Agent"), bf16 models: observation conversion,
// every layer of one net, and the Gaussian sampling epilogue.
//
// A workgroup of 8 waves owns R = 32 RT rows of ONE net (grid: row tiles x nets).  The two nets meet nowhere: action and
// log-density need the policy net, the value needs the value net.  Activations are row-major [row][feature] in LDS (rows
// of K + 8 elements: an odd number of 16-byte pieces, so that operand reads of consecutive rows hit different banks); layer
// l reads buffer l % 2 and writes the other one.  Products are computed transposed (32x32x16 matrix instruction, weights
// first operand from the fragment-major copy in L2, activations second).  An item is one 32-feature tile for one or two
// row tiles; items are dealt to the waves, and a wave requests the first kDepth weight blocks of its next item, also
// across a layer's barrier, before it leaves the present one.  The random draws are made while the observations and the
// first weights are on their way.
//
// Bound, few rows: the chain of latencies launch - observations - one weight round trip per kDepth k steps - heads -
// sampling.  Many rows: epilogue arithmetic and LDS operand reads.
//
// Sums run over k in ascending order from zero and the bias is added last: the results are those of rollout_collect
// (fused.hip, or this kernel and env.hip), bit for bit.
#include <algorithm>

#include "chain_kernel.h"
#include "rng.h"

namespace {
using namespace gmi_chain;

constexpr int kNT = 512, kNW = 8;
constexpr int kDepth = 8;                   // weight blocks (1 KiB) in flight per wave
constexpr int kMaxLayers = GMI_MAX_HIDDEN + 1;
constexpr size_t kLdsMax = 160 * 1024;

struct AgentLayer {
  const uint4* w;          // fragment-major W
  const float* bias;
  int K, F;                // padded widths
};
struct AgentArgs {
  AgentLayer l[2][kMaxLayers];
  int nl, net0;            // blockIdx.y = 0 is net net0
  int n, O, A;
  int y_off, f_off;        // LDS: second activation buffer (elements), float area (bytes)
  int vec_obs;             // the observations are 16-byte aligned
  int lp_blocks;           // log-density: 1 = blocks of 4 actions summed first, 0 = one action after the other
  uint32_t o_magic, k0, k1, step, env_offset;
  const float *log_std, *obs;
  float *act, *logp, *value, *mu_out;
};

__host__ __device__ __forceinline__ uint32_t magic(uint32_t d) { return d == 1 ? 0u : 0xFFFFFFFFu / d + 1u; }
__device__ __forceinline__ int div_magic(int n, uint32_t m) { return m ? (int)__umulhi((uint32_t)n, m) : n; }      // n * d < 2^32

// acc[i] += W tile x row tiles at xp, xp + xts; wq holds the first kDepth k steps' weight blocks of this lane.
template <int NRT>
__device__ __forceinline__ void k_loop(floatx16 (&acc)[NRT], uint4 (&wq)[kDepth], const uint4* wp, int nks, const uint16_t* xp, int xts) {
  uint4 x[2][NRT];
#pragma unroll
  for (int i = 0; i < NRT; ++i) x[0][i] = *reinterpret_cast<const uint4*>(xp + i * xts);
  auto step = [&](int ks, int u) {
    const int kn = min(ks + 1, nks - 1);
#pragma unroll
    for (int i = 0; i < NRT; ++i) x[(u + 1) & 1][i] = *reinterpret_cast<const uint4*>(xp + i * xts + 16 * kn);
#pragma unroll
    for (int i = 0; i < NRT; ++i)
      acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wq[u]), __builtin_bit_cast(bf16x8, x[u & 1][i]),
                                                       acc[i], 0, 0, 0);
  };
  int ks = 0;
  for (; ks + kDepth < nks; ks += kDepth)
#pragma unroll
    for (int u = 0; u < kDepth; ++u) {
      step(ks + u, u);
      wq[u] = wp[min(ks + u + kDepth, nks - 1) * 64];
    }
#pragma unroll
  for (int u = 0; u < kDepth; u += 2)      // nks is even
    if (ks + u < nks) {
      step(ks + u, u);
      step(ks + u + 1, u + 1);
    }
}

template <int RT>
__global__ __launch_bounds__(kNT, 4) void agent_kernel(AgentArgs a) {
  constexpr int R = 32 * RT;
  constexpr int PR = RT >= 2 ? 2 : 1;               // row tiles of a paired item
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  uint16_t* s_x = reinterpret_cast<uint16_t*>(smem_raw);
  const int net = a.net0 + blockIdx.y;
  const AgentLayer* N = a.l[net];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int s = lane & 31, h = lane >> 5;
  const int nl = a.nl, O = a.O, K0 = N[0].K, S0 = K0 + 8;
  const int ho = net == 0 ? a.A : 1, nb = (a.A + 3) >> 2;      // head outputs; blocks of 4 actions
  float4* s_noise = reinterpret_cast<float4*>(smem_raw + a.f_off);             // [R][nb]
  float* s_head = reinterpret_cast<float*>(s_noise + R * nb);                  // [R][ho]
  const int r0 = blockIdx.x * R, rows = min(R, a.n - r0);

  auto paired = [&](int nft) { return RT >= 2 && nft * (RT / 2) >= kNW; };
  uint4 wq[kDepth];
  auto request = [&](const AgentLayer& L, int item) {
    const int nft = L.F >> 5, nks = L.K >> 4, nrg = paired(nft) ? RT / PR : RT;
    const int ft = min(item / nrg, nft - 1);
    const uint4* wp = L.w + (int64_t)ft * nks * 64 + lane;
#pragma unroll
    for (int u = 0; u < kDepth; ++u) wq[u] = wp[min(u, nks - 1) * 64];
  };

  // the tile's observations are rows * O consecutive floats; 16-byte pieces of them may span two rows
  {
    const float* src = a.obs + (int64_t)r0 * O;
    const int cnt = rows * O, n4 = a.vec_obs ? cnt >> 2 : 0;
    for (int e0 = tid; e0 < n4; e0 += 4 * kNT) {
      float4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = reinterpret_cast<const float4*>(src)[min(e0 + u * kNT, n4 - 1)];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int e = 4 * min(e0 + u * kNT, n4 - 1);
        int r = div_magic(e, a.o_magic), c = e - r * O;
        const uint32_t w0 = pack_bf16(v[u].x, v[u].y), w1 = pack_bf16(v[u].z, v[u].w);
        if ((O & 3) == 0) {
          *reinterpret_cast<uint2*>(s_x + r * S0 + c) = make_uint2(w0, w1);
        } else {
          const uint16_t q[4] = {(uint16_t)w0, (uint16_t)(w0 >> 16), (uint16_t)w1, (uint16_t)(w1 >> 16)};
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            s_x[r * S0 + c] = q[i];
            if (++c == O) { c = 0; ++r; }
          }
        }
      }
    }
    for (int e = 4 * n4 + tid; e < cnt; e += kNT) {
      const int r = div_magic(e, a.o_magic);
      s_x[r * S0 + e - r * O] = (uint16_t)pack_bf16(src[e], 0.f);
    }
    // padding columns, and rows past the end (never stored: any finite value will do)
    const int np = K0 - O;
    for (int e = tid; e < 32 * R; e += kNT)
      if ((e & 31) < np) s_x[(e >> 5) * S0 + O + (e & 31)] = 0;
    for (int e = rows * S0 + tid; e < R * S0; e += kNT) s_x[e] = 0;
  }
  request(N[0], wave);
  if (net == 0 && a.act)
    for (int item = tid; item < rows * nb; item += kNT) {
      const int r = item / nb, b = item - r * nb;
      float z[4];
      gmi::normal_block(a.env_offset + (uint32_t)(r0 + r), a.step, gmi::kStreamAction, (uint32_t)b, a.k0, a.k1, z);
      s_noise[item] = make_float4(z[0], z[1], z[2], z[3]);
    }
  __syncthreads();

  for (int l = 0; l < nl; ++l) {
    const AgentLayer& L = N[l];
    const AgentLayer& Ln = N[min(l + 1, nl - 1)];
    const int nft = L.F >> 5, nks = L.K >> 4, sx = L.K + 8, sy = L.F + 8;
    const uint16_t* x = s_x + (l & 1 ? a.y_off : 0);
    uint16_t* y = s_x + (l & 1 ? 0 : a.y_off);
    const bool head = l == nl - 1;
    auto items = [&](auto nrt) {
      constexpr int NRT = decltype(nrt)::value;
      constexpr int nrg = RT / NRT;
      const int n_items = nft * nrg;
      for (int item = wave; item < n_items; item += kNW) {
        const int ft = item / nrg, rg = item % nrg;
        float4 b4[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) b4[q] = *reinterpret_cast<const float4*>(L.bias + 32 * ft + 8 * q + 4 * h);
        floatx16 acc[NRT];
#pragma unroll
        for (int i = 0; i < NRT; ++i)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
        k_loop<NRT>(acc, wq, L.w + (int64_t)ft * nks * 64 + lane, nks, x + (rg * NRT * 32 + s) * sx + 8 * h, 32 * sx);
        if (item + kNW < n_items) request(L, item + kNW); else request(Ln, wave);
        // lane (s, h) holds, per quad q, the features 32 ft + 8 q + 4 h + 0..3 of row s
#pragma unroll
        for (int i = 0; i < NRT; ++i) {
          const int r = (rg * NRT + i) * 32 + s;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int f = 32 * ft + 8 * q + 4 * h;
            const float v0 = acc[i][4 * q] + b4[q].x, v1 = acc[i][4 * q + 1] + b4[q].y;
            const float v2 = acc[i][4 * q + 2] + b4[q].z, v3 = acc[i][4 * q + 3] + b4[q].w;
            if (!head) {
              *reinterpret_cast<uint2*>(y + r * sy + f) = make_uint2(pack_bf16(elu_f(v0), elu_f(v1)), pack_bf16(elu_f(v2), elu_f(v3)));
            } else {
              float* d = s_head + r * ho + f;
              if (f + 0 < ho) d[0] = v0;
              if (f + 1 < ho) d[1] = v1;
              if (f + 2 < ho) d[2] = v2;
              if (f + 3 < ho) d[3] = v3;
            }
          }
        }
      }
      if (wave >= n_items) request(Ln, wave);
    };
    if (paired(nft)) items(std::integral_constant<int, PR>{}); else items(std::integral_constant<int, 1>{});
    __syncthreads();
  }

  if (net == 1) {
    for (int r = tid; r < rows; r += kNT) a.value[r0 + r] = s_head[r];
    return;
  }
  if (!a.act) {      // the means alone
    for (int e = tid; e < rows * a.A; e += kNT) a.mu_out[(int64_t)r0 * a.A + e] = s_head[e];
    return;
  }
  // act = mu + exp(log_std) * eps, one thread per element, which leaves its log-density term in place of its draw
  const int A = a.A;
  for (int item = tid; item < rows * nb * 4; item += kNT) {
    const int blk = item >> 2, r = blk / nb, j = 4 * (blk - r * nb) + (item & 3);
    float* zp = reinterpret_cast<float*>(s_noise) + item;
    float term = 0.f;
    if (j < A) {
      const float z = *zp, ls = a.log_std[j], m = s_head[r * A + j];
      const int64_t o = (int64_t)(r0 + r) * A + j;
      a.act[o] = fmaf(expf(ls), z, m);
      if (a.mu_out) a.mu_out[o] = m;
      term = -0.5f * z * z - ls - 0.918938533204672742f;
    }
    *zp = term;
  }
  __syncthreads();
  for (int r = tid; r < rows; r += kNT) {
    float lp = 0.f;
    for (int b = 0; b < nb; ++b) {
      const float4 t = s_noise[r * nb + b];
      lp = a.lp_blocks ? lp + (((t.x + t.y) + t.z) + t.w) : (((lp + t.x) + t.y) + t.z) + t.w;
    }
    a.logp[r0 + r] = lp;
  }
}

// LDS of a tile of R rows; the larger net head (the policy's) decides.
size_t agent_lds(const ModelLayout& L, int R, int* y_off, int* f_off) {
  int w[2] = {0, 0};
  for (int l = 0; l < L.n_layers; ++l) w[l & 1] = std::max(w[l & 1], L.net[0][l].in_pad + 8);
  const int nb = (L.act_dim + 3) / 4;
  *y_off = R * w[0];
  *f_off = R * (w[0] + w[1]) * 2;
  return (size_t)*f_off + (size_t)R * (nb * 16 + L.act_dim * 4);
}

template <int RT>
int launch(gmi_instance* g, const AgentArgs& a, int nets, size_t lds) {
  static bool attr = false;
  if (!attr) {
    GMI_HIP(hipFuncSetAttribute((const void*)agent_kernel<RT>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsMax));
    attr = true;
  }
  gmi::ProfScope ps(g, gmi::kClsFusedAgent);
  ps.launch(agent_kernel<RT>, dim3((a.n + 32 * RT - 1) / (32 * RT), nets), dim3(kNT), lds, a);
  GMI_LAUNCH_CHECK();
  return GMI_OK;
}

}  // namespace

namespace gmi {

// act NULL: the policy's means (mu_out) and the values only.  Returns GMI_ERR_UNSUPPORTED (no error message) where the per-layer
// path or the row-tile kernel has to be used instead.
int launch_agent(gmi_instance* g, gmi_model* m, const float* obs, int n, uint64_t seed, uint32_t step, uint32_t env_offset,
                 float* act, float* logp, float* value, float* mu_out, bool do_policy) {
  const ModelLayout& L = m->L;
  if (L.dtype != GMI_DTYPE_BF16) return GMI_ERR_UNSUPPORTED;
  if (use_tile_forward(m, n)) return GMI_ERR_UNSUPPORTED;
  AgentArgs a;
  // 32-row tiles while all workgroups are resident at once (two per compute unit: 5000 rows of 108:400:200:100:21 take 16 us
  // against 18 with 64 rows); beyond, 64-row tiles where two of them fit a compute unit's LDS (262144 rows of
  // 60:256:128:64:8: 183 / 287 us; 20000 of 108:400:200:100:21, where one fits: 47 / 40) or where the weights are so many
  // that fetching them half as often counts (65536 rows of 200:512:512:300:20: 228 / 258 us, 20000: 88 / 85)
  const int nets = do_policy ? 2 : 1;
  const int64_t groups32 = (int64_t)((n + 31) / 32) * nets, slots = 2 * (int64_t)g->cu_count;
  int R = 64;
  size_t lds = agent_lds(L, R, &a.y_off, &a.f_off);
  if (lds > kLdsMax || groups32 <= slots || (2 * lds > kLdsMax && (L.weight_bytes <= (1 << 20) || groups32 < 8 * slots))) {
    R = 32;
    lds = agent_lds(L, R, &a.y_off, &a.f_off);
    if (lds > kLdsMax) return GMI_ERR_UNSUPPORTED;
  }
  for (int net = 0; net < 2; ++net)
    for (int l = 0; l < L.n_layers; ++l) {
      const LayerInfo& li = L.net[net][l];
      a.l[net][l] = {reinterpret_cast<const uint4*>(m->shadow + li.sh_wf), reinterpret_cast<const float*>(m->shadow + li.sh_b), li.in_pad, li.out_pad};
    }
  a.nl = L.n_layers; a.net0 = do_policy ? 0 : 1;
  a.n = n; a.O = L.obs_dim; a.A = L.act_dim;
  a.vec_obs = ((uintptr_t)obs & 15) == 0 ? 1 : 0;
  a.lp_blocks = has_tile_forward(L) ? 0 : 1;      // the order in which this model's rollout_collect sums
  a.o_magic = magic((uint32_t)L.obs_dim);
  a.k0 = (uint32_t)seed; a.k1 = (uint32_t)(seed >> 32); a.step = step; a.env_offset = env_offset;
  a.log_std = reinterpret_cast<const float*>(m->shadow + L.sh_logstd);
  a.obs = obs; a.act = act; a.logp = logp; a.value = value; a.mu_out = mu_out;
  return R == 64 ? launch<2>(g, a, nets, lds) : launch<1>(g, a, nets, lds);
}

}  // namespace gmi
