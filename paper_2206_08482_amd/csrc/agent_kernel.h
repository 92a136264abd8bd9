// The agent's action decision in one launch (Section 3 of the paper, "DRL Agent"), bf16 and fp8 (E4M3): observation
// conversion, every layer of one net, and the Gaussian sampling epilogue.
//
// A workgroup of 8 (16) waves owns R = 32 RT rows of ONE net (grid: row tiles x nets).  The two nets meet nowhere: action and
// log-density need the policy net, the value needs the value net.  Activations are row-major [row][feature] in LDS (rows
// 16 bytes longer than their features: an odd number of 16-byte pieces, so that operand reads of consecutive rows hit
// different banks); layer l reads buffer l % 2 and writes the other one.  Products are computed transposed (weights first
// operand from the fragment-major copy in L2, activations second).  An item is one 32-feature tile for as many row tiles as
// still leave every wave an item; items are dealt to the waves, and a wave requests the first weight blocks of its next
// item, also across a layer's barrier, before it leaves the present one.  The random draws are made while the observations
// and the first weights are on their way.
//
// Bound, few rows: the chain of latencies launch - observations - one weight round trip per D k steps - heads -
// sampling.  Many rows: epilogue arithmetic, LDS operand reads, and weight blocks from L2 (once per workgroup).
//
// Sums run over k in ascending order from zero and the bias is added last: the bf16 results are those of rollout_collect
// (fused.hip, or this kernel and env.hip), bit for bit.
#pragma once
#include <algorithm>

#include "chain_stream.h"
#include "rng.h"

namespace gmi_agent {
using namespace gmi_chain;

constexpr int kMaxLayers = GMI_MAX_HIDDEN + 1;
constexpr size_t kLdsMax = 160 * 1024;

struct AgentLayer {
  const uint4* w;          // fragment-major W
  const float* bias;       // fp8: all layers' of a net one after the other
  const float* scale;      // fp8: what the layer's codes are multiples of
  int K, F;                // padded widths
};
struct AgentArgs {
  AgentLayer l[2][kMaxLayers];
  int nl, net0;            // blockIdx.y = 0 is net net0
  int n, O, A;
  int y_off, f_off;        // LDS bytes: second activation buffer, float area
  int bias_floats;         // of all layers, policy net (its head is the wider one)
  int vec_obs;             // the observations are 16-byte aligned
  int lp_blocks;           // log-density: 1 = blocks of 4 actions summed first, 0 = one action after the other
  uint32_t o_magic, pad_magic, nb_magic, k0, k1, step, env_offset;
  const float *log_std, *obs;
  float *act, *logp, *value, *mu_out;      // act NULL: means and values only
  // values_kernel: slot t < T reads obs + t obs_step and writes value + t val_step, slot T reads obs_last and writes value_last;
  // item = slot * tiles + row tile.
  int T, tiles, items;
  int64_t obs_step, val_step;
  const float* obs_last;
  float* value_last;
};

// 32x32x16 products of bf16.
struct Bf16 {
  static constexpr int size = 2, pieces = 1;      // bytes per element; 16-byte pieces of a lane's operand
  static constexpr bool bias_lds = false;         // biases in registers while an item is multiplied, or all of them in LDS
  static constexpr int align = 2;                 // k steps of a layer are a multiple of this
  static constexpr bool scaled = false;
  static __device__ __forceinline__ floatx16 mfma(const uint4 (&w)[1], const uint4 (&x)[1], floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w[0]), __builtin_bit_cast(bf16x8, x[0]), c, 0, 0, 0);
  }
  static __device__ __forceinline__ void store4(unsigned char* p, float a, float b, float c, float d) {
    *reinterpret_cast<uint2*>(p) = make_uint2(pack_bf16(a, b), pack_bf16(c, d));
  }
  static __device__ __forceinline__ void store_elu4(unsigned char* p, float a, float b, float c, float d) {
    store4(p, elu_f(a), elu_f(b), elu_f(c), elu_f(d));
  }
  static __device__ __forceinline__ void store1(unsigned char* p, float a) { *reinterpret_cast<uint16_t*>(p) = (uint16_t)pack_bf16(a, 0.f); }
};

// 32x32x64 products of E4M3: a lane's operand is 32 consecutive k of its row.
struct Fp8 {
  static constexpr int size = 1, pieces = 2;
  static constexpr bool bias_lds = true;          // (the operands leave no registers)
  static constexpr int align = 1;
  static constexpr bool scaled = true;
  static __device__ __forceinline__ intx8 join(const uint4 (&v)[2]) {
    const intx8 r = {(int)v[0].x, (int)v[0].y, (int)v[0].z, (int)v[0].w, (int)v[1].x, (int)v[1].y, (int)v[1].z, (int)v[1].w};
    return r;
  }
  static __device__ __forceinline__ floatx16 mfma(const uint4 (&w)[2], const uint4 (&x)[2], floatx16 c) {
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(join(w), join(x), c, 0, 0, 0, 0, 0, 0);
  }
  static __device__ __forceinline__ void store4(unsigned char* p, float a, float b, float c, float d) {
    *reinterpret_cast<uint32_t*>(p) = to_e4m3x4(a, b, c, d);
  }
  static __device__ __forceinline__ void store_elu4(unsigned char* p, float a, float b, float c, float d) {
    *reinterpret_cast<uint32_t*>(p) = elu_e4m3x4(a, b, c, d);
  }
  static __device__ __forceinline__ void store1(unsigned char* p, float a) { *p = (unsigned char)to_e4m3x4(a, 0.f, 0.f, 0.f); }
};

__host__ __device__ __forceinline__ uint32_t magic(uint32_t d) { return d == 1 ? 0u : 0xFFFFFFFFu / d + 1u; }
__device__ __forceinline__ int div_magic(int n, uint32_t m) { return m ? (int)__umulhi((uint32_t)n, m) : n; }      // n * d < 2^32

template <class P, int D>
using Ring = uint4[D][P::pieces];

// acc[i] += W tile x row tiles at xp, xp + xts bytes; w: the tile's weight blocks (wave-uniform), of which wq holds the first k
// steps' for this lane.
template <class P, int D, int NRT>
__device__ __forceinline__ void k_loop(floatx16 (&acc)[NRT], Ring<P, D>& wq, const uint4* w, int nks, const unsigned char* xp, int xts, int lane) {
  constexpr int B = 32 * P::pieces;      // bytes of a row per k step
  uint4 x[2][NRT][P::pieces];
  auto read = [&](int b, int ks) {
#pragma unroll
    for (int i = 0; i < NRT; ++i)
#pragma unroll
      for (int p = 0; p < P::pieces; ++p) x[b][i][p] = *reinterpret_cast<const uint4*>(xp + i * xts + B * ks + 16 * p);
  };
  read(0, 0);
  auto step = [&](int ks, int u) {
    read((u + 1) & 1, min(ks + 1, nks - 1));
#pragma unroll
    for (int i = 0; i < NRT; ++i) acc[i] = P::mfma(wq[u], x[u & 1][i], acc[i]);
  };
  int ks = 0;
  for (; ks + D < nks; ks += D)
#pragma unroll
    for (int u = 0; u < D; ++u) {
      step(ks + u, u);
#pragma unroll
      for (int p = 0; p < P::pieces; ++p)
        wq[u][p] = gmi::load_uniform(w, (min(ks + u + D, nks - 1) * P::pieces + p) * 1024, lane * 16);
    }
#pragma unroll
  for (int u = 0; u < D; u += P::align)
    if (ks + u < nks)
#pragma unroll
      for (int v = 0; v < P::align; ++v) step(ks + u + v, u + v);
}

// Row tiles of an item of a product with nft feature tiles: as many (at most MT) as still leave every wave an item.
template <int RT, int MT, int NW>
__device__ __forceinline__ int item_tiles(int nft) {
  return MT >= 2 && nft * (RT / 2) >= NW ? 2 : 1;
}

// Requests the first weight blocks of an item of layer L.
template <class P, int RT, int D, int MT, int NW>
__device__ __forceinline__ void request(Ring<P, D>& wq, const AgentLayer& L, int item, int lane) {
  const int nft = L.F >> 5, nks = L.K * P::size / (32 * P::pieces);
  const int ft = min(item / (RT / item_tiles<RT, MT, NW>(nft)), nft - 1);
  const uint4* w = L.w + (int64_t)ft * nks * 64 * P::pieces;
#pragma unroll
  for (int u = 0; u < D; ++u)
#pragma unroll
    for (int p = 0; p < P::pieces; ++p) wq[u][p] = gmi::load_uniform(w, (min(u, nks - 1) * P::pieces + p) * 1024, lane * 16);
}

// All layers of a net on the workgroup's 32 RT rows.  Layer 0 reads the rows at x0; odd layers read ya, even ones yb (which
// may be x0); a row of a layer's input takes K * P::size + 16 bytes.  The head's results go to s_head [row][ho].  wq holds
// the first blocks of layer 0 for item `wave`; AGAIN: so it does afterwards, for the next pass.  Ends with a barrier.
template <class P, int RT, int D, int MT, int NW, bool AGAIN>
__device__ __forceinline__ void net_layers(const AgentLayer* N, int nl, Ring<P, D>& wq, const unsigned char* x0, unsigned char* ya,
                                           unsigned char* yb, const float* s_bias, float* s_head, int ho, int wave, int lane) {
  constexpr int B = 32 * P::pieces;
  const int s = lane & 31, h = lane >> 5;
  const float* bias = s_bias + 4 * h;
  for (int l = 0; l < nl; ++l) {
    const AgentLayer& L = N[l];
    const AgentLayer& Ln = N[l + 1 < nl ? l + 1 : 0];
    const int nft = L.F >> 5, nks = L.K * P::size / B, sx = L.K * P::size + 16, sy = L.F * P::size + 16;
    const unsigned char* x = l == 0 ? x0 : l & 1 ? ya : yb;
    unsigned char* y = l & 1 ? yb : ya;
    const bool head = l == nl - 1;
    const bool more = AGAIN || !head;
    float scale = 1.f;
    if constexpr (P::scaled) scale = *L.scale;
    auto items = [&](auto nrt) {
      constexpr int NRT = decltype(nrt)::value;
      constexpr int nrg = RT / NRT;
      const int n_items = nft * nrg;
      // One kind of item and one pass (MT == 1, !AGAIN): a wave without an item goes through the motions, so that one place in the code
      // requests weights; where the registers of loads from two places meet, the compiler copies them, and a copy waits for the
      // load ahead of the layer's barrier.
      constexpr bool kGhost = MT == 1 && !AGAIN;
      for (int item = wave; kGhost ? item == wave || item < n_items : item < n_items; item += NW) {
        const int it = kGhost ? min(item, n_items - 1) : item, ft = it / nrg, rg = it % nrg;
        float4 b4[4];
        if constexpr (!P::bias_lds)
#pragma unroll
          for (int q = 0; q < 4; ++q) b4[q] = *reinterpret_cast<const float4*>(L.bias + 32 * ft + 8 * q + 4 * h);
        floatx16 acc[NRT];
#pragma unroll
        for (int i = 0; i < NRT; ++i)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
        if (!kGhost || item < n_items) k_loop<P, D, NRT>(acc, wq, L.w + (int64_t)ft * nks * 64 * P::pieces, nks, x + (rg * NRT * 32 + s) * sx + B / 2 * h, 32 * sx, lane);
        if constexpr (kGhost) {
          const bool again = item + NW < n_items;
          request<P, RT, D, MT, NW>(wq, again ? L : Ln, again ? item + NW : wave, lane);
          if (item >= n_items) break;
        } else {
          if (item + NW < n_items) request<P, RT, D, MT, NW>(wq, L, item + NW, lane);
          else if (more) request<P, RT, D, MT, NW>(wq, Ln, wave, lane);
        }
        // lane (s, h) holds, per quad q, the features 32 ft + 8 q + 4 h + 0..3 of row s
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int f = 32 * ft + 8 * q + 4 * h;
          float4 b;
          if constexpr (P::bias_lds) b = *reinterpret_cast<const float4*>(bias + 32 * ft + 8 * q);
          else b = b4[q];
#pragma unroll
          for (int i = 0; i < NRT; ++i) {
            const int r = (rg * NRT + i) * 32 + s;
            float v[4] = {acc[i][4 * q], acc[i][4 * q + 1], acc[i][4 * q + 2], acc[i][4 * q + 3]};
            if constexpr (P::scaled) {
              v[0] = fmaf(v[0], scale, b.x); v[1] = fmaf(v[1], scale, b.y); v[2] = fmaf(v[2], scale, b.z); v[3] = fmaf(v[3], scale, b.w);
            } else {
              v[0] += b.x; v[1] += b.y; v[2] += b.z; v[3] += b.w;
            }
            if (!head) {
              P::store_elu4(y + r * sy + f * P::size, v[0], v[1], v[2], v[3]);
            } else {
              float* d = s_head + r * ho + f;
#pragma unroll
              for (int e = 0; e < 4; ++e)
                if (f + e < ho) d[e] = v[e];
            }
          }
        }
      }
      if (!kGhost && wave >= n_items && more) request<P, RT, D, MT, NW>(wq, Ln, wave, lane);
    };
    const int nrt = item_tiles<RT, MT, NW>(nft);
    if (nrt == 1) items(std::integral_constant<int, 1>{});
    if constexpr (MT >= 2) if (nrt == 2) items(std::integral_constant<int, 2>{});
    bias += L.F;
    __syncthreads();
  }
}

// The workgroup's observation rows into LDS (rows of K0 elements).  They are rows * O consecutive floats at src; 16-byte pieces
// of them may span two rows.
template <class P, int RT, int NW>
__device__ __forceinline__ void stage_obs(const AgentArgs& a, int K0, const float* src, int rows, unsigned char* s_x, int tid) {
  constexpr int R = 32 * RT, kNT = 64 * NW;
  const int O = a.O, S0 = K0 * P::size + 16;
  const int cnt = rows * O, n4 = a.vec_obs ? cnt >> 2 : 0;
  for (int e0 = tid; e0 < n4; e0 += 4 * kNT) {
    float4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = reinterpret_cast<const float4*>(src)[min(e0 + u * kNT, n4 - 1)];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = 4 * min(e0 + u * kNT, n4 - 1);
      int r = div_magic(e, a.o_magic), c = e - r * O;
      if ((O & 3) == 0) {
        P::store4(s_x + r * S0 + c * P::size, v[u].x, v[u].y, v[u].z, v[u].w);
      } else {
        const float q[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          P::store1(s_x + r * S0 + c * P::size, q[i]);
          if (++c == O) { c = 0; ++r; }
        }
      }
    }
  }
  for (int e = 4 * n4 + tid; e < cnt; e += kNT) {
    const int r = div_magic(e, a.o_magic);
    P::store1(s_x + r * S0 + (e - r * O) * P::size, src[e]);
  }
  // padding columns, and rows past the end (never stored: any finite value will do)
  const int np = K0 - O;
  for (int e = tid; e < np * R; e += kNT) {
    const int r = div_magic(e, a.pad_magic);
    P::store1(s_x + r * S0 + (O + e - r * np) * P::size, 0.f);
  }
  for (int e = rows * (S0 >> 4) + tid; e < R * (S0 >> 4); e += kNT) reinterpret_cast<uint4*>(s_x)[e] = make_uint4(0u, 0u, 0u, 0u);
}

// D: weight blocks in flight per wave; MT: most row tiles of an item; WPS: waves per SIMD (registers); NW: waves.
template <class P, int RT, int D, int MT, int WPS, int NW>
__global__ __launch_bounds__(64 * NW, WPS) void agent_kernel(AgentArgs a) {
  constexpr int R = 32 * RT, kNT = 64 * NW;
  extern __shared__ __attribute__((aligned(16))) unsigned char s_x[];
  const int net = a.net0 + blockIdx.y;
  const AgentLayer* N = a.l[net];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nl = a.nl, K0 = N[0].K;
  const int ho = net == 0 ? a.A : 1, nb = a.act ? (a.A + 3) >> 2 : 0;          // head outputs; blocks of 4 actions
  float4* s_noise = reinterpret_cast<float4*>(s_x + a.f_off);                  // [R][nb]
  float* s_bias = reinterpret_cast<float*>(s_noise + R * nb);                  // of all layers, one after the other
  float* s_head = s_bias + a.bias_floats;                                      // [R][ho]
  const int r0 = blockIdx.x * R, rows = min(R, a.n - r0);

  Ring<P, D> wq;
  // this thread's first action element, its log_std requested ahead of everything
  auto element = [&](int item) {
    const int blk = item >> 2;
    return 4 * (blk - div_magic(blk, a.nb_magic) * nb) + (item & 3);
  };
  float ls = 0.f;
  if (net == 0 && nb > 0) ls = a.log_std[min(element(tid), a.A - 1)];
  // biases in LDS: requested here, stored after the observations
  float bv[P::bias_lds ? 4 : 1];
  if constexpr (P::bias_lds)
#pragma unroll
    for (int u = 0; u < 4; ++u) bv[u] = N[0].bias[min(tid + u * kNT, a.bias_floats - 1)];
  stage_obs<P, RT, NW>(a, K0, a.obs + (int64_t)r0 * a.O, rows, s_x, tid);
  request<P, RT, D, MT, NW>(wq, N[0], wave, lane);
  if constexpr (P::bias_lds) {
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (tid + u * kNT < a.bias_floats) s_bias[tid + u * kNT] = bv[u];
    for (int f = tid + 4 * kNT; f < a.bias_floats; f += kNT) s_bias[f] = N[0].bias[f];
  }
  if (net == 0)
    for (int item = tid; item < rows * nb; item += kNT) {
      const int r = div_magic(item, a.nb_magic), b = item - r * nb;
      float z[4];
      gmi::normal_block(a.env_offset + (uint32_t)(r0 + r), a.step, gmi::kStreamAction, (uint32_t)b, a.k0, a.k1, z);
      s_noise[item] = make_float4(z[0], z[1], z[2], z[3]);
    }
  __syncthreads();

  net_layers<P, RT, D, MT, NW, false>(N, nl, wq, s_x, s_x + a.y_off, s_x, s_bias, s_head, ho, wave, lane);

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
  float sigma = expf(ls);
  for (int item = tid; item < rows * nb * 4; item += kNT) {
    const int r = div_magic(item >> 2, a.nb_magic), j = element(item);
    if (item != tid && j < A) {
      ls = a.log_std[j];
      sigma = expf(ls);
    }
    float* zp = reinterpret_cast<float*>(s_noise) + item;
    float term = 0.f;
    if (j < A) {
      const float z = *zp, m = s_head[r * A + j];
      const int64_t o = (int64_t)(r0 + r) * A + j;
      a.act[o] = fmaf(sigma, z, m);
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

// Values of several steps at once, items one after the other: a collection's values would be thousands of workgroups (4096 envs
// and 32 steps: 4224, on 64 compute units in the four-agent pipeline), and a launch that its compute units cannot hold keeps
// kernels of other streams waiting.  The next item's first weights are on their way while the present one ends.
template <class P, int RT, int D, int MT, int WPS>
__global__ __launch_bounds__(512, WPS) void values_kernel(AgentArgs a) {
  static_assert(!P::bias_lds, "no room for biases in this layout");
  constexpr int R = 32 * RT, kNT = 512;
  extern __shared__ __attribute__((aligned(16))) unsigned char s_x[];
  const AgentLayer* N = a.l[1];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  float* s_head = reinterpret_cast<float*>(s_x + a.f_off);
  Ring<P, D> wq;
  request<P, RT, D, MT, 8>(wq, N[0], wave, lane);
  for (int item = blockIdx.x; item < a.items; item += gridDim.x) {
    const int t = item / a.tiles, r0 = (item - t * a.tiles) * R, rows = min(R, a.n - r0);
    stage_obs<P, RT, 8>(a, N[0].K, (t < a.T ? a.obs + t * a.obs_step : a.obs_last) + (int64_t)r0 * a.O, rows, s_x, tid);
    __syncthreads();
    // ends with a barrier: the rows may be replaced; s_head is written again behind the next pass's first barrier
    net_layers<P, RT, D, MT, 8, true>(N, a.nl, wq, s_x, s_x + a.y_off, s_x, nullptr, s_head, 1, wave, lane);
    float* dst = t < a.T ? a.value + t * a.val_step : a.value_last;
    for (int r = tid; r < rows; r += kNT) dst[r0 + r] = s_head[r];
  }
}

// Lays out the LDS of a tile of 32 rt rows and returns its bytes; sample: with the draws and log-density terms (else means only).
template <class P>
size_t agent_lds(AgentArgs& a, int rt, bool sample) {
  int w[2] = {0, 0};
  a.bias_floats = 0;
  for (int l = 0; l < a.nl; ++l) {
    w[l & 1] = std::max(w[l & 1], a.l[0][l].K * P::size + 16);
    if (P::bias_lds) a.bias_floats += a.l[0][l].F;
  }
  a.o_magic = magic((uint32_t)a.O);
  a.pad_magic = magic((uint32_t)std::max(a.l[0][0].K - a.O, 1));
  a.nb_magic = magic((uint32_t)((a.A + 3) / 4));
  a.y_off = 32 * rt * w[0];
  a.f_off = 32 * rt * (w[0] + w[1]);
  return (size_t)a.f_off + (size_t)32 * rt * ((sample ? (a.A + 3) / 4 * 16 : 0) + a.A * 4) + (size_t)a.bias_floats * 4;
}

template <class P, int RT, int D, int MT, int WPS, int NW = 8>
int launch(gmi_instance* g, AgentArgs& a, int nets, bool sample) {
  const size_t lds = agent_lds<P>(a, RT, sample);
  static gmi::DeviceSet allowed;
  const int rc = gmi::allow_lds((const void*)agent_kernel<P, RT, D, MT, WPS, NW>, kLdsMax, g->device, &allowed);
  if (rc != GMI_OK) return rc;
  gmi::ProfScope ps(g, gmi::kClsFusedAgent);
  ps.launch(agent_kernel<P, RT, D, MT, WPS, NW>, dim3((a.n + 32 * RT - 1) / (32 * RT), nets), dim3(64 * NW), lds, a);
  GMI_LAUNCH_CHECK();
  return GMI_OK;
}

template <class P, int RT, int D, int MT, int WPS>
int launch_slots(gmi_instance* g, AgentArgs& a) {
  const size_t lds = agent_lds<P>(a, RT, false);
  const void* kernel = (const void*)values_kernel<P, RT, D, MT, WPS>;
  static gmi::DeviceSet allowed;
  int rc = gmi::allow_lds(kernel, kLdsMax, g->device, &allowed);
  if (rc != GMI_OK) return rc;
  int64_t resident = 1;
  rc = gmi::resident_groups(g, kernel, 512, lds, &resident);
  if (rc != GMI_OK) return rc;
  a.tiles = (a.n + 32 * RT - 1) / (32 * RT);
  a.items = a.tiles * (a.T + (a.value_last ? 1 : 0));
  const int64_t rounds = (a.items + resident - 1) / resident;
  gmi::ProfScope ps(g, gmi::kClsFusedAgent);
  ps.launch(values_kernel<P, RT, D, MT, WPS>, dim3((unsigned)((a.items + rounds - 1) / rounds)), dim3(512), lds, a);
  GMI_LAUNCH_CHECK();
  return GMI_OK;
}

}  // namespace gmi_agent
