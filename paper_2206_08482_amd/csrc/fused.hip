// One-launch collection kernel: a workgroup owns a tile of R samples (envs), keeps the activations of the
// tile in LDS (bf16) from layer to layer, and streams each layer's bf16 weights from L2 straight into the
// matrix cores' weight operand.
#include "agent_kernel.h"
#include "rng.h"
#include "rollout.h"

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;
typedef float float2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));

using gmi::elu_f;
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  float2v v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2v));
}

struct FusedNet {
  const uint16_t* w[GMI_MAX_HIDDEN + 1];     // bf16, fragment-major copy of W [out_pad, in_pad]
  const float* bias[GMI_MAX_HIDDEN + 1];     // fp32 [out_pad]
  int in_pad[GMI_MAX_HIDDEN + 1], out_pad[GMI_MAX_HIDDEN + 1];
  int bias_off[GMI_MAX_HIDDEN + 1];          // offset (floats) of the layer's bias inside a net's LDS bias block
  int bias_total;                            // floats of that block
  int n_layers;
  int out_store;                             // logical outputs of the head
};

enum { kFEpiElu = 0, kFEpiHead = 1 };

// Copies the biases of all layers of a net into LDS (dst[bias_off[l] + f]); the caller synchronises.
__device__ __forceinline__ void stage_biases(const FusedNet& N, float* dst, int tid0, int nthreads) {
  for (int l = 0; l < N.n_layers; ++l)
    for (int f = tid0; f < N.out_pad[l]; f += nthreads) dst[N.bias_off[l] + f] = N.bias[l][f];
}


// ------------------------------------------------------------------------------------------------
// Experience collection of a whole horizon in one launch (Section 5.1, stage (i), with the simulator and
// the agent co-located in one instance as in Section 3): envs are independent of each other, so a workgroup
// can own R envs for all T steps and keep their state in LDS: per step it decides the actions (both nets +
// Gaussian sampling), records the experience slot, and advances the linear-Gaussian simulator; after the last
// step it evaluates the bootstrap value of the final state.  Arithmetic and Philox counters are those of
// agent_act / env_step / collect_experience called step by step.
struct RolloutArgs : RolloutEnv {
  FusedNet net[2];
  gmi_agent::AgentLayer policy[gmi_agent::kMaxLayers];      // the streaming form's view of the policy net
  int obs_pad, max_h;
  int mr_lds;                       // m_r: 2 = LDS copy kept for the whole launch, 1 = LDS copy made at every
                                    // step in the (then idle) hidden-activation space, 0 = read from global
  int ahead;                        // 1 = step t + 1's random draws are made beside step t's simulator (two buffers)
  // LDS bytes: next to the state rows at 0 ([2][rows_per_wg][OS] state | action, of this and the next step)
  int x0_off, hid_off, mu_off, val_off, lp_off, part_off, done_off, ls_off, bias_off, m_off, w_off, draw_off;
};

// ------------------------------------------------------------------------------------------------
// Weight-stationary form of the layers, for model shapes whose share of the weights fits a wave's registers:
// the one-launch rollout runs the same layers T + 1 times, so each wave fetches the operand blocks of ITS
// feature tiles once, at kernel start, and keeps them in registers for all steps (streamed from L2 they cost
// ~2000 cycles of latency per layer and step).  Same products in the same order as the streaming form: results are
// bit-identical.  DIMS = padded widths d[0..NL] (input, hidden..., head).
template <class WS> struct WsFrags { static constexpr int value = WS::n_frags(); };
template <> struct WsFrags<void> { static constexpr int value = 1; };

// Layers LDSL.. keep their operand blocks in LDS instead (one copy per net, fragment-major as in global memory):
// with every layer in registers the kernel needed more than the 256 registers two waves per SIMD leave and the
// compiler parked values in scratch memory, whose reloads sat in every phase of every step.
template <int LDSL, int... DIMS>
struct WsShape {
  static constexpr int NL = (int)sizeof...(DIMS) - 1;
  static constexpr int lds_from = LDSL;
  static constexpr int dim(int i) {
    constexpr int d[] = {DIMS...};
    return d[i];
  }
  static constexpr int max_tiles(int l) { return (dim(l + 1) / 32 + 3) / 4; }      // feature tiles of one wave
  static constexpr int frag_base(int l) {
    int n = 0;
    for (int i = 0; i < l && i < LDSL; ++i) n += max_tiles(i) * (dim(i) / 16);
    return n;
  }
  static constexpr int n_frags() { return frag_base(NL) > 0 ? frag_base(NL) : 1; }
  // the 16-env form (16x16x32 products): 16-feature tiles of one wave, and its register fragments before layer l
  static constexpr int max_tiles16(int l) { return (dim(l + 1) / 16 + 3) / 4; }
  static constexpr int frag_base16(int l) {
    int n = 0;
    for (int i = 0; i < l && i < LDSL; ++i) n += max_tiles16(i) * (dim(i) / 32);
    return n;
  }
  // bf16 elements of the LDS-resident layers before layer l / of all of them (one net)
  static constexpr int lds_base(int l) {
    int n = 0;
    for (int i = LDSL; i < l; ++i) n += (dim(i + 1) / 32) * (dim(i) / 16) * 512;
    return n;
  }
  static constexpr int lds_elems() { return lds_base(NL); }
};

template <class WS, int L>
__device__ __forceinline__ void ws_load(bf16x8* wreg, const FusedNet& N, int wave, int lane) {
  if constexpr (L < WS::NL && L < WS::lds_from) {
    constexpr int nks = WS::dim(L) / 16, nft = WS::dim(L + 1) / 32, base = WS::frag_base(L);
#pragma unroll
    for (int i = 0; i < WS::max_tiles(L); ++i) {
      const int tile = wave + 4 * i;
      const int tc = tile < nft ? tile : nft - 1;       // a wave without an i-th tile loads a valid block it never uses
      const uint16_t* p = N.w[L] + ((int64_t)tc * nks) * 512 + lane * 8;
#pragma unroll
      for (int ks = 0; ks < nks; ++ks) wreg[base + i * nks + ks] = *reinterpret_cast<const bf16x8*>(p + (int64_t)ks * 512);
    }
    ws_load<WS, L + 1>(wreg, N, wave, lane);
  }
}

// Copies the operand blocks of the LDS-resident layers of one net into s_w (all threads of the workgroup).
template <class WS, int L>
__device__ __forceinline__ void ws_stage(uint16_t* s_w, const FusedNet& N, int tid, int nthreads) {
  if constexpr (L < WS::NL) {
    if constexpr (L >= WS::lds_from) {
      constexpr int n16 = (WS::dim(L + 1) / 32) * (WS::dim(L) / 16) * 64;       // 16-byte pieces
      const uint4* src = reinterpret_cast<const uint4*>(N.w[L]);
      uint4* dst = reinterpret_cast<uint4*>(s_w + WS::lds_base(L));
      for (int i = tid; i < n16; i += nthreads) dst[i] = src[i];
    }
    ws_stage<WS, L + 1>(s_w, N, tid, nthreads);
  }
}

template <class WS, int L, int RT, int EPI>
__device__ __forceinline__ void ws_layer(const bf16x8* wreg, const uint16_t* s_w, const float* s_bias, const uint16_t* s_in, int stride_in,
                                         uint16_t* s_out, int stride_out, float* s_head, int head_stride,
                                         int out_store, int wave, int lane) {
  constexpr int nks = WS::dim(L) / 16, nft = WS::dim(L + 1) / 32, base = WS::frag_base(L);
  const int khalf = (lane >> 5) * 8;
  const uint16_t* xrow = s_in + (lane & 31) * stride_in + khalf;
#pragma unroll
  for (int i = 0; i < WS::max_tiles(L); ++i) {
    const int tile = wave + 4 * i;
    if (tile < nft) {                                   // wave-uniform
      floatx16 acc[RT];
#pragma unroll
      for (int j = 0; j < RT; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
#pragma unroll
      for (int ks = 0; ks < nks; ++ks)
#pragma unroll
        for (int j = 0; j < RT; ++j) {
          const bf16x8 b = *reinterpret_cast<const bf16x8*>(xrow + j * 32 * stride_in + ks * 16);
          bf16x8 w;
          if constexpr (L < WS::lds_from) w = wreg[base + i * nks + ks];
          else w = *reinterpret_cast<const bf16x8*>(s_w + WS::lds_base(L) + (tile * nks + ks) * 512 + lane * 8);
          acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, b, acc[j], 0, 0, 0);
        }
      const int fb = tile * 32;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int f = fb + g * 8 + (lane >> 5) * 4;
        const float4 bv = *reinterpret_cast<const float4*>(s_bias + f);
#pragma unroll
        for (int j = 0; j < RT; ++j) {
          const int r = j * 32 + (lane & 31);
          const float o0 = acc[j][g * 4 + 0] + bv.x, o1 = acc[j][g * 4 + 1] + bv.y;
          const float o2 = acc[j][g * 4 + 2] + bv.z, o3 = acc[j][g * 4 + 3] + bv.w;
          if (EPI == kFEpiElu) {
            *reinterpret_cast<uint2*>(&s_out[r * stride_out + f]) =
                make_uint2(pack_bf16(elu_f(o0), elu_f(o1)), pack_bf16(elu_f(o2), elu_f(o3)));
          } else {
            float* d = s_head + r * head_stride + f;
            if (f + 0 < out_store) d[0] = o0;
            if (f + 1 < out_store) d[1] = o1;
            if (f + 2 < out_store) d[2] = o2;
            if (f + 3 < out_store) d[3] = o3;
          }
        }
      }
    }
  }
}

// ---- The 16-env form of the weight-stationary nets (a workgroup that owns 16 envs): 16x16x32 products on
// 16-feature tiles, so that no row of a tile is padding -- half the matrix-instruction passes and half the epilogue
// arithmetic of the 32-row tiles.  The sums are bit-identical to those of the 32x32x16 products over the same k order
// (checked on the device over 256000 outputs of mixed magnitudes before this form was written), so the rollout stays
// bit-identical to the per-step kernels.
// Element offset, inside a layer's fragment-major array, of the 8 consecutive k values from k0 (a multiple of 8) of
// feature f: block (f / 32, k0 / 16), lane f % 32 + 32 * ((k0 / 8) % 2) of the 32x32x16 layout.
__device__ __forceinline__ int wfrag16_off(int f, int k0, int nks16) {
  return ((((f >> 5) * nks16 + (k0 >> 4)) * 64) + (f & 31) + 32 * ((k0 >> 3) & 1)) * 8;
}

template <class WS, int L>
__device__ __forceinline__ void ws_load16(bf16x8* wreg, const FusedNet& N, int wave, int lane) {
  if constexpr (L < WS::NL && L < WS::lds_from) {
    constexpr int nks = WS::dim(L) / 32, nks16 = WS::dim(L) / 16, nft = WS::dim(L + 1) / 16, base = WS::frag_base16(L);
    static_assert(WS::frag_base16(L + 1) <= WS::n_frags(), "the 16-env form fits the register fragments of the 32-env form");
#pragma unroll
    for (int i = 0; i < WS::max_tiles16(L); ++i) {
      const int tile = wave + 4 * i;
      const int tc = tile < nft ? tile : nft - 1;       // a wave without an i-th tile loads a valid block it never uses
      const int f = tc * 16 + (lane & 15);
#pragma unroll
      for (int ks = 0; ks < nks; ++ks)
        wreg[base + i * nks + ks] =
            *reinterpret_cast<const bf16x8*>(N.w[L] + wfrag16_off(f, ks * 32 + (lane >> 4) * 8, nks16));
    }
    ws_load16<WS, L + 1>(wreg, N, wave, lane);
  }
}

template <class WS, int L, int EPI>
__device__ __forceinline__ void ws_layer16(const bf16x8* wreg, const uint16_t* s_w, const float* s_bias, const uint16_t* s_in,
                                           int stride_in, uint16_t* s_out, int stride_out, float* s_head, int head_stride,
                                           int out_store, int wave, int lane) {
  constexpr int nks = WS::dim(L) / 32, nks16 = WS::dim(L) / 16, nft = WS::dim(L + 1) / 16, base = WS::frag_base16(L);
  const int q = lane >> 4, n = lane & 15;               // lane (n, q): env n, k values 8 q .. + 7 of a k step, features 4 q .. + 3 of a tile
  const uint16_t* xrow = s_in + n * stride_in + q * 8;
#pragma unroll
  for (int i = 0; i < WS::max_tiles16(L); ++i) {
    const int tile = wave + 4 * i;
    if (tile < nft) {                                   // wave-uniform
      floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < nks; ++ks) {
        const bf16x8 b = *reinterpret_cast<const bf16x8*>(xrow + ks * 32);
        bf16x8 w;
        if constexpr (L < WS::lds_from) w = wreg[base + i * nks + ks];
        else w = *reinterpret_cast<const bf16x8*>(s_w + WS::lds_base(L) + wfrag16_off(tile * 16 + n, ks * 32 + q * 8, nks16));
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, b, acc, 0, 0, 0);
      }
      const int f = tile * 16 + 4 * q;
      const float4 bv = *reinterpret_cast<const float4*>(s_bias + f);
      const float o0 = acc[0] + bv.x, o1 = acc[1] + bv.y, o2 = acc[2] + bv.z, o3 = acc[3] + bv.w;
      if (EPI == kFEpiElu) {
        *reinterpret_cast<uint2*>(&s_out[n * stride_out + f]) =
            make_uint2(pack_bf16(elu_f(o0), elu_f(o1)), pack_bf16(elu_f(o2), elu_f(o3)));
      } else {
        float* d = s_head + n * head_stride + f;
        if (f + 0 < out_store) d[0] = o0;
        if (f + 1 < out_store) d[1] = o1;
        if (f + 2 < out_store) d[2] = o2;
        if (f + 3 < out_store) d[3] = o3;
      }
    }
  }
}

template <class WS, int L, class Idle>
__device__ __forceinline__ void ws_net16(const bf16x8* wreg, const uint16_t* s_w, const FusedNet& N, const float* s_nb,
                                         const uint16_t* in, int stride_in, uint16_t* s_a, uint16_t* s_b, int stride_h,
                                         float* s_head, int head_stride, bool run, int wave, int lane, Idle idle) {
  if constexpr (L < WS::NL - 1) {
    uint16_t* out = (L & 1) ? s_b : s_a;
    if (run)
      ws_layer16<WS, L, kFEpiElu>(wreg, s_w, s_nb + N.bias_off[L], in, stride_in, out, stride_h, nullptr, 0, 0, wave, lane);
    __syncthreads();
    ws_net16<WS, L + 1>(wreg, s_w, N, s_nb, out, stride_h, s_a, s_b, stride_h, s_head, head_stride, run, wave, lane, idle);
  } else {
    if (run)
      ws_layer16<WS, L, kFEpiHead>(wreg, s_w, s_nb + N.bias_off[L], in, stride_in, nullptr, 0, s_head, head_stride,
                                   N.out_store, wave, lane);
    idle();
    __syncthreads();
  }
}

// All layers of one net from layer L on, hidden activations ping-ponging between s_a and s_b as in the
// streaming form; every layer ends with a workgroup barrier.
template <class WS, int L, int RT, class Idle>
__device__ __forceinline__ void ws_net(const bf16x8* wreg, const uint16_t* s_w, const FusedNet& N, const float* s_nb, const uint16_t* in,
                                       int stride_in, uint16_t* s_a, uint16_t* s_b, int stride_h, float* s_head,
                                       int head_stride, bool run, int wave, int lane, Idle idle) {
  if constexpr (L < WS::NL - 1) {
    uint16_t* out = (L & 1) ? s_b : s_a;
    if (run)
      ws_layer<WS, L, RT, kFEpiElu>(wreg, s_w, s_nb + N.bias_off[L], in, stride_in, out, stride_h, nullptr, 0, 0, wave, lane);
    __syncthreads();
    ws_net<WS, L + 1, RT>(wreg, s_w, N, s_nb, out, stride_h, s_a, s_b, stride_h, s_head, head_stride, run, wave, lane, idle);
  } else {
    if (run)
      ws_layer<WS, L, RT, kFEpiHead>(wreg, s_w, s_nb + N.bias_off[L], in, stride_in, nullptr, 0, s_head, head_stride,
                                     N.out_store, wave, lane);
    idle();
    __syncthreads();
  }
}

// Shapes with a weight-stationary rollout: the first two layers in registers (24 operand blocks = 96 registers per
// wave), the last two in LDS (20 KiB per net).
using WsAnt = WsShape<2, 64, 256, 128, 64, 32>;         // 60:256:128:64:8 (benchmark workload C2), 48:256:128:64:12
using WsSmallObs = WsShape<2, 32, 256, 128, 64, 32>;    // 24:256:128:64:3, 23:256:128:64:9

template <class WS>
bool ws_matches(const ModelLayout& L) {
  if (L.n_layers != WS::NL) return false;
  for (int net = 0; net < 2; ++net)
    for (int l = 0; l < WS::NL; ++l)
      if (L.net[net][l].in_pad != WS::dim(l) || L.net[net][l].out_pad != WS::dim(l + 1)) return false;
  return true;
}

// ---- The streaming form for 16 envs per workgroup: the policy net on 16x16x32 products, 16 features a tile, dealt to all 8 waves.
// With 32x32x16 tiles half of the products and of the epilogue's instructions are padding rows and half of the waves have no tile
// of a 128-wide layer: three layers of 45:128:128:12 took 8300 cycles.  wq holds the first weight blocks of layer 0 for this
// wave, and again afterwards.
// One place in the code requests weights, and no branch goes around it (clamped addresses instead): where the registers of loads
// from two places meet, the compiler copies them, and a copy waits for the load (2500 cycles a layer instead of 1500).
constexpr int kAhead16 = 8;
typedef uint4 Ring16[kAhead16];
struct Walk16 {
  const char* w;      // weights of the wave's tile: wave-uniform
  int nks;            // k steps
};
// Where the weights of tile `tile` (the last one if there are fewer) of a layer start; lane_off is the lane's place in a k step's
// 2 KiB.
__device__ __forceinline__ Walk16 walk16(const uint4* w, int K, int F, int tile) {
  const int t = min(tile, (F >> 4) - 1);
  return {reinterpret_cast<const char*>(w) + (int64_t)(t >> 1) * (K >> 4) * 1024 + 256 * (t & 1), K >> 5};
}
__device__ __forceinline__ void request16(Ring16& wq, const Walk16& k, uint32_t lane_off) {
#pragma unroll
  for (int u = 0; u < kAhead16; ++u) wq[u] = gmi::load_uniform(k.w, min(u, k.nks - 1) * 2048, lane_off);
}
// idle(): called once by wave 7, in the last layer, whose tiles are the fewest.
template <class Idle>
__device__ __forceinline__ void net_layers16(const gmi_agent::AgentLayer* N, int nl, Ring16& wq, const unsigned char* x0, unsigned char* ya,
                                             unsigned char* yb, const float* s_bias, float* s_head, int ho, int wave, int lane, Idle idle) {
  const int n = lane & 15, q = lane >> 4;      // lane (n, q): env n, k values 8 q .. + 7 of a k step, features 4 q .. + 3 of a tile
  const uint32_t lane_off = ((q >> 1) * 64 + n + 32 * (q & 1)) * 16;
  const uint4* w = N[0].w;
  int K = N[0].K, F = N[0].F;
  for (int l = 0; l < nl; ++l) {
    const gmi_agent::AgentLayer& Ln = N[l + 1 < nl ? l + 1 : 0];
    const uint4* wn = Ln.w;
    const int Kn = Ln.K, Fn = Ln.F;
    const int nt = F >> 4, sx = K * 2 + 16, sy = F * 2 + 16;
    const unsigned char* x = (l == 0 ? x0 : l & 1 ? ya : yb) + n * sx + 16 * q;
    unsigned char* y = (l & 1 ? yb : ya) + n * sy + 8 * q;
    const bool head = l == nl - 1;
    int tile = wave;
    do {      // a wave without a tile multiplies the last one again and drops it
      const Walk16 k = walk16(w, K, F, tile);
      const float4 b = *reinterpret_cast<const float4*>(s_bias + 16 * min(tile, nt - 1) + 4 * q);
      floatx4 acc = {0.f, 0.f, 0.f, 0.f};
      auto read = [&](int ks) { return *reinterpret_cast<const bf16x8*>(x + 64 * ks); };
      auto product = [&](int u, const bf16x8& xv) {
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wq[u]), xv, acc, 0, 0, 0);
      };
      int ks = 0;
      for (; ks + kAhead16 < k.nks; ks += kAhead16)
#pragma unroll
        for (int u = 0; u < kAhead16; ++u) {
          product(u, read(ks + u));
          wq[u] = gmi::load_uniform(k.w, min(ks + kAhead16 + u, k.nks - 1) * 2048, lane_off);
        }
      auto tail4 = [&](auto first) {
        constexpr int U = decltype(first)::value;
        bf16x8 xr[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) xr[u] = read(min(ks + U + u, k.nks - 1));
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (ks + U + u < k.nks) product(U + u, xr[u]);
      };
      tail4(std::integral_constant<int, 0>{});
      if (ks + 4 < k.nks) tail4(std::integral_constant<int, 4>{});
      const bool more = tile + 8 < nt;
      request16(wq, more ? walk16(w, K, F, tile + 8) : walk16(wn, Kn, Fn, wave), lane_off);
      const float v0 = acc[0] + b.x, v1 = acc[1] + b.y, v2 = acc[2] + b.z, v3 = acc[3] + b.w;
      if (tile >= nt) {
      } else if (!head) {
        *reinterpret_cast<uint2*>(y + 32 * tile) = make_uint2(pack_bf16(elu_f(v0), elu_f(v1)), pack_bf16(elu_f(v2), elu_f(v3)));
      } else {
        const int f = 16 * tile + 4 * q;
        float* d = s_head + n * ho + f;
        if (f + 0 < ho) d[0] = v0;
        if (f + 1 < ho) d[1] = v1;
        if (f + 2 < ho) d[2] = v2;
        if (f + 3 < ho) d[3] = v3;
      }
      tile += 8;
    } while (tile < nt);
    if (head && wave == 7) idle();
    __syncthreads();
    s_bias += F;
    w = wn; K = Kn; F = Fn;
  }
}

// 512 threads.
// WS: a WsShape whose widths the model has (weights held in registers for the whole launch): waves 0-3 run the policy net
// and waves 4-7 the value net at the same time (the two nets have the same hidden widths, so their layers finish together
// and share the barriers); every other phase uses all 8 waves.
// void: the policy net alone, on all 8 waves, its weights streamed from L2 at every step with the layer walk of the agent
// kernel (agent_kernel.h) or, 16 envs, the one above: the next item's blocks, across layers and steps, are on their way before
// the present one is left.  A compute unit draws weights at about 50 B/ns, which bounds the step of a wide net, so the value net
// -- which the simulator does not wait for -- is left to one launch over all slots afterwards (launch_values).
// R16: the 16-env form of the nets (rows_per_wg == 16).
// A step has three phases between barriers: the layers; sampling and stores; simulator, the next step's draws, sums.  The
// simulator writes the next state where the next step reads it (two buffers), so nothing is copied in between.
// Measured, us (the form with the simulator on the vector unit, 32-row products for 16 envs and a copy of the state): 4096 envs
// of 108:400:200:100:21, 32 steps 350 (470); 4096 envs of 60:256:128:64:8, 16 steps 107 (120); 1000 envs of 45:128:128:12, 24
// steps 126 (179).
template <int RT, class WS = void, bool R16 = false>
__global__ __launch_bounds__(512) void rollout_fused_kernel(RolloutArgs a) {
  constexpr int R = R16 ? 16 : RT * 32;              // rows of the products
  constexpr int NT = 512;
  constexpr bool kStationary = !std::is_void<WS>::value;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  const int O = a.obs_dim, A = a.act_dim, OA = O + A, OS = (OA + 3) & ~3, nbo = a.o4 >> 2, nba = (A + 3) >> 2;
  const int npr = nba + nbo + 1;                     // random blocks per env and step: action, env noise, done
  const int stride_x0 = a.obs_pad + 8, stride_h = a.max_h + 8;
  const int Rv = a.rows_per_wg;                      // envs owned by this workgroup: R
  float* s_in2 = reinterpret_cast<float*>(smem_raw);                                 // [2][Rv][OS] state | action
  uint16_t* s_x0 = reinterpret_cast<uint16_t*>(smem_raw + a.x0_off);                 // [R][obs_pad + 8]
  uint16_t* s_hid = reinterpret_cast<uint16_t*>(smem_raw + a.hid_off);               // [nets][2][R][stride_h]
  float* s_mu = reinterpret_cast<float*>(smem_raw + a.mu_off);                       // [R][A]
  float* s_val = reinterpret_cast<float*>(smem_raw + a.val_off);                     // [R]
  float* s_lp = reinterpret_cast<float*>(smem_raw + a.lp_off);                       // [Rv][nba]
  float* s_part = reinterpret_cast<float*>(smem_raw + a.part_off);                   // [Rv][nbo]
  int* s_done = reinterpret_cast<int*>(smem_raw + a.done_off);                       // [Rv]
  float* s_ls = reinterpret_cast<float*>(smem_raw + a.ls_off);                       // [A] log_std, [A] exp(log_std)
  float* s_bias = reinterpret_cast<float*>(smem_raw + a.bias_off);                   // policy biases, (stationary) value biases
  float* s_m = reinterpret_cast<float*>(smem_raw + a.m_off);                         // [o4][ms] when mr_lds
  uint16_t* s_wl = reinterpret_cast<uint16_t*>(smem_raw + a.w_off);                  // operand blocks of LDS-resident layers
  float4* s_draws = reinterpret_cast<float4*>(smem_raw + a.draw_off);                // [ahead + 1][Rv][npr]
  const int tid = threadIdx.x, lane = tid & 63;
  // wave-uniform values, so that the per-net kernel arguments are fetched by scalar loads
  const int half = __builtin_amdgcn_readfirstlane(tid >> 8), wave4 = __builtin_amdgcn_readfirstlane((tid >> 6) & 3);
  const int wave8 = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (int idx = tid; idx < R * (stride_x0 >> 3); idx += NT) reinterpret_cast<uint4*>(s_x0)[idx] = make_uint4(0u, 0u, 0u, 0u);
  for (int idx = tid; idx < Rv * OS; idx += NT) s_in2[Rv * OS + idx] = 0.f;
  for (int j = tid; j < A; j += NT) {
    const float ls = a.log_std[j];
    s_ls[j] = ls;
    s_ls[A + j] = expf(ls);
  }
  if constexpr (kStationary) {
    stage_biases(a.net[0], s_bias, tid, NT);
    stage_biases(a.net[1], s_bias + a.net[0].bias_total, tid, NT);
  }
  const int m4 = a.o4 * (a.ms >> 2);
  if (a.mr_lds == 2)
    for (int idx = tid; idx < m4; idx += NT) reinterpret_cast<float4*>(s_m)[idx] = reinterpret_cast<const float4*>(a.m_r)[idx];
  const FusedNet& N = a.net[half];
  uint16_t* s_a = s_hid + (size_t)half * 2 * R * stride_h;
  uint16_t* s_b = s_a + R * stride_h;
  float* s_head = half ? s_val : s_mu;
  const int head_stride = half ? 1 : A;
  const float* s_nb = s_bias + (half ? a.net[0].bias_total : 0);
  // this wave's weight operands, fetched once (a dummy single entry in the streaming form)
  bf16x8 wreg[WsFrags<WS>::value];
  const uint16_t* s_w = s_wl;
  if constexpr (kStationary) {
    if constexpr (R16) ws_load16<WS, 0>(wreg, N, wave4, lane);
    else ws_load<WS, 0>(wreg, N, wave4, lane);
    ws_stage<WS, 0>(s_wl, a.net[0], tid, NT);
    ws_stage<WS, 0>(s_wl + WS::lds_elems(), a.net[1], tid, NT);
    s_w = s_wl + (half ? WS::lds_elems() : 0);
  }

  // streaming form: the first weight blocks of this wave's first item are always on their way
  constexpr int kAhead = RT == 1 ? 8 : 4;
  gmi_agent::Ring<gmi_agent::Bf16, kAhead> wq;
  Ring16 wq16;
  if constexpr (!kStationary) {
    if constexpr (R16) {
      for (int f = tid; f < a.net[0].bias_total; f += NT) {      // the policy's biases, layer after layer
        int l = 0;
        while (l + 1 < a.net[0].n_layers && f >= a.net[0].bias_off[l + 1]) ++l;
        s_bias[f] = a.net[0].bias[l][f - a.net[0].bias_off[l]];
      }
      request16(wq16, walk16(a.policy[0].w, a.policy[0].K, a.policy[0].F, wave8),
                (((lane >> 5) * 64) + (lane & 15) + 32 * ((lane >> 4) & 1)) * 16);
    }
    else gmi_agent::request<gmi_agent::Bf16, RT, kAhead, RT, 8>(wq, a.policy[0], wave8, lane);
  }

  const SimLane sl = sim_lane(a, wave8, OS, lane);
  const int draw_top = draw_thread(a, npr);
  // The grid never exceeds what the instance's compute units hold at once: a workgroup takes the tiles
  // blockIdx.x, blockIdx.x + gridDim.x, ... one after the other, each through all T steps.  (Workgroups
  // that wait for a free compute unit would keep the dispatcher from placing other instances' kernels.)
  for (int tile = blockIdx.x; tile < a.n_tiles; tile += gridDim.x) {
    const int r0 = tile * Rv;
    load_states(a, r0, s_in2, OS, tid);
    // thread NT - 64 + e (e < Rv; the last wave, which has the fewest other items) carries env e's episode counter, makes its
    // done flag and writes its sums
    const int et = tid - (NT - 64);
    const bool env_thread = et >= 0 && et < Rv, env_ok = env_thread && r0 + et < a.n;
    uint32_t ep = 0;
    if (env_ok) ep = a.episode_step[r0 + et];
    if (a.ahead) draw_all(a, s_draws, a.step0, r0, npr, nba, tid);
    __syncthreads();
    // the nets' bf16 copy of the state; every later step's comes from the simulator
    {
      const int r = tid >> a.row_shift, c = tid & ((1 << a.row_shift) - 1), nc = 1 << a.row_shift;
      for (int k = c; k < O; k += nc) s_x0[r * stride_x0 + k] = (uint16_t)(pack_bf16(s_in2[r * OS + k], 0.f) & 0xFFFFu);
    }
    __syncthreads();

    int64_t slot0 = r0;
    auto reward = [&]() {      // of the step before
      if (env_ok) a.b_rew[slot0 - a.ld_envs + et] = -a.reward_scale * block_sum(s_part + et * nbo, nbo);
    };
    for (int t = 0; t <= a.T; ++t, slot0 += a.ld_envs) {
      float* s_in = s_in2 + (t & 1) * Rv * OS;
      float4* s_noise = s_draws + (a.ahead ? (t & 1) * Rv * npr : 0);
      const uint32_t step = a.step0 + (uint32_t)t;
      // beside the heads, whose tiles leave the last wave idle: the reward of the step before and, where the draws are there,
      // this step's done flags
      auto beside = [&]() {
        if (!env_thread) return;
        if (t > 0) reward();
        if (a.ahead && t < a.T) finish_env(a, r0, slot0, et, s_noise, npr, ep, s_done);
      };
      // both nets, layer by layer; after the last step only the value net (bootstrap value)
      if constexpr (kStationary) {
        const bool run = half == 1 || t < a.T;
        if constexpr (R16)
          ws_net16<WS, 0>(wreg, s_w, N, s_nb, s_x0, stride_x0, s_a, s_b, stride_h, s_head, head_stride, run, wave4, lane, beside);
        else
          ws_net<WS, 0, RT>(wreg, s_w, N, s_nb, s_x0, stride_x0, s_a, s_b, stride_h, s_head, head_stride, run, wave4, lane, beside);
      } else {
        if (t == a.T) {
          beside();
          break;
        }
        if constexpr (R16) {
          net_layers16(a.policy, a.net[0].n_layers, wq16, reinterpret_cast<const unsigned char*>(s_x0), reinterpret_cast<unsigned char*>(s_hid),
                       reinterpret_cast<unsigned char*>(s_hid + R * stride_h), s_bias, s_mu, A, wave8, lane, beside);
        } else {
          beside();
          gmi_agent::net_layers<gmi_agent::Bf16, RT, kAhead, RT, 8, true>(
              a.policy, a.net[0].n_layers, wq, reinterpret_cast<const unsigned char*>(s_x0), reinterpret_cast<unsigned char*>(s_hid),
              reinterpret_cast<unsigned char*>(s_hid + R * stride_h), nullptr, s_mu, A, wave8, lane);
        }
      }
      if (t == a.T) {
        if constexpr (kStationary)
          if (env_ok) a.last_value[r0 + et] = s_val[et];
        break;
      }
      if (!a.ahead) {
        draw_all(a, s_noise, step, r0, npr, nba, tid);
        __syncthreads();
        if (env_thread) finish_env(a, r0, slot0, et, s_noise, npr, ep, s_done);
      }
      sample_and_store(a, r0, slot0, s_in, OS, s_mu, A, s_noise, npr, nba, s_ls, s_lp, tid);
      __syncthreads();
      if (a.mr_lds == 1) {
        for (int idx = tid; idx < m4; idx += NT) reinterpret_cast<float4*>(s_m)[idx] = reinterpret_cast<const float4*>(a.m_r)[idx];
        __syncthreads();
      }
      float* s_nxt = s_in2 + ((t + 1) & 1) * Rv * OS;
      auto put = [&](int r, int o, const float (&v)[4]) {      // (what lies beyond the state belongs to the next step's actions)
        *reinterpret_cast<float4*>(s_nxt + r * OS + o) = make_float4(v[0], v[1], v[2], v[3]);
        const float w1 = o + 1 < O ? v[1] : 0.f, w2 = o + 2 < O ? v[2] : 0.f, w3 = o + 3 < O ? v[3] : 0.f;
        *reinterpret_cast<uint2*>(s_x0 + r * stride_x0 + o) = make_uint2(pack_bf16(v[0], w1), pack_bf16(w2, w3));
      };
      // an LDS pointer or a global pointer, kept apart: one that may be either makes every access a flat load
      if (a.mr_lds != 0) sim_items(a, r0, step, sl, s_in, OS, s_m, s_part, s_done, s_noise, npr, nba, wave8, lane, put);
      else sim_items(a, r0, step, sl, s_in, OS, a.m_r, s_part, s_done, s_noise, npr, nba, wave8, lane, put);
      if (env_ok) {
        a.b_logp[slot0 + et] = block_sum(s_lp + et * nba, nba);
        if constexpr (kStationary) a.b_val[slot0 + et] = s_val[et];
      }
      if (a.ahead && t + 1 < a.T) draw_rest(a, s_draws + ((t + 1) & 1) * Rv * npr, step + 1u, r0, npr, nba, tid, draw_top);
      __syncthreads();
    }
    // the final state
    {
      const float* s_in = s_in2 + (a.T & 1) * Rv * OS;
      const int r = tid >> a.row_shift, c = tid & ((1 << a.row_shift) - 1), nc = 1 << a.row_shift;
      if (r0 + r < a.n)
        for (int k = c; k < O; k += nc) a.obs_state[(int64_t)(r0 + r) * O + k] = s_in[r * OS + k];
    }
    if (env_ok) a.episode_step[r0 + et] = ep;
    __syncthreads();                                   // the next tile overwrites the state rows
  }
}

// floats of one net's LDS bias block (the two nets have the same padded widths except for the head,
// whose padded width is at least as large for the policy net)
size_t bias_floats(const gmi_model* m, int net) {
  size_t n = 0;
  for (int l = 0; l < m->L.n_layers; ++l) n += m->L.net[net][l].out_pad;
  return n;
}

void fill_net(const gmi_model* m, int net, FusedNet* N) {
  const ModelLayout& L = m->L;
  N->n_layers = L.n_layers;
  for (int l = 0; l < L.n_layers; ++l) {
    const LayerInfo& li = L.net[net][l];
    N->w[l] = reinterpret_cast<const uint16_t*>(m->shadow + li.sh_wf);
    N->bias[l] = reinterpret_cast<const float*>(m->shadow + li.sh_b);
    N->in_pad[l] = li.in_pad;
    N->out_pad[l] = li.out_pad;
    N->bias_off[l] = l ? N->bias_off[l - 1] + N->out_pad[l - 1] : 0;
  }
  N->bias_total = N->bias_off[L.n_layers - 1] + N->out_pad[L.n_layers - 1];
  N->out_store = L.net[net][L.n_layers - 1].out;
}

// LDS of the operand blocks that the weight-stationary form keeps there (both nets); 0 for other shapes.
size_t rollout_ws_lds_bytes(const ModelLayout& L) {
  if (ws_matches<WsAnt>(L)) return 2 * (size_t)WsAnt::lds_elems() * 2;
  if (ws_matches<WsSmallObs>(L)) return 2 * (size_t)WsSmallObs::lds_elems() * 2;
  return 0;
}

int max_hidden_pad(const ModelLayout& L) {
  int w = 32;
  for (int l = 0; l < L.n_hidden; ++l) w = std::max(w, L.net[0][l].out_pad);
  return w;
}

// What the first form of the streaming kernel, which held both nets' activations, took for a tile of R envs: decides the tile
// height and which models are refused.
size_t admission_bytes(const gmi_model* m, int R) {
  const ModelLayout& L = m->L;
  const int max_h = max_hidden_pad(L), O = L.obs_dim, A = L.act_dim, o4 = (O + 3) & ~3;
  const size_t hid = 4 * (size_t)R * (max_h + 8) * 2;
  const size_t used = (((size_t)R * o4 * 4 + 15) & ~(size_t)15) + (size_t)R * ((A + 3) / 4 + o4 / 4 + 1) * 16;
  const size_t region = ((hid > used ? hid : used) + 15) & ~(size_t)15;
  return (size_t)R * ((O + A + 3) & ~3) * 4 + (size_t)R * (gmi::pad32(O) + 8) * 2 + region +
         (size_t)(R * (A + 1 + (A + 3) / 4 + o4 / 4) + ((R + 3) & ~3)) * 4 + ((bias_floats(m, 0) + bias_floats(m, 1) + 3) & ~(size_t)3) * 4 +
         rollout_ws_lds_bytes(L);
}

// Lays out the LDS of a tile of Rv envs and returns its bytes.
size_t rollout_lds(const gmi_model* m, int Rv, int nets, int mr_lds, int ahead, RolloutArgs* a) {
  const ModelLayout& L = m->L;
  const int O = L.obs_dim, A = L.act_dim, o4 = (O + 3) & ~3, nba = (A + 3) / 4, nbo = o4 / 4;
  const size_t mr_bytes = (size_t)o4 * gmi::env_row_stride(O, A) * 4, draws = (size_t)Rv * (nba + nbo + 1) * 16;
  const size_t hid = 2 * nets * (size_t)Rv * (max_hidden_pad(L) + 8) * 2;
  size_t off = 2 * (size_t)Rv * ((O + A + 3) & ~3) * 4;
  auto take = [&](int* field, size_t bytes) { *field = (int)off; off = (off + bytes + 15) & ~(size_t)15; };
  take(&a->x0_off, (size_t)Rv * (gmi::pad32(O) + 8) * 2);
  // the hidden activations' space is idle outside the nets: a step's draws, where they are not made ahead, and the simulator's
  // matrix, where it is staged at every step, lie there too
  take(&a->hid_off, std::max(hid, (ahead ? 0 : draws) + (mr_lds == 1 ? mr_bytes : 0)));
  take(&a->mu_off, (size_t)Rv * A * 4);
  take(&a->val_off, nets == 2 ? (size_t)Rv * 4 : 0);
  take(&a->lp_off, (size_t)Rv * nba * 4);
  take(&a->part_off, (size_t)Rv * nbo * 4);
  take(&a->done_off, (size_t)Rv * 4);
  take(&a->ls_off, 2 * (size_t)A * 4);
  take(&a->bias_off, (bias_floats(m, 0) + (nets == 2 ? bias_floats(m, 1) : 0)) * 4);
  take(&a->w_off, rollout_ws_lds_bytes(L));
  take(&a->m_off, mr_lds == 2 ? mr_bytes : 0);
  if (mr_lds == 1) a->m_off = a->hid_off + (int)(ahead ? 0 : draws);
  take(&a->draw_off, ahead ? 2 * draws : 0);
  if (!ahead) a->draw_off = a->hid_off;
  a->mr_lds = mr_lds;
  a->ahead = ahead;
  return off;
}

}  // namespace

extern "C" int rollout_collect(gmi_t g, gmi_model_t m, gmi_env_t env, gmi_buffer_t b, float* obs, uint64_t seed,
                               uint32_t step0, uint32_t env_offset, float* last_value) {
  if (!valid(g)) GMI_FAIL(GMI_ERR_BAD_HANDLE, "rollout_collect: bad instance");
  if (!valid(m)) GMI_FAIL(GMI_ERR_BAD_HANDLE, "rollout_collect: bad model");
  if (!valid(env)) GMI_FAIL(GMI_ERR_BAD_HANDLE, "rollout_collect: bad env");
  if (!valid(b)) GMI_FAIL(GMI_ERR_BAD_HANDLE, "rollout_collect: bad buffer");
  const ModelLayout& L = m->L;
  const gmi_buffer_desc& bd = b->d;
  const int shape_rc = check_rollout("rollout_collect", m, env, b);
  if (shape_rc != GMI_OK) return shape_rc;
  if (bd.n_envs == 0 || bd.horizon == 0) return GMI_OK;
  if (!obs || !last_value) GMI_FAIL(GMI_ERR_INVALID_ARG, "rollout_collect: NULL pointer");
  if (L.dtype != GMI_DTYPE_BF16)
    GMI_FAIL(GMI_ERR_UNSUPPORTED, "rollout_collect: BF16 models only; use agent_act / env_step / collect_experience");
  // as for the fused agent kernel: every tile streams all weights from L2 at every step, which loses to the
  // per-layer large-tile kernels beyond ~1 MB of bf16 weights (measured on a [512,512,256,128] model with
  // 16384 envs and 16 steps: 4.1 ms in one launch against 3.3 ms step by step)
  if (L.weight_bytes > (1 << 20)) {
    // ... where the model has a forward-only kernel of its own, the stage is two launches per step instead
    const int rc = gmi::rollout_stepwise(g, m, env, b, obs, seed, step0, env_offset, last_value);
    if (rc != GMI_ERR_UNSUPPORTED) return rc;
  }
  if (L.weight_bytes > (1 << 20))
    GMI_FAIL(GMI_ERR_UNSUPPORTED, "rollout_collect: model too large for the one-launch kernel (%lld bytes of bf16 "
             "weights, limit %d); use agent_act / env_step / collect_experience", (long long)L.weight_bytes, 1 << 20);
  constexpr size_t kLdsMax = 160 * 1024;
  const int n = bd.n_envs;
  const int nets = ws_matches<WsAnt>(L) || ws_matches<WsSmallObs>(L) ? 2 : 1;      // the streaming form runs the policy alone
  // Height and refusal go by the bytes of both nets' activations, also for the streaming form, which holds one net's: what was
  // refused stays refused, and heights change with envs for all models at one line.  (With the streaming form's own bytes
  // 60:256:256:8 would take 64 envs: 364 us instead of 417 for 16384 envs and 16 steps, but 637 instead of 588 for 20000.)
  int R = 64;
  if (admission_bytes(m, R) > kLdsMax || (n + 63) / 64 < g->cu_count) R = 32;
  if (admission_bytes(m, R) > kLdsMax)
    GMI_FAIL(GMI_ERR_UNSUPPORTED, "rollout_collect: a 32-env tile of this model needs %zu bytes of LDS (limit %zu); "
             "use agent_act / env_step / collect_experience", admission_bytes(m, R), kLdsMax);
  RolloutArgs a;
  fill_net(m, 0, &a.net[0]);
  fill_net(m, 1, &a.net[1]);
  for (int l = 0; l < L.n_layers; ++l)
    a.policy[l] = {reinterpret_cast<const uint4*>(a.net[0].w[l]), a.net[0].bias[l], nullptr, L.net[0][l].in_pad, L.net[0][l].out_pad};
  a.log_std = reinterpret_cast<const float*>(m->shadow + L.sh_logstd);
  fill_rollout_env(m, env, b, obs, seed, step0, env_offset, last_value, &a);
  a.obs_pad = gmi::pad32(L.obs_dim);
  a.max_h = max_hidden_pad(L);
  // fewer 32-env tiles than compute units: 16 envs per workgroup use twice as many of them.  So do the models whose two rows of
  // state per env leave no room for more.
  int rows_per_wg = (R == 32 && (n + 31) / 32 < g->cu_count) ? 16 : R;
  while (rows_per_wg > 16 && rollout_lds(m, rows_per_wg, nets, 0, 0, &a) > kLdsMax) rows_per_wg >>= 1;
  // what else the LDS holds: the simulator's matrix for the whole launch, draws one step ahead, else the matrix step by step
  size_t lds = 0;
  {
    static const int order[][2] = {{2, 1}, {1, 1}, {2, 0}, {0, 1}, {1, 0}, {0, 0}};
    const size_t hid = 2 * nets * (size_t)rows_per_wg * (a.max_h + 8) * 2;
    for (const auto& o : order) {
      lds = rollout_lds(m, rows_per_wg, nets, o[0], o[1], &a);
      // staged at every step only into space that is there anyway
      if (lds <= kLdsMax && (o[0] != 1 || (size_t)a.m_off + (size_t)a.o4 * a.ms * 4 <= (size_t)a.hid_off + hid)) break;
    }
  }
  if (lds > kLdsMax)
    GMI_FAIL(GMI_ERR_UNSUPPORTED, "rollout_collect: a 16-env tile of this model needs %zu bytes of LDS (limit %zu)", lds, kLdsMax);
  set_rows(&a, rows_per_wg);
  // weight-stationary variant where this model's padded widths have one (both nets share them)
  typedef void (*rollout_fn)(RolloutArgs);
  rollout_fn kfn = rows_per_wg == 64 ? rollout_fused_kernel<2> : rollout_fused_kernel<1>;
  int variant = rows_per_wg == 64 ? 1 : 0;
  if (ws_matches<WsAnt>(L)) { kfn = rows_per_wg == 64 ? rollout_fused_kernel<2, WsAnt> : rollout_fused_kernel<1, WsAnt>; variant += 2; }
  else if (ws_matches<WsSmallObs>(L)) {
    kfn = rows_per_wg == 64 ? rollout_fused_kernel<2, WsSmallObs> : rollout_fused_kernel<1, WsSmallObs>;
    variant += 4;
  }
  // 16 envs per workgroup: the nets on 16-row products
  if (rows_per_wg == 16) {
    if (variant == 2) { kfn = rollout_fused_kernel<1, WsAnt, true>; variant = 6; }
    else if (variant == 4) { kfn = rollout_fused_kernel<1, WsSmallObs, true>; variant = 7; }
    else { kfn = rollout_fused_kernel<1, void, true>; variant = 8; }
  }
  static gmi::DeviceSet allowed[9];
  const int lds_rc = gmi::allow_lds((const void*)kfn, kLdsMax, g->device, &allowed[variant]);
  if (lds_rc != GMI_OK) return lds_rc;
  // no more workgroups than the instance's compute units hold at once; the rest of the tiles are taken
  // by the same workgroups in turn
  int64_t resident = 1;
  const int occ_rc = gmi::resident_groups(g, (const void*)kfn, 512, lds, &resident);
  if (occ_rc != GMI_OK) return occ_rc;
  const int grid = (int)(a.n_tiles < resident ? a.n_tiles : resident);
  {
    gmi::ProfScope ps(g, gmi::kClsFusedRollout);
    ps.launch(kfn, dim3(grid), dim3(512), lds, a);
    GMI_LAUNCH_CHECK();
  }
  // the simulator needs no values: the streaming form leaves them to one pass over all slots and the final states
  return nets == 2 ? GMI_OK : gmi::launch_values(g, m, bd.obs, bd.horizon, n, bd.ld_envs, bd.val, obs, last_value);
}
