// What the row-tile trainer kernel (tile_kernel.h) and its host side (chain.hip) share: the weight stream that it reads -- the bf16
// weights of one net as 1 KiB operand blocks in the order of its products -- its arguments, and the activation functions.
#pragma once
#include "internal.h"

namespace gmi_chain {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;
typedef float float2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
typedef int intx8 __attribute__((ext_vector_type(8)));

using gmi::elu_f;
// ELU'(z) from the stored output h = ELU(z) >= -1: 1 if h > 0 else h + 1, as one add with the [0, 1] clamp
__device__ __forceinline__ float elu_grad_f(float h) { return __builtin_amdgcn_fmed3f(h + 1.0f, 0.f, 1.f); }
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  float2v v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2v));
}
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

__device__ __forceinline__ uint32_t to_e4m3x4(float a, float b, float c, float d) {
  // the conversion rounds to nearest even; its inputs are kept within the format's range, so it never overflows
  a = __builtin_amdgcn_fmed3f(a, -448.f, 448.f); b = __builtin_amdgcn_fmed3f(b, -448.f, 448.f);
  c = __builtin_amdgcn_fmed3f(c, -448.f, 448.f); d = __builtin_amdgcn_fmed3f(d, -448.f, 448.f);
  int v = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, 0, false);
  v = __builtin_amdgcn_cvt_pk_fp8_f32(c, d, v, true);
  return (uint32_t)v;
}

// ---------------------------------------------------------------------------------------------------------
// ELU, then E4M3.  Its results are never below -1, so the upper bound of the format's range is the only one to keep, and one median of
// three is both ELU's maximum and that bound.
__device__ __forceinline__ uint32_t elu_e4m3x4(float a, float b, float c, float d) {
  float log2e, most;
  asm("s_mov_b32 %0, 0x3fb8aa3b" : "=s"(log2e));      // 1.44269504
  asm("s_mov_b32 %0, 0x43e00000" : "=s"(most));       // 448
  auto elu = [&](float z) {
    const float e = __builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(z * log2e), 0.f, 1.f) - 1.0f;
    float y;
    asm("v_med3_f32 %0, %1, %2, %3" : "=v"(y) : "v"(z), "v"(e), "s"(most));
    return y;
  };
  int v = __builtin_amdgcn_cvt_pk_fp8_f32(elu(a), elu(b), 0, false);
  v = __builtin_amdgcn_cvt_pk_fp8_f32(elu(c), elu(d), v, true);
  return (uint32_t)v;
}

// The plan: which 1 KiB weight blocks the row-tile kernel (tile_kernel.h) consumes in which order.  Pure functions of the padded layer
// widths d[0..nl] (d[0] = input, d[nl] = head), used at compile time by the kernel and at run time by the
// host when it describes the stream to the packing kernel.
//
// Segment s < nl is the forward product of layer s (K = d[s] in, F = d[s+1] out); segment s >= nl is the
// input-gradient product of layer l = 2 nl - 1 - s (K = d[l+1], F = d[l]), l = nl-1 .. 1.  A segment's F/32
// feature tiles are cut into groups of 4, then 2, then 1 tiles; a group's blocks are ordered k step major
// (block (ks, t) = tile t of the group, k step ks).
struct ChainDims {
  int nl;
  int d[GMI_MAX_HIDDEN + 2];
};
constexpr int kGroupTiles = 4;
__host__ __device__ constexpr int cd_nseg(const ChainDims& D) { return 2 * D.nl - 1; }
__host__ __device__ constexpr int cd_layer(const ChainDims& D, int s) { return s < D.nl ? s : 2 * D.nl - 1 - s; }
__host__ __device__ constexpr int cd_K(const ChainDims& D, int s) { return s < D.nl ? D.d[s] : D.d[cd_layer(D, s) + 1]; }
__host__ __device__ constexpr int cd_F(const ChainDims& D, int s) { return s < D.nl ? D.d[s + 1] : D.d[cd_layer(D, s)]; }
__host__ __device__ constexpr int cd_seg_blocks(const ChainDims& D, int s) { return (cd_F(D, s) / 32) * (cd_K(D, s) / 16); }
__host__ __device__ constexpr int cd_nblocks(const ChainDims& D) {
  int n = 0;
  for (int s = 0; s < cd_nseg(D); ++s) n += cd_seg_blocks(D, s);
  return n;
}
__host__ __device__ constexpr int cd_maxdim(const ChainDims& D) {
  int m = 0;
  for (int i = 0; i <= D.nl; ++i) m = D.d[i] > m ? D.d[i] : m;
  return m;
}

// ---------------------------------------------------------------------------------------------------------
struct ChainArgs {
  const char* wstream[2];                          // chain stream of the policy / value net
  const float* bias[2][GMI_MAX_HIDDEN + 1];        // fp32 [out_pad] per layer
  uint16_t* x0;                                    // [rows, d[0]] bf16: the minibatch's observations (x0_ready == 1)
  uint16_t* h[2][GMI_MAX_HIDDEN + 1];              // h[net][l], l = 1 .. nl-1: input of layer l
  uint16_t* dz[2][GMI_MAX_HIDDEN + 1];             // dz[net][l], l = 0 .. nl-1: gradient at layer l's output
  const float* log_std;
  // the experience buffer the minibatch is drawn from: sample idx[r] lives at slot
  // (idx[r] / n_envs) * ld_envs + idx[r] % n_envs of its time-major arrays
  const int32_t* idx;                              // [rows]
  const float *b_obs, *b_act, *b_logp, *b_adv, *b_ret;
  int n_envs, ld_envs, obs_dim;
  int x0_ready;                                    // 1: x0 already holds the gathered rows (observation rows that cannot
                                                   // be read as 16-byte pieces are gathered by gather_kernel beforehand);
                                                   // 2: the rows are gathered from x16; 3 (inference): rows of at least 4
                                                   // floats, in order, that start at any 4-byte address
  const uint16_t* x16;                             // bf16 copy of all observations, [sample index][d[0]] (x0_ready == 2)
  int rows, act_dim;
  int stream;                                      // host: TileShapeStream
  float clip, c_v;
  float* stat_part;                                // [tiles][kStatStride + act_dim]
  // inference (TileShapeFwd): workgroup row y works on net net0 + y; results of the heads
  int net0;
  float* mu_out;                                   // [rows, act_dim] policy means, or NULL
  float *act_out, *logp_out;                       // [rows, act_dim] sampled actions and [rows] their log-densities, or NULL
  uint32_t k0, k1, step, env_offset;               // of the draws
  // inference over several slots of rows: slot t < T reads b_obs + t obs_step and writes val_out + t val_step, slot T reads obs_last
  // and writes val_last; item = slot * slot_tiles + row tile
  int T, slot_tiles, items;
  int64_t obs_step, val_step;
  const float* obs_last;
  float* val_last;
  int wf_off[2][GMI_MAX_HIDDEN + 1];               // TileShapeNat, TileShapeFp8: bytes from wstream to a layer's weights
  const float* scale;                              // TileShapeFp8: [2 nl]
  float* val_out;                                  // [rows] values
  uint16_t* x0b;                                   // the minibatch's observations as the first layer's operand blocks, written here for
                                                   // the weight-gradient kernel (by the policy net's workgroups)
  double reread;                                   // host: bytes of hidden activations that the backward pass reads again from memory
                                                   // unless they stay in LDS (TileShapeKeep)
};

}  // namespace gmi_chain
