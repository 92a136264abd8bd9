// Device-side counter-based random numbers: Philox4x32-10 (Salmon et al., SC'11) and the
// bit-reproducible Box-Muller map used for all Gaussian draws of the hot path.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gmi {

enum : uint32_t { kStreamAction = 0, kStreamEnv = 1, kStreamDone = 2, kStreamReset = 3, kStreamShuffle = 4 };

struct Words4 { uint32_t w[4]; };

// a ^ b ^ c as one instruction (the compiler makes two).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) { return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96); }

// counter = (c0,c1,c2,c3), key = (k0,k1); ten rounds, key advanced by the Weyl constants.
__device__ __forceinline__ Words4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                                uint32_t k0, uint32_t k1) {
  constexpr uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    // one 32 x 32 -> 64 bit multiply per product (integer multiplies run at a quarter of the vector rate, and the
    // separate high / low forms take one such instruction each)
    const uint64_t p0 = (uint64_t)M0 * c0, p1 = (uint64_t)M1 * c2;
    const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0;
    const uint32_t hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
    const uint32_t n0 = xor3(hi1, c1, k0);
    const uint32_t n2 = xor3(hi0, c3, k1);
    c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  Words4 o;
  o.w[0] = c0; o.w[1] = c1; o.w[2] = c2; o.w[3] = c3;
  return o;
}

// num / den, correctly rounded, y within an ulp of 1 / den: a Newton-Raphson step for the reciprocal, then two corrections of the quotient
// by its exact residual (Markstein's division; a den of all ones, of j = 8388607, is the theorem's exception: there y has to be the nearest one,
// which the unit gives).  No scaling: these operands -- 0 or at least 2^-24 over a number between 1.7 and 2.5 -- never need it.
__host__ __device__ __forceinline__ float quotient_from(float y, float num, float den) {
#pragma clang fp contract(off)
  y = fmaf(fmaf(-den, y, 1.0f), y, y);
  float t = num * y;
  t = fmaf(fmaf(-den, t, num), y, t);
  return fmaf(fmaf(-den, t, num), y, t);
}
// sqrt(x), correctly rounded, r0 within an ulp of it: the product of two neighbours lies beside the square of the number half way between
// them by less than x's own spacing, so the sign of x - (neighbour) * r0, formed without rounding, says on which side of it the root is
// (Tuckerman's test).  x is between 1e-7 and 34: no scaling.
__host__ __device__ __forceinline__ float root_from(float r0, float x) {
  const uint32_t bits = __builtin_bit_cast(uint32_t, r0);
  const float down = __builtin_bit_cast(float, bits - 1u), up = __builtin_bit_cast(float, bits + 1u);
  const float r = fmaf(-down, r0, x) <= 0.0f ? down : r0;
  return fmaf(-up, r0, x) > 0.0f ? up : r;
}

// Two words -> two standard normals.  Every floating-point step is one correctly rounded
// add / multiply / divide / sqrt in the order written: contraction into FMA is switched off so that
// a CPU implementation of the same recipe reproduces the bits.
//   u1 = (2 (wa >> 9) + 1) / 2^24 written as m * 2^e, m folded to [sqrt(1/2), sqrt(2));
//   ln m = 2 atanh((m-1)/(m+1)), 6-term series; ln u1 = (e-24) ln2 + ln m, ln2 in two words;
//   r = sqrt(-2 ln u1);  quadrant = wb >> 30; x = (pi/2) (2 ((wb>>7) & 0x7FFFFF) + 1) / 2^24;
//   sin x / cos x by Taylor polynomials of degree 13 / 14, rotated by the quadrant.
// Draws are bound by their instructions (env_step, the collections): without the scaling of the general divide and square root, with
// the quadrant by sign bits and the generator's xors three at a time a block of four takes 226 vector instructions and 31 scalar ones
// instead of 268 and 60.  Quotient and root are correctly rounded for every radius, whichever estimates the units give within the ulp that
// they are specified to (the host checks go through all of them).  Collections in which the draws are part of the chain, us: 8:32:32:2 (64 envs, 16
// steps) 67 -> 64, 108:400:200:100:21 (4096 envs, 32 steps) 388 -> 355.
__device__ __forceinline__ void normal_pair(uint32_t wa, uint32_t wb, float& z0, float& z1) {
#pragma clang fp contract(off)
  const uint32_t j = ((wa >> 9) << 1) | 1u;
  const float fj = (float)j;
  const uint32_t bits = __float_as_uint(fj);
  int e = (int)(bits >> 23) - 127;
  float m = __uint_as_float((bits & 0x7FFFFFu) | 0x3F800000u);
  if (m > 0x1.6a09e6p+0f) { m = m * 0.5f; e += 1; }
  const float num = m - 1.0f, den = m + 1.0f;
  const float t = quotient_from(__builtin_amdgcn_rcpf(den), num, den);
  const float t2 = t * t;
  float p = 0x1.745d18p-4f;
  p = p * t2 + 0x1.c71c72p-4f;
  p = p * t2 + 0x1.24924ap-3f;
  p = p * t2 + 0x1.99999ap-3f;
  p = p * t2 + 0x1.555556p-2f;
  p = p * t2 + 1.0f;
  const float q = t * p;
  const float lnm = q + q;
  const float k = (float)(e - 24);
  const float lnu = k * 0x1.62e4p-1f + (k * 0x1.7f7d1cp-20f + lnm);
  const float x2l = lnu * -2.0f;
  const float r = root_from(__builtin_amdgcn_sqrtf(x2l), x2l);

  const uint32_t jf = (((wb >> 7) & 0x7FFFFFu) << 1) | 1u;
  const float f = (float)jf * 0x1p-24f;
  const float x = f * 0x1.921fb6p+0f;
  const float x2 = x * x;
  float ps = 0x1.612462p-33f;
  ps = ps * x2 + -0x1.ae6456p-26f;
  ps = ps * x2 + 0x1.71de3ap-19f;
  ps = ps * x2 + -0x1.a01a02p-13f;
  ps = ps * x2 + 0x1.111112p-7f;
  ps = ps * x2 + -0x1.555556p-3f;
  const float s = x * (ps * x2 + 1.0f);
  float pc = -0x1.93974ap-37f;
  pc = pc * x2 + 0x1.1eed8ep-29f;
  pc = pc * x2 + -0x1.27e4fcp-22f;
  pc = pc * x2 + 0x1.a01a02p-16f;
  pc = pc * x2 + -0x1.6c16c2p-10f;
  pc = pc * x2 + 0x1.555556p-5f;
  pc = pc * x2 + -0x1p-1f;
  const float c = pc * x2 + 1.0f;
  // quadrant 0: (c, s), 1: (-s, c), 2: (-c, -s), 3: (s, -c)
  const bool odd = (wb & 0x40000000u) != 0u;
  const float ct = __uint_as_float(__float_as_uint(odd ? s : c) ^ ((wb + 0x40000000u) & 0x80000000u));
  const float st = __uint_as_float(__float_as_uint(odd ? c : s) ^ (wb & 0x80000000u));
  z0 = r * ct;
  z1 = r * st;
}

// Four normals of one block: elements 4*block .. 4*block+3 of env `env` at (stream, step).
__device__ __forceinline__ void normal_block(uint32_t env, uint32_t step, uint32_t stream,
                                             uint32_t block, uint32_t k0, uint32_t k1, float z[4]) {
  const Words4 w = philox4x32_10(env, step, stream, block, k0, k1);
  normal_pair(w.w[0], w.w[1], z[0], z[1]);
  normal_pair(w.w[2], w.w[3], z[2], z[3]);
}

// Alternating unbalanced Feistel network on `bits` bits with cycle walking: a bijection of [0,n).
// Round function = word 0 of Philox(counter = (R, iteration, 4, epoch*256 + round)).
__device__ __forceinline__ uint32_t feistel_perm(uint32_t i, uint32_t n, int bits, uint32_t iteration,
                                                 uint32_t epoch, uint32_t k0, uint32_t k1) {
  if (n <= 1) return 0;
  uint32_t y = i;
  do {
    int wl = bits / 2, wr = bits - bits / 2;
#pragma unroll 1
    for (int r = 0; r < 6; ++r) {
      const uint32_t left = y >> wr;
      const uint32_t right = y & ((1u << wr) - 1u);
      const Words4 f = philox4x32_10(right, iteration, kStreamShuffle, (epoch << 8) + (uint32_t)r, k0, k1);
      y = (right << wl) | (left ^ (f.w[0] & ((1u << wl) - 1u)));
      const int tmp = wl; wl = wr; wr = tmp;
    }
  } while (y >= n);
  return y;
}

// A block's part of a step's cost: the sum of squares of its state elements plus 0.01 times that of its actions, two roundings
// wherever it is computed.
__device__ __forceinline__ float reward_part(float ps, float pa) {
#pragma clang fp contract(off)
  return ps + 0.01f * pa;
}

}  // namespace gmi
