// Linear layers of the policy / value MLPs: forward, input-gradient and weight-gradient products.
//
// BF16 path: v_mfma_f32_32x32x16_bf16 (bf16 operands, fp32 accumulate).  A wavefront of 64 lanes
// feeds the matrix core with 8 consecutive contraction elements per lane for both operands, so both
// operands are staged in LDS with the contraction index contiguous; the weight-gradient product
// contracts over samples, whose index is strided in memory, and reads its operands through the transposing LDS
// read.  F32 path: plain FMA loops (gmi_set_fusion 0, and models whose rows do not fit the fp32 kernels' LDS tiles).
#include <algorithm>

#include "internal.h"

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;

constexpr int kBK = 64;          // contraction elements staged per step
constexpr int kLds = kBK + 8;    // LDS row stride in bf16 elements (144 B: conflict-free 16 B reads)

typedef float float2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));

using gmi::elu_f;
// ELU'(z) from the stored output h = ELU(z) >= -1: 1 if h > 0 else h + 1, as one add with the [0, 1] clamp
__device__ __forceinline__ float elu_grad_f(float h) { return __builtin_amdgcn_fmed3f(h + 1.0f, 0.f, 1.f); }
__device__ __forceinline__ float bf16_to_f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
// two fp32 -> packed bf16 pair, round to nearest even (one v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  float2v v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2v));
}

// ------------------------------------------------------------------------------------------------
// y[r, f] = epi(sum_k x[r,k] w[f,k]).  Matrix-core rows = features (weights), columns = samples, so a
// lane ends up with 4 consecutive features of one sample per accumulator quad.
// Workgroup = 4 waves arranged WF x WR; a wave computes TFM x TRM tiles of 32 x 32.
template <int WF, int WR, int TFM, int TRM, int EPI>
__global__ __launch_bounds__(256) void linear_bf16_kernel(gmi::LinearBatch batch, int rows) {
  constexpr int TF = WF * TFM * 32, TR = WR * TRM * 32;
  constexpr int CH_W = TF * (kBK / 8), CH_X = TR * (kBK / 8);      // 16-byte chunks per stage
  constexpr int NCH = (CH_W + CH_X + 255) / 256;
  __shared__ __attribute__((aligned(16))) uint16_t s_w[TF * kLds];
  __shared__ __attribute__((aligned(16))) uint16_t s_x[TR * kLds];

  const gmi::LinearProblem& P = batch.p[blockIdx.z];
  const int f0 = blockIdx.y * TF;
  if (f0 >= P.F) return;
  const int r0 = blockIdx.x * TR;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wf = wave / WR, wr = wave % WR;
  const uint16_t* __restrict__ gw = (const uint16_t*)P.w;
  const uint16_t* __restrict__ gx = (const uint16_t*)P.x;

  floatx16 acc[TFM][TRM];
#pragma unroll
  for (int i = 0; i < TFM; ++i)
#pragma unroll
    for (int j = 0; j < TRM; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  uint4 stage[NCH];
  auto load_stage = [&](int k0) {
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int ch = tid + c * 256;
      uint4 v = make_uint4(0, 0, 0, 0);
      if (ch < CH_W) {
        const int row = ch >> 3, kc = ch & 7;
        const int f = f0 + row, k = k0 + kc * 8;
        if (f < P.F && k < P.K) v = *reinterpret_cast<const uint4*>(gw + (int64_t)f * P.ldw + k);
      } else if (ch < CH_W + CH_X) {
        const int c2 = ch - CH_W;
        const int row = c2 >> 3, kc = c2 & 7;
        const int r = r0 + row, k = k0 + kc * 8;
        if (r < rows && k < P.K) v = *reinterpret_cast<const uint4*>(gx + (int64_t)r * P.ldx + k);
      }
      stage[c] = v;
    }
  };
  auto store_stage = [&]() {
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int ch = tid + c * 256;
      if (ch < CH_W) {
        const int row = ch >> 3, kc = ch & 7;
        *reinterpret_cast<uint4*>(&s_w[row * kLds + kc * 8]) = stage[c];
      } else if (ch < CH_W + CH_X) {
        const int c2 = ch - CH_W;
        const int row = c2 >> 3, kc = c2 & 7;
        *reinterpret_cast<uint4*>(&s_x[row * kLds + kc * 8]) = stage[c];
      }
    }
  };

  const int nk = (P.K + kBK - 1) / kBK;
  load_stage(0);
  for (int kt = 0; kt < nk; ++kt) {
    store_stage();
    __syncthreads();
    if (kt + 1 < nk) load_stage((kt + 1) * kBK);
#pragma unroll
    for (int kk = 0; kk < kBK / 16; ++kk) {
      bf16x8 a[TFM], b[TRM];
      const int ko = kk * 16 + (lane >> 5) * 8;
#pragma unroll
      for (int i = 0; i < TFM; ++i)
        a[i] = *reinterpret_cast<const bf16x8*>(&s_w[((wf * TFM + i) * 32 + (lane & 31)) * kLds + ko]);
#pragma unroll
      for (int j = 0; j < TRM; ++j)
        b[j] = *reinterpret_cast<const bf16x8*>(&s_x[((wr * TRM + j) * 32 + (lane & 31)) * kLds + ko]);
#pragma unroll
      for (int i = 0; i < TFM; ++i)
#pragma unroll
        for (int j = 0; j < TRM; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    __syncthreads();
  }

  // epilogue: accumulator v of lane l holds feature 8*(v/4) + 4*(l/32) + v%4, sample l%32 of the tile
#pragma unroll
  for (int i = 0; i < TFM; ++i) {
    const int fb = f0 + (wf * TFM + i) * 32;
    if (fb >= P.F) continue;
#pragma unroll
    for (int j = 0; j < TRM; ++j) {
      const int r = r0 + (wr * TRM + j) * 32 + (lane & 31);
      if (r >= rows) continue;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int f = fb + q * 8 + (lane >> 5) * 4;
        float o[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) o[t] = acc[i][j][q * 4 + t];
        if (EPI == gmi::kEpiBiasElu) {
          const float4 bv = *reinterpret_cast<const float4*>(P.bias + f);
          o[0] = elu_f(o[0] + bv.x); o[1] = elu_f(o[1] + bv.y);
          o[2] = elu_f(o[2] + bv.z); o[3] = elu_f(o[3] + bv.w);
          uint2 pk = make_uint2(pack_bf16(o[0], o[1]), pack_bf16(o[2], o[3]));
          *reinterpret_cast<uint2*>((uint16_t*)P.y + (int64_t)r * P.ldy + f) = pk;
        } else if (EPI == gmi::kEpiBiasHead) {
          float* y = (float*)P.y + (int64_t)r * P.ldy;
#pragma unroll
          for (int t = 0; t < 4; ++t)
            if (f + t < P.F_store) y[f + t] = o[t] + P.bias[f + t];
        } else {
          const uint2 hv = *reinterpret_cast<const uint2*>((const uint16_t*)P.h + (int64_t)r * P.ldh + f);
          const float h0 = bf16_to_f((uint16_t)(hv.x & 0xFFFF)), h1 = bf16_to_f((uint16_t)(hv.x >> 16));
          const float h2 = bf16_to_f((uint16_t)(hv.y & 0xFFFF)), h3 = bf16_to_f((uint16_t)(hv.y >> 16));
          o[0] *= elu_grad_f(h0); o[1] *= elu_grad_f(h1);
          o[2] *= elu_grad_f(h2); o[3] *= elu_grad_f(h3);
          uint2 pk = make_uint2(pack_bf16(o[0], o[1]), pack_bf16(o[2], o[3]));
          *reinterpret_cast<uint2*>((uint16_t*)P.y + (int64_t)r * P.ldy + f) = pk;
        }
      }
    }
  }
}

// ------------------------------------------------------------------------------------------------
// Large-tile variant for wide layers: workgroup tile (WRN*TRW*32 rows) x (2*TFW*32 features), 2 x WRN
// waves, each wave TFW x TRW matrix-core tiles, so one 16-byte LDS fragment feeds TRW (or TFW) MFMAs and
// LDS bandwidth stays below the matrix cores' appetite.  The launcher uses 2 x 4 waves of 4 x 2 (or 2 x 2)
// tiles: two waves per SIMD cover each other's LDS and epilogue latencies, which measured 8-17 % faster
// than 2 x 2 waves of 4 x 4 tiles on the same 256 x 256 workgroup tile (the epilogue alone - ELU on 256
// values per lane - took a third of a workgroup's time with one wave per SIMD).
// K is staged 64 at a time (a full 128-byte line per
// row) into double-buffered LDS (144-byte row stride: conflict-free 16-byte reads), one barrier per
// stage.  Two further stages are in flight in registers: the row operand is first-touch data from
// HBM / the memory-side cache, and with one workgroup per CU only a deep prefetch covers that latency
// (measured: with a single stage in flight the kernel ran at the pace of one memory round trip per stage).
// The accumulators leave through LDS so that the epilogue runs and stores with features contiguous across
// lanes (whole 64..256-byte row segments per store).  Workgroup ids are decoded so that the workgroups
// sharing a row tile run back to back on the same accelerator die (ids are dealt round-robin over the 8
// dies), which keeps that tile in the die's L2.
template <int TFW, int TRW, int EPI, int WRN>
__global__ __launch_bounds__(128 * WRN) void linear_bf16_big_kernel(gmi::LinearBatch batch, int rows, int n_rt,
                                                                    int n_rt_pad, int n_ft) {
  constexpr int NT = 128 * WRN;                                  // 2 x WRN waves
  constexpr int TF = 2 * TFW * 32, TR = WRN * TRW * 32;
  constexpr int CH_W = TF * (kBK / 8), CH_X = TR * (kBK / 8);
  constexpr int NCH = (CH_W + CH_X) / NT;
  constexpr int RPP = NT / 8;                                    // rows staged per pass of the workgroup
  static_assert((CH_W + CH_X) % NT == 0 && CH_W % NT == 0, "stage must divide evenly over the threads");
  constexpr int kStageElems = (TF + TR) * kLds;                  // bf16 elements of one LDS stage
  constexpr int kOutStride = TFW * 32 + 4;                       // floats per staged output row
  constexpr int kMainBytes = 2 * kStageElems * 2;
  constexpr int kOutBytes = 2 * WRN * 32 * kOutStride * 4;
  constexpr int kSmemBytes = kMainBytes > kOutBytes ? kMainBytes : kOutBytes;
  __shared__ __attribute__((aligned(16))) unsigned char smem[kSmemBytes];
  uint16_t* s_stage = reinterpret_cast<uint16_t*>(smem);

  // workgroup id -> (net, feature tile, row tile)
  const int per_net = n_rt_pad * n_ft;
  const int z = blockIdx.x / per_net;
  const int w = blockIdx.x % per_net;
  const int die = w & 7, slot = w >> 3;
  const int ft = slot % n_ft;
  const int rt = (slot / n_ft) * 8 + die;
  if (rt >= n_rt) return;
  const gmi::LinearProblem& P = batch.p[z];
  const int f0 = ft * TF, r0 = rt * TR;
  if (f0 >= P.F) return;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wf = wave / WRN, wr = wave % WRN;
  const uint16_t* __restrict__ gw = (const uint16_t*)P.w;
  const uint16_t* __restrict__ gx = (const uint16_t*)P.x;

  floatx16 acc[TFW][TRW];
#pragma unroll
  for (int i = 0; i < TFW; ++i)
#pragma unroll
    for (int j = 0; j < TRW; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // chunk = 8 consecutive k of one row; thread t handles rows (t >> 3) + 32 c, k-chunk t & 7.
  // Loads are unconditional (no branches, so the compiler can keep two stages in flight and wait only for
  // the older one): row indices are clamped into the operand (rows past the end only feed outputs that
  // are never stored) and the k offset is clamped into the row, with a select to zero past K.
  constexpr int NCW = CH_W / NT, NCX = CH_X / NT;
  const int crow = tid >> 3, kc8 = (tid & 7) * 8;
  const uint16_t* src_w[NCW];
  const uint16_t* src_x[NCX];
#pragma unroll
  for (int c = 0; c < NCW; ++c) src_w[c] = gw + (int64_t)min(f0 + crow + RPP * c, P.F - 1) * P.ldw;
#pragma unroll
  for (int c = 0; c < NCX; ++c) src_x[c] = gx + (int64_t)min(r0 + crow + RPP * c, rows - 1) * P.ldx;
  const int dst0 = crow * kLds + kc8;
  const int k_last = P.K - 8;
  uint4 st0[NCH], st1[NCH];
  auto load_stage = [&](uint4* st, int k0) {
    const int k = k0 + kc8;
    const bool k_ok = k < P.K;
    const int kq = min(k, k_last);
#pragma unroll
    for (int c = 0; c < NCW; ++c) {
      const uint4 v = *reinterpret_cast<const uint4*>(src_w[c] + kq);
      st[c] = k_ok ? v : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int c = 0; c < NCX; ++c) st[NCW + c] = *reinterpret_cast<const uint4*>(src_x[c] + kq);
  };
  auto store_stage = [&](const uint4* st, int buf) {
    uint16_t* base = s_stage + buf * kStageElems + dst0;
#pragma unroll
    for (int c = 0; c < NCW; ++c) *reinterpret_cast<uint4*>(base + c * RPP * kLds) = st[c];
#pragma unroll
    for (int c = 0; c < NCX; ++c) *reinterpret_cast<uint4*>(base + (TF + c * RPP) * kLds) = st[NCW + c];
  };
  auto compute = [&](int buf) {
    const uint16_t* sw = s_stage + buf * kStageElems;
    const uint16_t* sx = sw + TF * kLds;
#pragma unroll 2
    for (int kk = 0; kk < kBK / 16; ++kk) {
      bf16x8 a[TFW], b[TRW];
      const int ko = kk * 16 + (lane >> 5) * 8;
#pragma unroll
      for (int i = 0; i < TFW; ++i)
        a[i] = *reinterpret_cast<const bf16x8*>(&sw[((wf * TFW + i) * 32 + (lane & 31)) * kLds + ko]);
#pragma unroll
      for (int j = 0; j < TRW; ++j)
        b[j] = *reinterpret_cast<const bf16x8*>(&sx[((wr * TRW + j) * 32 + (lane & 31)) * kLds + ko]);
#pragma unroll
      for (int i = 0; i < TFW; ++i)
#pragma unroll
        for (int j = 0; j < TRW; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
  };

  // stage s lives in LDS buffer s & 1; st1 carries odd stages, st0 even stages.  Stages past K load as
  // zeros (weight operand), so the loop body needs no conditions: a trailing odd stage multiplies by zero.
  const int nk = (P.K + kBK - 1) / kBK;
  load_stage(st0, 0);
  load_stage(st1, kBK);
  store_stage(st0, 0);
  load_stage(st0, 2 * kBK);
  for (int kt = 0; kt < nk; kt += 2) {
    __syncthreads();
    store_stage(st1, 1);
    load_stage(st1, (kt + 3) * kBK);
    compute(0);
    __syncthreads();
    store_stage(st0, 0);
    load_stage(st0, (kt + 4) * kBK);
    compute(1);
  }
  __syncthreads();   // every wave is done reading the stages: LDS becomes the output staging area

  // Each wave owns a [32 rows][TFW*32 features] fp32 staging region and drains one row tile at a time.
  // Everything below is branch-free up to the final predicated store, and the problem's fields live in
  // registers: a conditional block per row made the compiler wait for every earlier store to be
  // acknowledged before each LDS read, which serialised the whole epilogue on memory round trips.
  float* s_out = reinterpret_cast<float*>(smem) + wave * 32 * kOutStride;
  constexpr int kLanesPerRow = TFW * 8;             // lanes covering one row with 4 features each
  constexpr int kRowsPerIter = 64 / kLanesPerRow;
  constexpr int NIT = 32 / kRowsPerIter;
  const int fl = (lane % kLanesPerRow) * 4;         // feature offset inside the wave's feature range
  const int f = f0 + wf * TFW * 32 + fl;
  const bool f_ok = f < P.F;
  const int fq = f_ok ? f : 0;
  uint16_t* __restrict__ yp = (uint16_t*)P.y + fq;
  const uint16_t* __restrict__ hp = (const uint16_t*)P.h + fq;
  const int ldy = P.ldy, ldh = P.ldh;
  float4 bias4 = make_float4(0.f, 0.f, 0.f, 0.f);
  if (EPI == gmi::kEpiBiasElu) bias4 = *reinterpret_cast<const float4*>(P.bias + fq);
  const int rl0 = lane / kLanesPerRow;
#pragma unroll
  for (int j = 0; j < TRW; ++j) {
    const int rbase = r0 + (wr * TRW + j) * 32 + rl0;
    uint2 hv[NIT];
    if (EPI == gmi::kEpiEluGrad) {
#pragma unroll
      for (int it = 0; it < NIT; ++it)
        hv[it] = *reinterpret_cast<const uint2*>(hp + (int64_t)min(rbase + it * kRowsPerIter, rows - 1) * ldh);
    }
#pragma unroll
    for (int i = 0; i < TFW; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float4 v4 = make_float4(acc[i][j][q * 4 + 0], acc[i][j][q * 4 + 1], acc[i][j][q * 4 + 2], acc[i][j][q * 4 + 3]);
        *reinterpret_cast<float4*>(&s_out[(lane & 31) * kOutStride + i * 32 + q * 8 + (lane >> 5) * 4]) = v4;
      }
    __builtin_amdgcn_wave_barrier();     // wave-private region: LDS serves one wave's requests in order
    float4 o[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it)
      o[it] = *reinterpret_cast<const float4*>(&s_out[(it * kRowsPerIter + rl0) * kOutStride + fl]);
    __builtin_amdgcn_wave_barrier();
    // Make every pending global load (bias, h rows) land here, once per pass: otherwise each predicated
    // store block below starts with a wait for *all* outstanding memory operations, earlier stores included.
    if (EPI == gmi::kEpiBiasElu) {
      asm volatile("" : "+v"(bias4.x), "+v"(bias4.y), "+v"(bias4.z), "+v"(bias4.w));
    } else {
#pragma unroll
      for (int it = 0; it < NIT; ++it) asm volatile("" : "+v"(hv[it].x), "+v"(hv[it].y));
    }
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      float4 v = o[it];
      if (EPI == gmi::kEpiBiasElu) {
        v.x = elu_f(v.x + bias4.x); v.y = elu_f(v.y + bias4.y); v.z = elu_f(v.z + bias4.z); v.w = elu_f(v.w + bias4.w);
      } else {
        const float h0 = bf16_to_f((uint16_t)(hv[it].x & 0xFFFF)), h1 = bf16_to_f((uint16_t)(hv[it].x >> 16));
        const float h2 = bf16_to_f((uint16_t)(hv[it].y & 0xFFFF)), h3 = bf16_to_f((uint16_t)(hv[it].y >> 16));
        v.x *= elu_grad_f(h0); v.y *= elu_grad_f(h1);
        v.z *= elu_grad_f(h2); v.w *= elu_grad_f(h3);
      }
      const uint2 pk = make_uint2(pack_bf16(v.x, v.y), pack_bf16(v.z, v.w));
      const int r = rbase + it * kRowsPerIter;
      if (r < rows && f_ok) *reinterpret_cast<uint2*>(yp + (int64_t)r * ldy) = pk;
    }
  }
}

// ------------------------------------------------------------------------------------------------
// Weight gradient: D[o, i] = sum_r dz[r, o] x[r, i].  Tile 256 (o) x 256 (i), 8 waves of 4 x 2 matrix-core tiles; the
// contraction runs over the rows of one split, 32 rows per stage.  Both operands go from memory straight into LDS (16
// bytes per lane, no registers in between) as they lie there, through a ring of five stages: up to four (128 KiB) are in
// flight while one is multiplied.  The contraction index is the strided one; the transposing LDS read (per 16 lanes: 4 rows x 16
// features) delivers operands.  Bias gradients are row sums of the first operand (two-element dot products with ones).
//
// Bound: HBM / L2 traffic.  A tile reads 1 KiB per row; with 128 x 128 tiles (through registers, transposed there) the
// same features were fetched by twice as many workgroups, whose second and third rounds found them evicted: 616 MB per
// 32768-row minibatch of 211:512:512:256:128:20 for 403 MB of operands.  All workgroups now run in one round with at most
// one per compute unit, and half as many splits are enough (their partials are another 6 MB each, written here and read
// by Adam): 467 MB fetched, 52 written.  Every layer has its own number of splits and a matrix's tiles are of equal size (plan_wgrad);
// between two barriers there is one wait and no switch, and the bias sums are shared out among the waves.  us, with the same splits for
// all layers / split per layer / as it is: 32768 rows of 60:256:128:64:8 29.9 / 26.7 / 24.4, of 108:400:200:100:21 56.9 / 51.1 / 42.9, of
// 211:512:512:256:128:20 109 / 108 / 91.5.  Without its loads the last takes 57, without its products and reads of LDS 50.
constexpr int kWgradT = 256;                            // features per operand and tile
constexpr int kWgradRows = 32;                          // rows per stage
constexpr int kWgradOperand = kWgradT * kWgradRows * 2; // bytes
constexpr int kWgradStage = 2 * kWgradOperand;
constexpr int kWgradRing = 5;
constexpr int kWgradLds = kWgradRing * kWgradStage;
constexpr int64_t kCacheBytes = (int64_t)216 << 20;      // beyond_cache
constexpr int kWgradGroups = 256, kSplitMin = 4, kSplitMax = 64, kWgradNarrow = 224;      // plan_wgrad
__device__ const uint4 g_zero_piece = {0, 0, 0, 0};     // what rows past the end load

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) s16x4* lds_s16x4;

// 16 bytes per lane from base + off to LDS bytes [lds, lds + 1024) in lane order.  Inline assembly: the compiler would
// wait for every such load in flight before any LDS read.  m0 (the LDS address) is a register that the compiler never
// allocates, and says so of a clobber; it does write m0 for instructions of its own, and has to know of this write.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load_to_lds(const void* base, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off), "s"(base) : "m0", "memory");
}
__device__ __forceinline__ void load_to_lds(const void* src, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(src) : "m0", "memory");
}
// Four of the first kind, from base + off[k] to lds + 1024 k; STREAM: streaming loads.
template <bool STREAM>
__device__ __forceinline__ void load4_to_lds(const void* base, const uint32_t (&off)[4], uint32_t lds) {
#define GMI_LOAD4_TO_LDS(NT)                                                                                                       \
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %5" NT "\n\t"                                            \
               "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %5" NT "\n\t"                                     \
               "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %3, %5" NT "\n\t"                                     \
               "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %4, %5" NT                                            \
               ::"s"(lds), "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(base) : "m0", "scc", "memory")
  if constexpr (STREAM) GMI_LOAD4_TO_LDS(" nt"); else GMI_LOAD4_TO_LDS("");
#undef GMI_LOAD4_TO_LDS
}
#pragma clang diagnostic pop

// LAYOUT: 0 both operands row-major, 1 both in the block layout of the row-tile trainer kernel; STREAM (blocks): beyond_cache.
template <int LAYOUT, bool STREAM>
__global__ __launch_bounds__(512) void wgrad_bf16_kernel(gmi::WgradBatch batch, int rows, float* __restrict__ part, int64_t part_stride) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  // workgroup -> (entry, split and net, tile): the tiles of a split read the same rows, so they belong on one die (ids go round-robin
  // over the 8 dies): whole eights of (split, net) pairs tile by tile, what is left over as it comes
  int ei = 0;
  while (ei + 1 < batch.n_entries && (int)blockIdx.x >= batch.e[ei + 1].start) ++ei;
  const gmi::WgradEntry& E = batch.e[ei];
  const int local = blockIdx.x - E.start, pairs = E.n_split * E.n_nets, whole = pairs & ~7;
  int pair, tile;
  if (local < whole * E.n_tiles) {
    pair = (local >> 3) / E.n_tiles * 8 + (local & 7);
    tile = (local >> 3) % E.n_tiles;
  } else {
    pair = whole + (local - whole * E.n_tiles) % (pairs - whole);
    tile = (local - whole * E.n_tiles) / (pairs - whole);
  }
  const int sp = pair / E.n_nets;
  const gmi::WgradProblem& P = batch.p[pair % E.n_nets ? E.second : E.first];
  const int To = gmi::wgrad_tile(P.out_pad), Ti = gmi::wgrad_tile(P.in_pad);
  const int n_ti = (P.in_pad + Ti - 1) / Ti;
  const int o0 = (tile / n_ti) * To, i0 = (tile % n_ti) * Ti;
  const int o_end = min(P.out_pad, o0 + To), i_end = min(P.in_pad, i0 + Ti);
  const int row_begin = sp * P.chunk;
  const int row_end = min(rows, row_begin + P.chunk);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // ---- loading: waves 0-3 the dz features, waves 4-7 the x features, four 1 KiB pieces per wave and stage
  const bool is_x = wave >= 4;
  const int fmax = is_x ? P.in_pad : P.out_pad, f0 = is_x ? i0 : o0, fend = is_x ? i_end : o_end;
  const char* opnd = is_x ? (const char*)P.x : (const char*)P.dz;
  const int ld = is_x ? P.ldx : P.lddz;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
  const uint32_t lds_w = lds0 + (is_x ? kWgradOperand : 0) + (wave & 3) * 4096;
  // row-major: piece j = rows 2 j, 2 j + 1; lane = (row, 16-byte slot c), slot c holds the features of chunk
  // c ^ 4 (row % 4), so that the four rows and two feature halves of half a wave's transposing read lie in different banks
  const int rl = lane >> 5;
  // blocks: piece j = feature step j of the tile's 16; lane slot L holds (row s, half h) with L = 8 (s / 4) + 4 h + s % 4,
  // in odd steps L ^ 8 (for the same reason)
  const int bs = (lane >> 3) * 4 + (lane & 3), bh = (lane >> 2) & 1;      // odd steps: row bs ^ 4
  const int nks_op = fmax >> 4;
  const int j0 = (wave & 3) * 4;
  // Blocks: a wave has n_ld pieces in the tile.  One with none loads nothing, any other issues four loads a stage, the last piece again
  // in place of those past the tile (what the LDS holds there feeds results that are never stored): with the same number for all
  // waves the wait for them is one instruction.  (As a switch over n_ld and the stages left it was 30 scalar instructions and 8
  // branches, all of a compute unit's waves at the same time between two barriers.)
  const int n_ld = LAYOUT == 1 ? min(max(((fend - f0) >> 4) - j0, 0), 4) : 4;
  // per-lane byte offsets, everything else of an address is wave-uniform: of piece k; row-major, of pieces with even and odd k, and
  // whether the lane's features exist
  uint32_t voff[LAYOUT == 1 ? 4 : 2];
  bool f_ok[2];
  if constexpr (LAYOUT == 1) {
#pragma unroll
    for (int k = 0; k < 4; ++k) voff[k] = ((bs ^ (4 * (k & 1))) + 32 * bh) * 16 + min(k, max(n_ld, 1) - 1) * 4096;
  } else {
#pragma unroll
    for (int par = 0; par < 2; ++par) {
      const int f = f0 + 8 * ((lane & 31) ^ (((2 * par + rl) & 3) << 2));
      voff[par] = (uint32_t)(rl * ld + f) * 2;
      f_ok[par] = f < fend;
    }
  }
  uint32_t put = lds_w;      // where the next stage goes
  auto issue = [&](int stage) {
    const int r0 = row_begin + stage * kWgradRows;
    const uint32_t dst = put;
    put = put == lds_w + (kWgradRing - 1) * kWgradStage ? lds_w : put + kWgradStage;
    if constexpr (LAYOUT == 1) {
      const char* base = opnd + ((((int64_t)(r0 >> 7) * nks_op + (f0 >> 4) + j0) * 4 + ((r0 >> 5) & 3)) << 10);
      if (n_ld > 0) load4_to_lds<STREAM>(base, voff, dst);
    } else if (r0 + kWgradRows <= row_end) {
      const char* base = opnd + (int64_t)(r0 + 2 * j0) * ld * 2;
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (f_ok[k & 1]) load_to_lds(base + (int64_t)k * ld * 4, voff[k & 1], dst + k * 1024);
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int row = r0 + 2 * (j0 + k);
        const void* src = row + rl < row_end ? (const void*)(opnd + (int64_t)row * ld * 2 + voff[k & 1]) : &g_zero_piece;
        if (f_ok[k & 1]) load_to_lds(src, dst + k * 1024);
      }
    }
  };

  // ---- reading: lane group q = lane / 16 takes features 16 (q % 2) .. + 15 and rows 8 (q / 2) .. + 7 of a 32-feature,
  // 16-row operand; a lane addresses row i / 4 (of 4) and features 4 (i % 4) .. + 3, i = lane % 16
  const int i16 = lane & 15, fh = (lane >> 4) & 1, rh = lane >> 5;
  // Waves share the tile's 32 x 32 tiles as a 2 x 4 grid (4 x 2 where there are at most two input tiles), so that a narrow
  // matrix still gives every wave its part: wave (wo, wi) has the output tiles ot0 .. ot0 + nz - 1 and the input tiles
  // xt0 .. xt0 + nx - 1.
  const int n_ot = (o_end - o0) >> 5, n_xt = (i_end - i0) >> 5;
  const int go = n_xt <= 2 ? 4 : 2, gi = 8 / go, wo = wave / gi, wi = wave % gi;
  const int zmax = (n_ot + go - 1) / go, xmax = (n_xt + gi - 1) / gi;
  const int ot0 = wo * zmax, xt0 = wi * xmax;
  const int nz = max(0, min(zmax, n_ot - ot0)), nx = max(0, min(xmax, n_xt - xt0));
  // LDS addresses of the first 4 rows of z tile i and x tile j; *4: of the next 4.  In block layout a tile is 2 KiB after the
  // one before it (an immediate of the read); row-major the swizzle reaches into the tile index.
  constexpr int kRowStep16 = LAYOUT == 1 ? 512 : 8192;      // bytes between rows r and r + 16
  constexpr int kBases = LAYOUT == 1 ? 1 : 4;
  const unsigned char *za[kBases], *za4[kBases], *xa[kBases > 1 ? 2 : 1], *xa4[kBases > 1 ? 2 : 1];
  if constexpr (LAYOUT == 1) {
    const int c = i16 & 3, r = i16 >> 2;
    const bool nat = P.x_blocks == 2;
    const int hz = c & 1, lz = c >> 1, hx = nat ? c >> 1 : c & 1, lx = nat ? c & 1 : c >> 1;
    const int row4 = 2 * rh + fh, row44 = 2 * rh + 1 - fh;      // 4-row groups 2 rh and 2 rh + 1, swapped in odd steps
    const unsigned char* p = smem + (2 * ot0 + fh) * 1024 + (hz * 4 + r) * 16 + 8 * lz;
    const unsigned char* q = smem + kWgradOperand + (2 * xt0 + fh) * 1024 + (hx * 4 + r) * 16 + 8 * lx;
    za[0] = p + row4 * 128; za4[0] = p + row44 * 128;
    xa[0] = q + row4 * 128; xa4[0] = q + row44 * 128;
  } else {
    const int r = i16 >> 2;
    const unsigned char* p = smem + (8 * rh + r) * 512 + 8 * (i16 & 1);
#pragma unroll
    for (int i = 0; i < kBases; ++i) {
      za[i] = p + ((4 * ((ot0 + i) & 7) + 2 * fh + ((i16 & 3) >> 1)) ^ (r << 2)) * 16;
      za4[i] = za[i] + 2048;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if (j >= (kBases > 1 ? 2 : 1)) break;
      xa[j] = p + kWgradOperand + ((4 * ((xt0 + j) & 7) + 2 * fh + ((i16 & 3) >> 1)) ^ (r << 2)) * 16;
      xa4[j] = xa[j] + 2048;
    }
  }
  auto operand = [&](const unsigned char* p, const unsigned char* p4) {
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(p));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(p4));
    const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
  };

  // Bias sums: the na waves that share output tiles divide them, wave wi takes tiles wi and wi + na, through operands of its own.  (All
  // of them by wave 0 from the operands that it has, every wave waited for it at every barrier: 10 of 110 us of
  // 211:512:512:256:128:20.)
  const int na = xmax > 0 ? (n_xt + xmax - 1) / xmax : 1;
  const bool do_bias = i0 == 0 && nx > 0 && wi < nz;
  const int n_bias = do_bias ? (wi + na < nz ? 2 : 1) : 0;
  const unsigned char *zb[2], *zb4[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int i = min(wi + t * na, 3);
    if constexpr (LAYOUT == 1) {
      zb[t] = za[0] + i * 2048;
      zb4[t] = za4[0] + i * 2048;
    } else {
      const int r = i16 >> 2;
      zb[t] = smem + (8 * rh + r) * 512 + 8 * (i16 & 1) + ((4 * ((ot0 + i) & 7) + 2 * fh + ((i16 & 3) >> 1)) ^ (r << 2)) * 16;
      zb4[t] = zb[t] + 2048;
    }
  }

  floatx16 acc[4][2];
  float sum[2][2] = {{0.f, 0.f}, {0.f, 0.f}};      // of a stage's two steps
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
  const bf2 one = {(__bf16)1.0f, (__bf16)1.0f};

  struct Operands { bf16x8 z[4], x[2], b[2]; };
  constexpr int kAhead = kWgradRing - 1;
  const int nst = row_begin < row_end ? (row_end - row_begin + kWgradRows - 1) / kWgradRows : 0;
  // The stage loop of a wave with NZ x NX tiles.  The barrier of iteration s: every wave's pieces of the stages up to s + 1
  // are in LDS, and every wave has read stage s - 1, whose place the newest stage takes.  Operands are read one 16-row step
  // ahead of their products, across the stage boundary: the waves leave the barrier together, and reads before products
  // would leave the matrix cores idle meanwhile.
  auto run = [&](auto nzc, auto nxc, auto biasc) {
    constexpr int NZ = decltype(nzc)::value, NX = decltype(nxc)::value;
    constexpr int NB = decltype(biasc)::value;
    auto read = [&](int off, int k) {
      Operands q;
      const int o = off + k * kRowStep16;
#pragma unroll
      for (int i = 0; i < NZ; ++i) {
        if constexpr (LAYOUT == 1) q.z[i] = operand(za[0] + o + i * 2048, za4[0] + o + i * 2048);
        else q.z[i] = operand(za[i] + o, za4[i] + o);
      }
#pragma unroll
      for (int j = 0; j < NX; ++j) {
        if constexpr (LAYOUT == 1) q.x[j] = operand(xa[0] + o + j * 2048, xa4[0] + o + j * 2048);
        else q.x[j] = operand(xa[j] + o, xa4[j] + o);
      }
#pragma unroll
      for (int t = 0; t < NB; ++t) q.b[t] = operand(zb[t] + o, zb4[t] + o);
      return q;
    };
    // Two sums over the rows, of the even and the odd steps, where the accumulators allow it (wgrad_sums): the layers of small tiles have
    // fewer splits (plan_wgrad).
    constexpr bool kTwo = NX < 2 || NZ <= 2;
    auto second = [&](int i, int j) -> floatx16& { return NX < 2 ? acc[i][1] : acc[i + 2 & 3][j]; };
    auto multiply = [&](const Operands& q, auto step) {
      constexpr int K = decltype(step)::value;
#pragma unroll
      for (int i = 0; i < NZ; ++i)
#pragma unroll
        for (int j = 0; j < NX; ++j) {
          floatx16& a = kTwo && K ? second(i, j) : acc[i][j];
          a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q.z[i], q.x[j], a, 0, 0, 0);
        }
#pragma unroll
      for (int t = 0; t < NB; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bf2 v = {q.b[t][2 * e], q.b[t][2 * e + 1]};
          sum[t][K] = __builtin_amdgcn_fdot2_f32_bf16(v, one, sum[t][K], false);
        }
    };
    // the reads of the next step between the products of this one: a wave issues in order, and a product keeps the matrix
    // core busy for 32 cycles
    auto interleave = [&]() {
      constexpr int kProducts = NZ * NX > 0 ? NZ * NX : 1;
      constexpr int kReads = (2 * (NZ + NX + NB) + kProducts - 1) / kProducts;
#pragma unroll
      for (int m = 0; m < kProducts; ++m) {
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);               // a product
        __builtin_amdgcn_sched_group_barrier(0x2, 2 * kReads, 0);      // vector instructions (addresses)
        __builtin_amdgcn_sched_group_barrier(0x100, kReads, 0);        // LDS reads
      }
    };
    Operands cur;
    int off = 0;      // LDS offset of stage s
    if constexpr (NZ > 0) cur = read(0, 0);
    auto stage = [&](int s, auto more) {
      const int off1 = off == (kWgradRing - 1) * kWgradStage ? 0 : off + kWgradStage;
      if constexpr (NZ > 0) {
        const Operands nxt = read(off, 1);
        multiply(cur, std::integral_constant<int, 0>{});
        interleave();
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (decltype(more)::value) issue(s + kAhead);      // behind products that are on their way
        __builtin_amdgcn_sched_barrier(0);
        cur = read(s + 1 < nst ? off1 : off, 0);
        multiply(nxt, std::integral_constant<int, 1>{});
        interleave();
        __builtin_amdgcn_sched_barrier(0);
      } else {
        if constexpr (decltype(more)::value) issue(s + kAhead);
      }
      off = off1;
    };
    int s = 0;
    for (; s < nst - kAhead; ++s) {
      // the two newest stages may be outstanding
      asm volatile("s_waitcnt vmcnt(8)\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      stage(s, std::true_type{});
    }
    for (; s < nst; ++s) {
      asm volatile("s_waitcnt vmcnt(0)\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      stage(s, std::false_type{});
    }
    if constexpr (kTwo)
#pragma unroll
      for (int i = 0; i < NZ; ++i)
#pragma unroll
        for (int j = 0; j < NX; ++j) acc[i][j] += second(i, j);
  };
  if (nst > 0) {
    for (int s = 0; s < min(kAhead, nst); ++s) issue(s);
    if (nst >= kAhead) asm volatile("s_waitcnt vmcnt(12)" ::: "memory");      // the first stage is there
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    asm volatile("s_barrier" ::: "memory");
    auto pick = [&](auto bias) {
#define GMI_WGRAD_RUN(Z, X) run(std::integral_constant<int, Z>{}, std::integral_constant<int, X>{}, bias)
      if (nz == 0 || nx == 0) GMI_WGRAD_RUN(0, 0);
      else if (nx == 1) {
        if (nz == 1) GMI_WGRAD_RUN(1, 1); else if (nz == 2) GMI_WGRAD_RUN(2, 1); else if (nz == 3) GMI_WGRAD_RUN(3, 1); else GMI_WGRAD_RUN(4, 1);
      } else {
        if (nz == 1) GMI_WGRAD_RUN(1, 2); else if (nz == 2) GMI_WGRAD_RUN(2, 2); else if (nz == 3) GMI_WGRAD_RUN(3, 2); else GMI_WGRAD_RUN(4, 2);
      }
#undef GMI_WGRAD_RUN
    };
    if (n_bias == 0) pick(std::integral_constant<int, 0>{});
    else if (n_bias == 1) pick(std::integral_constant<int, 1>{});
    else pick(std::integral_constant<int, 2>{});
  }

  // tiled partials (ModelLayout::part_floats): a quad of results of a 32 x 32 tile is one 16-byte store per lane
  float* dst = part + (int64_t)sp * part_stride;
  const int n_it = P.in_pad >> 5;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (i >= nz) break;
    const int ot = (o0 >> 5) + ot0 + i;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (32 * ot + 8 * q >= P.out) continue;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int it = (i0 >> 5) + xt0 + j;
        if (j < nx)
          gmi::store_through(dst + P.w_off + (((int64_t)ot * n_it + it) * 4 + q) * 256, lane * 16,
                             acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
      }
    }
  }
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    if (t >= n_bias) break;
    const float h = sum[t][0] + sum[t][1], b = h + __shfl_xor(h, 32, 64);      // the other half of the rows
    if (lane < 32) dst[P.b_off + 32 * ((o0 >> 5) + ot0 + wi + t * na) + lane] = b;
  }
}

// ------------------------------------------------------------------------------------------------
// F32 path: one thread per output element.
template <int EPI>
__global__ void linear_f32_kernel(gmi::LinearBatch batch, int rows) {
  const gmi::LinearProblem& P = batch.p[blockIdx.z];
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)rows * P.F) return;
  const int r = (int)(idx / P.F), f = (int)(idx % P.F);
  const float* x = (const float*)P.x + (int64_t)r * P.ldx;
  const float* w = (const float*)P.w + (int64_t)f * P.wsf;
  float acc = 0.f;
  for (int k = 0; k < P.K; ++k) acc = fmaf(x[k], w[(int64_t)k * P.wsk], acc);
  if (EPI == gmi::kEpiBiasElu) {
    const float z = acc + P.bias[f];
    ((float*)P.y)[(int64_t)r * P.ldy + f] = z > 0.f ? z : expm1f(z);
  } else if (EPI == gmi::kEpiBiasHead) {
    if (f < P.F_store) ((float*)P.y)[(int64_t)r * P.ldy + f] = acc + P.bias[f];
  } else {
    const float h = ((const float*)P.h)[(int64_t)r * P.ldh + f];
    ((float*)P.y)[(int64_t)r * P.ldy + f] = acc * elu_grad_f(h);
  }
}

// grid.x over (out*in + out) outputs of one problem, grid.y = split, grid.z = problem
__global__ void wgrad_f32_kernel(gmi::WgradBatch batch, int rows, int chunk, float* __restrict__ part,
                                 int64_t part_stride) {
  const gmi::WgradProblem& P = batch.p[blockIdx.z];
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  const int nw = P.out * P.in;
  if (idx >= nw + P.out) return;
  const int sp = blockIdx.y;
  const int rb = sp * chunk, re = min(rows, rb + chunk);
  const float* dz = (const float*)P.dz;
  const float* x = (const float*)P.x;
  float acc = 0.f;
  float* dst = part + (int64_t)sp * part_stride;
  if (idx < nw) {
    const int o = idx / P.in, i = idx % P.in;
    for (int r = rb; r < re; ++r) acc = fmaf(dz[(int64_t)r * P.lddz + o], x[(int64_t)r * P.ldx + i], acc);
    dst[P.w_off + idx] = acc;
  } else {
    const int o = idx - nw;
    for (int r = rb; r < re; ++r) acc += dz[(int64_t)r * P.lddz + o];
    dst[P.b_off + o] = acc;
  }
}

template <int TFW, int TRW, int WRN>
int launch_bf16_big(gmi::ProfScope& ps, int epi, int rows, const gmi::LinearBatch& b, int maxF) {
  constexpr int TF = 2 * TFW * 32, TR = WRN * TRW * 32;
  const int n_rt = (rows + TR - 1) / TR, n_ft = (maxF + TF - 1) / TF;
  const int n_rt_pad = (n_rt + 7) & ~7;
  const unsigned grid = (unsigned)(n_rt_pad * n_ft * b.n);
  if (epi == gmi::kEpiBiasElu)
    ps.launch(linear_bf16_big_kernel<TFW, TRW, gmi::kEpiBiasElu, WRN>, dim3(grid), dim3(128 * WRN), 0, b, rows, n_rt,
              n_rt_pad, n_ft);
  else
    ps.launch(linear_bf16_big_kernel<TFW, TRW, gmi::kEpiEluGrad, WRN>, dim3(grid), dim3(128 * WRN), 0, b, rows, n_rt,
              n_rt_pad, n_ft);
  GMI_LAUNCH_CHECK();
  return GMI_OK;
}

template <int WF, int WR, int TFM, int TRM>
int launch_bf16_cfg(gmi::ProfScope& ps, int epi, int rows, const gmi::LinearBatch& b, int maxF) {
  constexpr int TF = WF * TFM * 32, TR = WR * TRM * 32;
  dim3 grid((rows + TR - 1) / TR, (maxF + TF - 1) / TF, b.n);
  switch (epi) {
    case gmi::kEpiBiasElu:
      ps.launch(linear_bf16_kernel<WF, WR, TFM, TRM, gmi::kEpiBiasElu>, dim3(grid), dim3(256), 0, b, rows); break;
    case gmi::kEpiBiasHead:
      ps.launch(linear_bf16_kernel<WF, WR, TFM, TRM, gmi::kEpiBiasHead>, dim3(grid), dim3(256), 0, b, rows); break;
    default:
      ps.launch(linear_bf16_kernel<WF, WR, TFM, TRM, gmi::kEpiEluGrad>, dim3(grid), dim3(256), 0, b, rows); break;
  }
  GMI_LAUNCH_CHECK();
  return GMI_OK;
}

}  // namespace

namespace gmi {

int launch_linear(gmi_instance* g, int dtype, int epi, int rows, const LinearBatch& b) {
  if (rows <= 0 || b.n <= 0) return GMI_OK;
  int maxF = 0;
  for (int i = 0; i < b.n; ++i) maxF = b.p[i].F > maxF ? b.p[i].F : maxF;
  if (dtype != GMI_DTYPE_F32) {
    for (int i = 0; i < b.n; ++i) {
      const LinearProblem& p = b.p[i];
      if ((p.K & 31) || (p.F & 31) || (p.ldx & 7) || (p.ldw & 7) || (epi != kEpiBiasHead && (p.ldy & 3)) ||
          (epi == kEpiEluGrad && (p.ldh & 3)))
        GMI_FAIL(GMI_ERR_BAD_SHAPE, "launch_linear: bf16 path needs padded dims (K=%d F=%d)", p.K, p.F);
    }
  }
  // kernel variant (see KernelClass): large tiles for wide layers of big batches, else by feature count
  int variant;
  if (dtype == GMI_DTYPE_F32) {
    variant = 5;
  } else if (epi != kEpiBiasHead && rows >= 8192 && maxF > 64) {
    // choose the large tile whose padding waste over the feature range is smallest
    const int waste256 = (maxF + 255) / 256 * 256 - maxF, waste128 = (maxF + 127) / 128 * 128 - maxF;
    variant = (maxF > 128 && waste256 <= waste128) ? 0 : 1;
  } else if (maxF % 128 == 0 || maxF > 256) {
    variant = 2;
  } else if (maxF % 64 == 0) {
    variant = 3;
  } else if (maxF <= 96) {
    variant = 4;
  } else {
    variant = 2;
  }
  const int role = epi == kEpiEluGrad ? 2 : (epi == kEpiBiasHead ? 1 : 0);
  ProfScope ps(g, variant == 5 ? (int)kClsLinearF32 : kClsLinear + 3 * variant + role);
  {
    // algorithmic work: 2 K F flops per row; each row's input and output once (heads write fp32, the
    // input-gradient product also reads the layer's stored activation), the weights once
    const double es = dtype == GMI_DTYPE_F32 ? 4.0 : 2.0;
    double fl = 0.0, by = 0.0;
    for (int i = 0; i < b.n; ++i) {
      const double K = b.p[i].K_log > 0 ? b.p[i].K_log : b.p[i].K, F = b.p[i].F_log > 0 ? b.p[i].F_log : b.p[i].F;
      fl += 2.0 * rows * K * F;
      by += rows * (K * es + F * (role == 1 ? 4.0 : es) + (role == 2 ? F * es : 0.0)) + K * F * es;
    }
    ps.work(fl, by);
  }
  switch (variant) {
    case 5: {
      dim3 grid((unsigned)(((int64_t)rows * maxF + 255) / 256), 1, b.n);
      switch (epi) {
        case kEpiBiasElu: ps.launch(linear_f32_kernel<kEpiBiasElu>, dim3(grid), dim3(256), 0, b, rows); break;
        case kEpiBiasHead: ps.launch(linear_f32_kernel<kEpiBiasHead>, dim3(grid), dim3(256), 0, b, rows); break;
        default: ps.launch(linear_f32_kernel<kEpiEluGrad>, dim3(grid), dim3(256), 0, b, rows); break;
      }
      GMI_LAUNCH_CHECK();
      return GMI_OK;
    }
    case 0: return launch_bf16_big<4, 2, 4>(ps, epi, rows, b, maxF);
    case 1: return launch_bf16_big<2, 2, 4>(ps, epi, rows, b, maxF);
    case 2: return launch_bf16_cfg<2, 2, 2, 2>(ps, epi, rows, b, maxF);
    case 3: return launch_bf16_cfg<1, 4, 2, 2>(ps, epi, rows, b, maxF);
    default: return launch_bf16_cfg<1, 4, 1, 2>(ps, epi, rows, b, maxF);
  }
}

// The rest of the cache holds weights, rows and partial gradients.  us per minibatch with its weight gradients and update, without / with the
// streams: 60:256:128:64:8 49152 rows (195 MB) 96 / 98, 53248 109 / 108, 57344 (228 MB) 119 / 111, 65536 137 / 123; 108:400:200:100:21 30000
// (204 MB) 126 / 137, 32768 (222 MB) 135 / 138, 34816 154 / 156, 36000 (244 MB) 160 / 155, 65536 282 / 258; 108:200:400:100:21 32768 136 / 142,
// 40960 177 / 173.
bool beyond_cache(const ModelLayout& L, int rows) {
  int64_t n = 0;
  bool shared = false;
  for (int net = 0; net < 2; ++net)
    for (const LayerInfo& li : L.net[net]) {
      n += li.in_pad + li.out_pad;
      shared = shared || wgrad_tiles(li.out_pad, li.in_pad) >= 4;
    }
  // Matrices of four tiles and more read the same rows through the die's cache, and only the weight gradients of their shapes stream: up to
  // half as much again no difference beyond the runs' own, above it a gain.  211:512:512:256:128:20 20480 rows (252 MB) 211 / 213, 24576 (302 MB)
  // 232 / 228 and 233 / 236, 28672 (352 MB) 267 / 264, 32768 286 / 280, 36864 350 / 336, 40960 375 / 356, 65536 514 / 508;
  // 211:512:512:512:256:20 20480 298 / 302, 24576 307 / 302, 32768 353 / 350, 40960 495 / 488, 65536 678 / 678.
  return 2 * n * rows > (shared ? kCacheBytes / 2 * 3 : kCacheBytes);
}

int even_splits(int n_tiles) { return std::min(std::max(kWgradGroups / n_tiles / 4 * 4, 2 * kSplitMin), kSplitMax / 2); }

// Splits of each layer's rows such that its workgroups read about as much as any other's: as many workgroups in all as keep the
// launch in one round of one per compute unit.  A workgroup's time goes by the bytes of its rows, its tile's features of both operands
// (a stage of few features is bound by the round trip instead, as if it had kWgradNarrow of them: us per minibatch with update for 32 / 192 /
// 224 / 320, 60:256:128:64:8 4096 rows 31.5 / 31.6 / 30.4 / 30.9, 108:200:400:100:21 32768 rows 132 / 137 / 132 / 139, 108:400:200:100:21 134.8 /
// 133.9 / 134.5 / 137.3; 512-wide shapes within 1 %), and with the same splits for all layers the launch
// took as long as the widest tile's.  No layer forms fewer partial sums of its rows (splits times wgrad_sums) than the same splits for all would:
// each addition rounds.  Error of the weights' gradients against 64-bit sums, root mean square over the tensors, 32768 rows as collected, with
// the same splits / per layer, one sum each / as it is: 60:256:128:64:8 7.7e-8 / 7.6e-8 / 6.5e-8, 108:400:200:100:21 1.13e-7 / 1.15e-7 / 0.94e-7,
// 211:512:512:256:128:20 1.57e-7 / 1.64e-7 / 1.41e-7 (its policy head 1.5 times as far off with one sum).
WgradSplits plan_wgrad(const int* out_pad, const int* in_pad, int n) {
  WgradSplits r = {};
  int tiles[kMaxWgradProblems], feats[kMaxWgradProblems], all = 0, used = 0;
  for (int i = 0; i < n; ++i) {
    tiles[i] = wgrad_tiles(out_pad[i], in_pad[i]);
    feats[i] = std::max(wgrad_tile(out_pad[i]) + wgrad_tile(in_pad[i]), kWgradNarrow);
    all += tiles[i];
  }
  const int same = even_splits(all);
  for (int i = 0; i < n; ++i) {
    r.n[i] = same / wgrad_sums(out_pad[i], in_pad[i]);
    used += tiles[i] * r.n[i];
  }
  for (;;) {
    int most = 0;
    for (int i = 1; i < n; ++i)
      if (feats[i] * r.n[most] > feats[most] * r.n[i]) most = i;
    int add = 0;      // all problems alike, i.e. both nets' layers of one shape, together
    auto alike = [&](int i) { return out_pad[i] == out_pad[most] && in_pad[i] == in_pad[most] && r.n[i] == r.n[most]; };
    for (int i = 0; i < n; ++i) add += alike(i) ? tiles[i] : 0;
    if (used + add > kWgradGroups || r.n[most] == kSplitMax) return r;
    used += add;
    const int to = r.n[most] + 1;
    for (int i = n - 1; i >= 0; --i)
      if (i != most && alike(i)) r.n[i] = to;
    r.n[most] = to;
  }
}

int launch_wgrad(gmi_instance* g, int dtype, int rows, int n_split, int chunk, WgradBatch& b, float* part,
                 int64_t part_stride, bool stream) {
  if (b.n <= 0) return GMI_OK;
  ProfScope ps(g, kClsWgrad);
  {
    // algorithmic work: 2 in out flops per row; every layer's input and output gradient read once, one
    // fp32 partial per split written
    const double es = dtype == GMI_DTYPE_F32 ? 4.0 : 2.0;
    double fl = 0.0, by = 0.0;
    for (int i = 0; i < b.n; ++i) {
      fl += 2.0 * rows * (double)b.p[i].in * b.p[i].out;
      by += rows * es * (b.p[i].in + b.p[i].out) +
            4.0 * (dtype == GMI_DTYPE_F32 ? n_split : b.p[i].n_split) * ((double)b.p[i].in * b.p[i].out + b.p[i].out);
    }
    ps.work(fl, by);
  }
  if (dtype == GMI_DTYPE_F32) {
    int maxn = 0;
    for (int i = 0; i < b.n; ++i) {
      const int n = b.p[i].out * b.p[i].in + b.p[i].out;
      maxn = n > maxn ? n : maxn;
    }
    dim3 grid((maxn + 255) / 256, n_split, b.n);
    ps.launch(wgrad_f32_kernel, dim3(grid), dim3(256), 0, b, rows, chunk, part, part_stride);
    GMI_LAUNCH_CHECK();
    return GMI_OK;
  }
  // problems 0 .. n / 2 - 1 are the policy net's layers, the rest the value net's
  const int half = b.n / 2;
  int total = 0;
  b.n_entries = 0;
  auto entry = [&](int first, int second, int n_nets) {
    const WgradProblem& p = b.p[first];
    WgradEntry& e = b.e[b.n_entries++];
    e.first = first; e.second = second; e.n_nets = n_nets;
    e.n_tiles = wgrad_tiles(p.out_pad, p.in_pad); e.n_split = p.n_split; e.start = total;
    total += n_nets * e.n_tiles * e.n_split;
  };
  for (int i = 0; i < (b.n % 2 ? b.n : half); ++i) {
    const WgradProblem &p = b.p[i], &q = b.p[(i + half) % b.n];
    if (b.n % 2) entry(i, i, 1);
    else if (p.out_pad == q.out_pad && p.in_pad == q.in_pad && p.n_split == q.n_split && p.chunk == q.chunk) entry(i, i + half, 2);
    else { entry(i, i, 1); entry(i + half, i + half, 1); }
  }
  static DeviceSet allowed[3];
  const int variant = b.p[0].dz_blocks ? (stream ? 2 : 1) : 0;
  const auto kernel = variant == 2 ? wgrad_bf16_kernel<1, true> : variant == 1 ? wgrad_bf16_kernel<1, false> : wgrad_bf16_kernel<0, false>;
  const int rc = allow_lds((const void*)kernel, kWgradLds, g->device, &allowed[variant]);
  if (rc != GMI_OK) return rc;
  ps.launch(kernel, dim3(total), dim3(512), kWgradLds, b, rows, part, part_stride);
  GMI_LAUNCH_CHECK();
  return GMI_OK;
}

}  // namespace gmi
