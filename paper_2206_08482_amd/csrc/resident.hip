// Resident trainer kernel (bf16 models, any layer widths whose tile fits LDS): minibatch gather, forward pass,
// clipped-surrogate / value loss and the whole backward pass of a row tile with the tile's activations resident in LDS
// from the gather to the last gradient (stage (ii) of Section 5.1 of the paper, the "DRL Trainer" role of Section 3).
//
// A workgroup of 8 waves owns R = 32 RT rows of one net.  Activations are row-major [row][feature] in LDS (rows of
// K + 8 elements: an odd number of 16-byte pieces, so that 16-byte operand reads of consecutive rows hit different banks);
// the gradient at a hidden layer's output takes the place of that layer's output, element for element, in the epilogue
// that multiplies by ELU'.  Products are computed transposed (32x32x16 matrix instruction, weights first operand from
// the fragment-major copies in L2, activations second): an item is one 32-feature tile for one or two row tiles, items
// are dealt to the waves, and a wave requests the first weight blocks of its next item before it leaves the present one.
//
// Weight gradients, where the net's 64x64 blocks of dW number at most 8 NS (NS = 1, 2): block b belongs to wave b % 8,
// which keeps it in registers (64 per block) over all row tiles of its workgroup.  dW contracts over rows, the strided
// index of both operands: the transposing LDS read (4 rows x 16 features per 16 lanes) delivers them in operand order, so
// neither activations nor gradients ever leave the compute unit; what does is one partial gradient per workgroup.  Bias
// gradients are row sums of the same operands (two-element dot products with ones).  Against storing activations and
// gradients for a second kernel this replaces about 7.6 KB of traffic per row (written, read back for ELU', read again)
// by the observation row, at 4 bytes of partial gradient per parameter and workgroup.
// NS = 0: nets with more weights; activations and gradients go to memory row-major for wgrad_bf16_kernel.
//
// Bound: LDS operand reads (1 KiB per matrix instruction with items of two row tiles: the rate of the LDS) and the
// epilogues' vector arithmetic.
#include <algorithm>

#include "chain_stream.h"

namespace {
using namespace gmi_chain;

__device__ __forceinline__ float wave_sum64(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4* lds_s16x4;

constexpr int kNT = 512, kNW = 8;
constexpr int kTouchLayers = 4;
constexpr int kMaxLayers = GMI_MAX_HIDDEN + 1;
constexpr size_t kLdsMax = 160 * 1024;
constexpr int kDzStride = 32 + 8;           // head gradient rows

struct ResLayer {
  const uint4* wf;         // fragment-major W: operand blocks of the forward product
  const uint4* wtf;        // fragment-major W^T: of the input-gradient product
  const float* bias;
  uint16_t *h_out, *dz_out;      // NS = 0: where the layer's input and output gradient go
  int K, F;                // padded widths
  int in, out;             // logical widths
  int x_off, b_off;        // LDS: the layer's input rows (elements), its biases (floats)
  int w_par, b_par;        // offsets into a row of gradient partials (ModelLayout::part_floats)
};
struct ResNet {
  ResLayer l[kMaxLayers];
};
struct ResArgs {
  ResNet net[2];
  int nl, rows, n_tiles, obs_dim, act_dim, n_envs, ld_envs, vec_obs;
  int dz_off;              // LDS elements: head gradient rows
  int f_off;               // LDS bytes: float area
  int bias_floats;
  uint32_t o_magic, a_magic;
  const float* log_std;
  const int32_t* idx;
  const float *b_obs, *b_act, *b_logp, *b_adv, *b_ret;
  float clip, c_v;
  float* part; int64_t part_stride;
  float* stat_part;
  int n_grp[2];            // 64x64 blocks of dW per net
  uint32_t grp[2][16];     // layer << 24 | first output block << 12 | first input block (in units of 32)
};

__device__ __forceinline__ bf16x8 tr_read(const uint16_t* p, int stride4) {
  // 8 rows x the lane's feature: rows 0..3 and 4..7 of the lane group's block (stride4 = 4 rows in elements)
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(p));
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(p + stride4));
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  return __builtin_bit_cast(bf16x8, v);
}

__device__ __forceinline__ float row_sum8(bf16x8 v, float acc) {
  typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
  const bf2 one = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const bf2 e = {v[2 * q], v[2 * q + 1]};
    acc = __builtin_amdgcn_fdot2_f32_bf16(e, one, acc, false);
  }
  return acc;
}

__host__ __device__ __forceinline__ uint32_t magic(uint32_t d) { return d == 1 ? 0u : 0xFFFFFFFFu / d + 1u; }
__device__ __forceinline__ int div_magic(int n, uint32_t m) { return m ? (int)__umulhi((uint32_t)n, m) : n; }      // n * d < 2^32

// One product of the walk: segment s < nl is layer s forward, s >= nl the input gradient of layer 2 nl - 1 - s.
struct SegInfo {
  const uint4* w;
  int K, F, x_off, y_off;
  bool bwd;
  int l;
};
__device__ __forceinline__ SegInfo seg_info(const ResArgs& a, const ResNet& N, int s) {
  SegInfo g;
  g.bwd = s >= a.nl;
  g.l = g.bwd ? 2 * a.nl - 1 - s : s;
  const ResLayer& L = N.l[g.l];
  g.w = g.bwd ? L.wtf : L.wf;
  g.K = g.bwd ? L.F : L.K;
  g.F = g.bwd ? L.K : L.F;
  const int nxt = g.l + 1 < a.nl ? N.l[g.l + 1].x_off : a.dz_off;      // where the layer's output / its gradient lives
  g.x_off = g.bwd ? nxt : L.x_off;
  g.y_off = g.bwd ? L.x_off : nxt;
  return g;
}

// acc[i] += W tile x row tiles at xp, xp + xts; w: the tile's weight blocks (wave-uniform), of which wq holds the first 4 k
// steps' for this lane.  Addresses in scalar registers: with a vector address per load a minibatch of 4096 rows of
// 211:512:512:256:128:20 took 92 us instead of 87, of 108:400:200:100:21 52.9 instead of 50.9.
template <int NRT>
__device__ __forceinline__ void k_loop(floatx16 (&acc)[NRT], uint4 (&wq)[4], const uint4* w, int nks, const uint16_t* xp, int xts, int lane) {
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
    wq[u] = gmi::load_uniform(w, min(ks + 4, nks - 1) * 1024, lane * 16);
  };
  for (int ks = 0; ks < nks; ks += 4) {      // nks is even
    step(ks, 0);
    step(ks + 1, 1);
    if (ks + 2 < nks) {
      step(ks + 2, 2);
      step(ks + 3, 3);
    }
  }
}

// Results of an item (features f0 .. f0 + 31 of NRT row tiles at y): lane (s, h) holds, per quad q, the features
// f0 + 8 q + 4 h + 0..3 of row s.  Forward: ELU (the bias is in the sums).  Backward: times ELU' of the stored output,
// which the product then replaces.
template <int NRT, bool BWD>
__device__ __forceinline__ void epilogue(const floatx16 (&acc)[NRT], uint16_t* y, int sy, int f0, int lane) {
  uint16_t* p = y + (lane & 31) * sy + f0 + 4 * (lane >> 5);
  uint2 hv[NRT][4];
  if constexpr (BWD) {
#pragma unroll
    for (int i = 0; i < NRT; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) hv[i][q] = *reinterpret_cast<const uint2*>(p + i * 32 * sy + 8 * q);
  }
#pragma unroll
  for (int i = 0; i < NRT; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float v0 = acc[i][4 * q + 0], v1 = acc[i][4 * q + 1], v2 = acc[i][4 * q + 2], v3 = acc[i][4 * q + 3];
      if constexpr (BWD) {
        v0 *= elu_grad_f(bf16_lo(hv[i][q].x)); v1 *= elu_grad_f(bf16_hi(hv[i][q].x));
        v2 *= elu_grad_f(bf16_lo(hv[i][q].y)); v3 *= elu_grad_f(bf16_hi(hv[i][q].y));
      } else {
        v0 = elu_f(v0); v1 = elu_f(v1); v2 = elu_f(v2); v3 = elu_f(v3);
      }
      *reinterpret_cast<uint2*>(p + i * 32 * sy + 8 * q) = make_uint2(pack_bf16(v0, v1), pack_bf16(v2, v3));
    }
}

// The workgroup's rows of one activation (or gradient) array, LDS -> memory, 16 bytes per lane.
__device__ __forceinline__ void rows_out(const uint16_t* src, int width, int R, uint16_t* dst, int wave, int lane) {
  const int np = width >> 3;
  int lpr = 4;
  while (lpr < 64 && lpr < np) lpr <<= 1;
  const int rpw = 64 / lpr, c0 = lane & (lpr - 1), rl = lane / lpr;
#pragma unroll 2
  for (int r = wave * rpw + rl; r < R; r += kNW * rpw)
    for (int c = c0; c < np; c += lpr)
      gmi::store_through(dst, (uint32_t)(r * width + 8 * c) * 2, *reinterpret_cast<const uint4*>(src + r * (width + 8) + 8 * c));
}

template <int RT, int NS>
__global__ __launch_bounds__(kNT) void train_resident_kernel(ResArgs a) {
  constexpr int R = 32 * RT;
  constexpr int PR = RT >= 2 ? 2 : 1;               // row tiles of a paired item
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  uint16_t* s_x = reinterpret_cast<uint16_t*>(smem_raw);
  float* s_bias = reinterpret_cast<float*>(smem_raw + a.f_off);
  float* s_ls = s_bias + a.bias_floats;             // [32] log_std, [32] exp(-log_std), zero beyond act_dim
  float* s_scal = s_ls + 64;                        // [3][R] old log-prob, advantage, return
  int64_t* s_slot = reinterpret_cast<int64_t*>(s_scal + 3 * R);      // [R]
  float* s_red = reinterpret_cast<float*>(s_slot + R);               // [RT][40]
  float* s_act = s_red + RT * 40;                   // [R][act_dim]
  const int net = blockIdx.y;
  const ResNet& N = a.net[net];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int s = lane & 31, h = lane >> 5;
  const int nl = a.nl, O = a.obs_dim, A = a.act_dim, K0 = N.l[0].K, S0 = K0 + 8;
  const float inv_m = 1.0f / (float)a.rows;

  // this workgroup's gradient blocks and their bias sums, statistics and log_std gradient of this lane's samples
  floatx16 gw[NS > 0 ? NS : 1][2][2];
  float gb[NS > 0 ? NS : 1][2];
  uint32_t gd[NS > 0 ? NS : 1];
  if constexpr (NS > 0) {
#pragma unroll
    for (int n = 0; n < NS; ++n) {
      gd[n] = wave + kNW * n < a.n_grp[net] ? a.grp[net][wave + kNW * n] : 0xFF000000u;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        gb[n][i] = 0.f;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) gw[n][i][j][v] = 0.f;
      }
    }
  }
  float s_pl = 0.f, s_vl = 0.f, s_kl = 0.f, s_cf = 0.f, dls = 0.f;

  for (int f = tid; f < a.bias_floats; f += kNT) {      // all layers' biases at once
    int l = 0;
    while (l + 1 < nl && f >= N.l[l + 1].b_off) ++l;
    s_bias[f] = N.l[l].bias[f - N.l[l].b_off];
  }
  if (tid < 32) {
    const float ls = a.log_std[tid < A ? tid : A - 1];
    s_ls[tid] = tid < A ? ls : 0.f;
    s_ls[32 + tid] = tid < A ? expf(-ls) : 0.f;
  }
  {   // padding columns of the observation rows, once
    const int np = K0 - O;
    for (int r = tid; r < R; r += kNT)
      for (int c = 0; c < np; ++c) s_x[N.l[0].x_off + r * S0 + O + c] = 0;
  }

  // items of a product with nft feature tiles: (feature tile, pair of row tiles) where that gives every wave one, else
  // (feature tile, row tile); the first weight blocks of this wave's first item are requested ahead (wq)
  auto paired = [&](int nft) { return RT >= 2 && nft * (RT / 2) >= kNW; };
  uint4 wq[4];
  auto request = [&](const SegInfo& g, int item) {
    const int nft = g.F >> 5, nks = g.K >> 4, nrg = paired(nft) ? RT / PR : RT;
    const int ft = min(item / nrg, nft - 1);
    const uint4* w = g.w + (int64_t)ft * nks * 64;
#pragma unroll
    for (int u = 0; u < 4; ++u) wq[u] = gmi::load_uniform(w, min(u, nks - 1) * 1024, lane * 16);
  };
  // dW block n of this wave += dz^T x over the tile's rows
  auto wgrad = [&](int l) {
    if constexpr (NS > 0) {
#pragma unroll
      for (int n = 0; n < NS; ++n) {
        if ((int)(gd[n] >> 24) == l) {
          const ResLayer& L = N.l[l];
          const int ob = (gd[n] >> 12) & 0xFFF, ib = gd[n] & 0xFFF;      // in units of 32 features
          const int sz = (l + 1 < nl ? L.F + 8 : kDzStride), sx = L.K + 8;
          const uint16_t* zb = s_x + (l + 1 < nl ? N.l[l + 1].x_off : a.dz_off);
          const uint16_t* xb = s_x + L.x_off;
          // lane group (lane / 16): features 16 * (group % 2) of the tile, rows 8 * (group / 2); a lane addresses row
          // (lane % 16) / 4, features 4 * (lane % 4) of its group's block.  A second tile that does not exist is the first.
          const int o1 = ob + 1 < (L.F >> 5) ? 1 : 0, i1 = ib + 1 < (L.K >> 5) ? 1 : 0;
          const int rl = 8 * h + ((lane & 15) >> 2), cl = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
          const uint16_t* zp = zb + rl * sz + 32 * ob + cl;
          const uint16_t* xp = xb + rl * sx + 32 * ib + cl;
#pragma unroll 2
          for (int r = 0; r < R; r += 16) {
            bf16x8 z[2], x[2];
            z[0] = tr_read(zp + r * sz, 4 * sz);
            z[1] = tr_read(zp + r * sz + 32 * o1, 4 * sz);
            x[0] = tr_read(xp + r * sx, 4 * sx);
            x[1] = tr_read(xp + r * sx + 32 * i1, 4 * sx);
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
              for (int j = 0; j < 2; ++j)
                gw[n][i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(z[i], x[j], gw[n][i][j], 0, 0, 0);
            if (ib == 0) {
#pragma unroll
              for (int i = 0; i < 2; ++i) gb[n][i] = row_sum8(z[i], gb[n][i]);
            }
          }
        }
      }
    }
  };

  SegInfo g = seg_info(a, N, 0);
  request(g, wave);
  // sample of row tid of the present tile (rows past the batch take its last sample; their gradient is zero)
  int sample = tid < R ? a.idx[min((int)blockIdx.x * R + tid, a.rows - 1)] : 0;
  // One word of each of the weights' 128-byte lines (the first kNT of a matrix), so that they are on their way to the die's cache while the
  // rows are: Adam has just written them, and every layer's products waited for them from beyond it.
  // (45:128:128:12, us per iteration 665 without, 658 with.)
  uint32_t touched[kTouchLayers][2];
#pragma unroll
  for (int i = 0; i < kTouchLayers; ++i) {
    const ResLayer& L = N.l[min(i, nl - 1)];
    const int line = min(tid, (L.K * L.F >> 6) - 1);
    touched[i][0] = reinterpret_cast<const uint32_t*>(L.wf)[32 * line];
    touched[i][1] = reinterpret_cast<const uint32_t*>(i > 0 ? L.wtf : L.wf)[32 * line];
  }
  for (int tile = blockIdx.x; tile < a.n_tiles; tile += gridDim.x) {
    const int r0 = tile * R;
    if (tid < R) s_slot[tid] = (int64_t)(sample / a.n_envs) * a.ld_envs + (sample % a.n_envs);
    __syncthreads();
    {   // the gather: every load of a batch is issued before the first result is stored
      float sc0 = 0.f, sc1 = 0.f;
      if (tid < R) {
        const int64_t slot = s_slot[tid];
        sc0 = net == 0 ? a.b_logp[slot] : a.b_ret[slot];
        sc1 = a.b_adv[slot];
        sample = a.idx[min((tile + (int)gridDim.x) * R + tid, a.rows - 1)];      // the next tile's
      }
      float av[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int e = min(tid + u * kNT, R * A - 1), r = div_magic(e, a.a_magic);
        av[u] = net == 0 ? a.b_act[s_slot[r] * A + e - r * A] : 0.f;
      }
      uint16_t* x0 = s_x + N.l[0].x_off;
      if (a.vec_obs) {
        const int n4 = O >> 2, n = R * n4;
        for (int e0 = tid; e0 < n; e0 += 4 * kNT) {
          float4 v[4];
          int d[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int e = min(e0 + u * kNT, n - 1), r = div_magic(e, a.o_magic), c = 4 * (e - r * n4);
            v[u] = *reinterpret_cast<const float4*>(a.b_obs + s_slot[r] * O + c);
            d[u] = r * S0 + c;
          }
#pragma unroll
          for (int u = 0; u < 4; ++u)
            *reinterpret_cast<uint2*>(x0 + d[u]) = make_uint2(pack_bf16(v[u].x, v[u].y), pack_bf16(v[u].z, v[u].w));
        }
      } else {
        const int n = R * O;
        for (int e0 = tid; e0 < n; e0 += 8 * kNT) {
          float v[8];
          int d[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const int e = min(e0 + u * kNT, n - 1), r = div_magic(e, a.o_magic), c = e - r * O;
            v[u] = a.b_obs[s_slot[r] * O + c];
            d[u] = r * S0 + c;
          }
#pragma unroll
          for (int u = 0; u < 8; ++u) x0[d[u]] = (uint16_t)pack_bf16(v[u], 0.f);
        }
      }
      if (tid < R) { s_scal[net == 0 ? tid : 2 * R + tid] = sc0; s_scal[R + tid] = sc1; }
      if (net == 0) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
          if (tid + u * kNT < R * A) s_act[tid + u * kNT] = av[u];
        for (int e = tid + 2 * kNT; e < R * A; e += kNT) {
          const int r = div_magic(e, a.a_magic);
          s_act[e] = a.b_act[s_slot[r] * A + e - r * A];
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kTouchLayers; ++i) asm volatile("" ::"v"(touched[i][0]), "v"(touched[i][1]));

    for (int sg = 0; sg < 2 * nl - 1; ++sg) {
      const int nft = g.F >> 5, nks = g.K >> 4;
      const uint16_t* x = s_x + g.x_off;
      uint16_t* y = s_x + g.y_off;
      const int sx = g.K + 8, sy = g.F + 8;
      const float* bias = s_bias + N.l[g.l].b_off;
      if constexpr (NS == 0) {      // this segment's input to memory, for the weight gradients
        uint16_t* dst = g.bwd ? N.l[g.l].dz_out : N.l[g.l].h_out;
        if (g.bwd || g.l > 0 || net == 0) rows_out(x, g.K, R, dst + (int64_t)r0 * g.K, wave, lane);
      } else if (g.bwd) {
        wgrad(g.l);
      }
      const SegInfo gn = seg_info(a, N, sg + 1 < 2 * nl - 1 ? sg + 1 : 0);
      if (!g.bwd && g.l == nl - 1) {
        // head (one feature tile) and loss: wave w < RT has row tile w; lane (s, h): sample s, features 8 q + 4 h + e
        if (wave < RT) {
          floatx16 acc[1];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const float4 b4 = *reinterpret_cast<const float4*>(bias + 8 * q + 4 * h);
            acc[0][4 * q] = b4.x; acc[0][4 * q + 1] = b4.y; acc[0][4 * q + 2] = b4.z; acc[0][4 * q + 3] = b4.w;
          }
          k_loop<1>(acc, wq, g.w, nks, x + (wave * 32 + s) * sx + 8 * h, 0, lane);
          const int r = wave * 32 + s;
          const bool ok = r0 + r < a.rows;
          uint2* dzp = reinterpret_cast<uint2*>(y + r * kDzStride + 4 * h);      // head gradient, 4 features per piece
          if (net == 0) {
            float z[16], lp = 0.f;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int f0 = 8 * q + 4 * h;
              const float4 ls4 = *reinterpret_cast<const float4*>(s_ls + f0), ig4 = *reinterpret_cast<const float4*>(s_ls + 32 + f0);
              const float lsv[4] = {ls4.x, ls4.y, ls4.z, ls4.w}, igv[4] = {ig4.x, ig4.y, ig4.z, ig4.w};
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const int i = 4 * q + e;
                z[i] = (s_act[r * A + min(f0 + e, A - 1)] - acc[0][i]) * igv[e];      // 0 beyond the actions
                lp += f0 + e < A ? -0.5f * z[i] * z[i] - lsv[e] - 0.918938533204672742f : 0.f;
              }
            }
            lp += __shfl_xor(lp, 32, 64);
            float g_lp = 0.f;
            if (ok) {
              const float lo = s_scal[r], ad = s_scal[R + r];
              const float ratio = expf(lp - lo);
              const float u1 = ratio * ad;
              const float u2 = fminf(fmaxf(ratio, 1.0f - a.clip), 1.0f + a.clip) * ad;
              g_lp = (u1 <= u2) ? -(ad * ratio) * inv_m : 0.f;
              if (h == 0) {
                s_pl += -fminf(u1, u2);
                s_kl += lo - lp;
                s_cf += fabsf(ratio - 1.0f) > a.clip ? 1.f : 0.f;
              }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int f0 = 8 * q + 4 * h;
              const float4 ig4 = *reinterpret_cast<const float4*>(s_ls + 32 + f0);
              dzp[2 * q] = make_uint2(pack_bf16(g_lp * z[4 * q] * ig4.x, g_lp * z[4 * q + 1] * ig4.y),
                                      pack_bf16(g_lp * z[4 * q + 2] * ig4.z, g_lp * z[4 * q + 3] * ig4.w));
#pragma unroll
              for (int e = 0; e < 4; ++e) z[4 * q + e] = f0 + e < A ? g_lp * (z[4 * q + e] * z[4 * q + e] - 1.0f) : 0.f;
            }
            // log_std gradient: sum over the 32 samples, halving the features a lane carries at every exchange; lane s
            // ends with feature index i whose bits 3, 2, 1, 0 are bits 0, 1, 2, 3 of s
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              const int half = 8 >> k;
              const bool up = (s >> k) & 1;
#pragma unroll
              for (int j = 0; j < half; ++j) {
                const float keep = up ? z[j + half] : z[j], send = up ? z[j] : z[j + half];
                z[j] = keep + __shfl_xor(send, 1 << k, 64);
              }
            }
            dls += z[0] + __shfl_xor(z[0], 16, 64);
          } else {
            float d0 = 0.f;
            if (ok && h == 0) {
              const float dv = acc[0][0] - s_scal[2 * R + r];
              s_vl += dv * dv;
              d0 = 2.0f * a.c_v * dv * inv_m;
            }
            dzp[0] = make_uint2(pack_bf16(d0, 0.f), 0u);
#pragma unroll
            for (int q = 1; q < 4; ++q) dzp[2 * q] = make_uint2(0u, 0u);
          }
        }
        request(gn, wave);
      } else {
        auto items = [&](auto nrt, auto bwd) {
          constexpr int NRT = decltype(nrt)::value;
          constexpr bool BWD = decltype(bwd)::value;
          constexpr int nrg = RT / NRT;
          const int n_items = nft * nrg;
          bool waited = !(NS > 0 && BWD);      // weight gradients read the rows that the epilogue overwrites
          for (int item = wave; item < n_items; item += kNW) {
            const int ft = item / nrg, rg = item % nrg;
            floatx16 acc[NRT];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              float4 b4 = make_float4(0.f, 0.f, 0.f, 0.f);
              if constexpr (!BWD) b4 = *reinterpret_cast<const float4*>(bias + 32 * ft + 8 * q + 4 * h);
#pragma unroll
              for (int i = 0; i < NRT; ++i) { acc[i][4 * q] = b4.x; acc[i][4 * q + 1] = b4.y; acc[i][4 * q + 2] = b4.z; acc[i][4 * q + 3] = b4.w; }
            }
            k_loop<NRT>(acc, wq, g.w + (int64_t)ft * nks * 64, nks, x + (rg * NRT * 32 + s) * sx + 8 * h, 32 * sx, lane);
            const bool more = item + kNW < n_items;
            if (more) request(g, item + kNW); else request(gn, wave);
            if (!waited) { __syncthreads(); waited = true; }
            epilogue<NRT, BWD>(acc, y + rg * NRT * 32 * sy, sy, ft * 32, lane);
          }
          if (wave >= n_items) request(gn, wave);
          if (!waited) __syncthreads();
        };
        typedef std::integral_constant<int, PR> Pair;
        typedef std::integral_constant<int, 1> One;
        if (paired(nft)) {
          if (g.bwd) items(Pair{}, std::true_type{}); else items(Pair{}, std::false_type{});
        } else {
          if (g.bwd) items(One{}, std::true_type{}); else items(One{}, std::false_type{});
        }
      }
      __syncthreads();
      g = gn;
    }
    // the first layer's weight gradient, or its inputs to memory
    if constexpr (NS > 0) {
      wgrad(0);
    } else {
      const int off = nl > 1 ? N.l[1].x_off : a.dz_off;
      rows_out(s_x + off, N.l[0].F, R, N.l[0].dz_out + (int64_t)r0 * N.l[0].F, wave, lane);
    }
    __syncthreads();
  }

  if constexpr (NS > 0) {
    float* part = a.part + (int64_t)blockIdx.x * a.part_stride;
#pragma unroll
    for (int n = 0; n < NS; ++n) {
      const int l = (int)(gd[n] >> 24);
      if (l < nl) {
        const ResLayer& L = N.l[l];
        const int ob = (gd[n] >> 12) & 0xFFF, ib = gd[n] & 0xFFF, n_it = L.K >> 5;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            if (32 * (ob + i) + 8 * q >= L.out) continue;
#pragma unroll
            for (int j = 0; j < 2; ++j)
              if (ib + j < n_it)
                gmi::store_through(part + L.w_par + ((((ob + i) * n_it + ib + j) * 4 + q) << 8), lane * 16,
                                   gw[n][i][j][4 * q], gw[n][i][j][4 * q + 1], gw[n][i][j][4 * q + 2], gw[n][i][j][4 * q + 3]);
          }
        if (ib == 0) {
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const float b = gb[n][i] + __shfl_xor(gb[n][i], 32, 64);
            if (h == 0 && 32 * (ob + i) + s < L.F) part[L.b_par + 32 * (ob + i) + s] = b;
          }
        }
      }
    }
  }
  // statistics: lanes -> wave -> workgroup
  if (wave < RT) {
    s_pl = wave_sum64(s_pl); s_vl = wave_sum64(s_vl); s_kl = wave_sum64(s_kl); s_cf = wave_sum64(s_cf);
    float* red = s_red + wave * 40;
    if (lane == 0) { red[0] = s_pl; red[1] = s_vl; red[2] = s_kl; red[3] = s_cf; }
    const int i = 8 * (s & 1) + 4 * ((s >> 1) & 1) + 2 * ((s >> 2) & 1) + ((s >> 3) & 1);
    if (s < 16) red[8 + 8 * (i >> 2) + 4 * h + (i & 3)] = dls;
  }
  __syncthreads();
  float* out = a.stat_part + (int64_t)blockIdx.x * (gmi::kStatStride + A);
  auto total = [&](int k) {
    float v = 0.f;
    for (int w = 0; w < RT; ++w) v += s_red[w * 40 + k];
    return v;
  };
  if (net == 0) {
    if (tid == 0) { out[0] = total(0); out[3] = total(2); out[4] = total(3); out[5] = out[6] = out[7] = 0.f; }
    if (tid == 1) {
      float ent = 0.f;
      if (blockIdx.x == 0)
        for (int j = 0; j < A; ++j) ent += s_ls[j] + 1.418938533204672742f;
      out[2] = ent;
    }
    if (tid >= 64 && tid < 64 + A) out[gmi::kStatStride + tid - 64] = total(8 + tid - 64);
  } else if (tid == 0) {
    out[1] = total(1);
  }
}

// ------------------------------------------------------------------------------------------------
struct Plan {
  int RT, NS;
  size_t lds;
  int f_off, x_off[kMaxLayers], dz_off, b_off[kMaxLayers], bias_floats;
};

int n_blocks(const ModelLayout& L, int net) {
  int n = 0;
  for (const LayerInfo& li : L.net[net]) n += ((li.out_pad + 63) / 64) * ((li.in_pad + 63) / 64);
  return n;
}

bool plan_lds(const ModelLayout& L, int RT, Plan* p) {
  const int R = 32 * RT;
  int off = 0, b = 0;
  for (int l = 0; l < L.n_layers; ++l) {
    p->x_off[l] = off;
    off += R * (L.net[0][l].in_pad + 8);
    p->b_off[l] = b;
    b += L.net[0][l].out_pad;
  }
  p->dz_off = off;
  off += R * kDzStride;
  p->f_off = (off * 2 + 15) & ~15;
  p->bias_floats = b;
  p->RT = RT;
  p->lds = (size_t)p->f_off + 4 * ((size_t)b + 64 + 3 * R + 2 * R + RT * 40 + R * L.act_dim);
  return p->lds <= kLdsMax;
}

// Shape conditions alone: one 32-wide head per net, equal padded widths, a 32-row tile in LDS.
bool shape_ok(const ModelLayout& L) {
  if (L.dtype != GMI_DTYPE_BF16 || L.act_dim > 32) return false;
  if (L.part_floats >= (1ll << 31)) return false;
  Plan p;
  return plan_lds(L, 1, &p);
}

// Sets of dW blocks that a wave keeps in registers (0: too many, gradients go to memory).
int grad_sets(const ModelLayout& L) {
  const int blocks = std::max(n_blocks(L, 0), n_blocks(L, 1));
  return blocks <= kNW ? 1 : (blocks <= 2 * kNW ? 2 : 0);
}

// The row tiles per workgroup for `rows` rows: the fewest with which `groups` workgroups per net hold them all, else as many as
// fit LDS (and the compiled variants).
int pick_tiles(const ModelLayout& L, int64_t rows, int groups, Plan* p) {
  int RT = 0;
  for (int rt = 1; rt <= (grad_sets(L) > 0 ? 4 : 2); rt <<= 1) {
    Plan q;
    if (!plan_lds(L, rt, &q)) break;
    *p = q;
    RT = rt;
    if (rows <= 32 * (int64_t)rt * groups) break;
  }
  return RT;
}

template <int RT, int NS>
int launch(gmi_instance* g, const ResArgs& a, int grid, size_t lds) {
  static gmi::DeviceSet allowed;
  const int rc = gmi::allow_lds((const void*)train_resident_kernel<RT, NS>, kLdsMax, g->device, &allowed);
  if (rc != GMI_OK) return rc;
  gmi::ProfScope ps(g, gmi::kClsChainTrain);
  ps.launch(train_resident_kernel<RT, NS>, dim3(grid, 2), dim3(kNT), lds, a);
  GMI_LAUNCH_CHECK();
  return GMI_OK;
}

}  // namespace

namespace gmi {

bool resident_supported(const ModelLayout& L) { return shape_ok(L); }
// Where a row-tile kernel is compiled for the shape too.  Per minibatch with Adam, us, this kernel / that one:
//   60:256:128:64:8: 31.4 / 27.5 at 1000 rows, 41.5 / 29.8 at 4096, 49.1 / 33.7 at 8192, 55.7 / 41.7 at 16384; on 128 compute units 52.0 / 42.2
//     at 8192; on 120 33.2 / 29.9 at 1000; on 96 33.3 / 29.7 at 1000, 43.5 / 37.2 at 3000, 49.1 / 47.2 at 6144;
//     on 88 41.1 / 39.7 at 1760, 66.7 / 47.5 at 2816, 78.1 / 60.5 at 5632; on 80 40.6 / 39.0 at 1304, 41.2 / 42.8 at 1600, 41.5 / 40.0 at 1800, 41.9 / 44.5 at 2000,
//     66.4 / 48.6 at 2560, 47.4 / 48.0 at 3000, 47.3 / 51.2 at 3840, 78.2 / 59.8 at 4480; on 72 40.9 / 39.5 at 1440, 66.6 / 50.2 at 2304,
//     47.4 / 50.4 at 3456, 78.2 / 59.8 at 4608; on 64 34.0 / 32.3 at 752, 35.4 / 33.4 at 1000, 40.3 / 38.9 at 1280, 40.3 / 40.0 at 1536,
//     41.1 / 40.4 at 1792, 42.2 / 45.2 at 2000, 47.2 / 48.6 at 3000, 48.0 / 49.7 at 4096; on 48 41.6 / 44.9 at 960, 67.6 / 55.0 at 1152, 81.3 /
//     76.7 at 3072; on 32 34.7 / 31.7 at 256, 35.3 / 36.0 at 512, 42.1 / 41.5 at 640, 42.2 / 42.4 at 768, 42.2 / 46.2 at 1000, 49.1 / 66.8 at
//     2048; on 16 42.3 / 42.6 at 192, 42.3 / 43.3 at 256, 49.1 / 48.9 at 384, 48.8 / 53.1 at 512, 55.3 / 74.9 at 1024; on 8 56.3 / 55.7 at 96,
//     62.4 / 62.6 at 192, 63.0 / 67.5 at 256, 69.7 / 89.3 at 512;
//   108:400:200:100:21: 44.8 / 41.8 at 1000, 60.7 / 50.1 at 8192; on 64 compute units 62.1 / 59.1 at 1024, 79.6 / 68.0 at 2048; on 8 155 / 144
//     at 256;
//   211:512:512:256:128:20: 77.0 / 72.8 at 1000, 84.5 / 79.3 at 4096; on 64 compute units 119 / 114 at 1000; on 8 356 / 353 at 128;
//   211:512:512:512:256:20: 94.8 / 90.0 at 1000, 105 / 102 at 4096; on 64 compute units 148 / 143 at 1000; on 8 493 / 490 at 128.
// So this kernel serves such a shape only on fewer than 96 compute units, where it keeps the gradients in registers, from 12 rows per
// compute unit on (one line for all: up to 24 rows it loses up to 6 % on 64 to 88 compute units and wins up to 7 % on fewer), and while
// every workgroup (two per row tile) has a compute unit at once.  Of those that the four shader engines of a
// die do not share evenly (2816 rows on 88 compute units, 2560 on 80, 2304 on 72, 1152 on 48) not all get one: a second round.
bool use_resident(const ModelLayout& L, int rows, int cus) {
  if (!shape_ok(L)) return false;
  if (!chain_compiled(L)) return true;
  if (cus >= 96 || grad_sets(L) == 0 || rows < 12 * (int64_t)cus) return false;
  Plan p;
  const int height = 32 * pick_tiles(L, rows, trainer_groups(cus), &p), groups = 2 * ((rows + height - 1) / height);
  return groups <= (cus < 32 ? cus : cus / 32 * 32);
}

// Rows of gradient partials the kernel may fill with this model.
int resident_part_rows(const ModelLayout& L) {
  return shape_ok(L) && grad_sets(L) > 0 ? trainer_groups(INT32_MAX) : 0;
}

int launch_train_resident(gmi_instance* g, gmi_model* m, gmi_buffer* b, const gmi_ppo_hparams* hp, const int32_t* idx, int rows,
                          int cus, int* n_parts, int* n_stat_rows) {
  const ModelLayout& L = m->L;
  if (!shape_ok(L) || rows < 1 || rows > m->max_rows) return GMI_ERR_UNSUPPORTED;
  const int NS = grad_sets(L);
  Plan p;
  const int groups = trainer_groups(cus);
  const int RT = pick_tiles(L, rows, groups, &p);
  ResArgs a;
  a.nl = L.n_layers; a.rows = rows; a.obs_dim = L.obs_dim; a.act_dim = L.act_dim;
  a.n_envs = b->d.n_envs; a.ld_envs = b->d.ld_envs;
  a.vec_obs = (L.obs_dim % 4 == 0 && ((uintptr_t)b->d.obs & 15) == 0) ? 1 : 0;
  a.o_magic = magic(a.vec_obs ? L.obs_dim / 4 : L.obs_dim);
  a.a_magic = magic(L.act_dim);
  a.n_tiles = (rows + 32 * RT - 1) / (32 * RT);
  a.dz_off = p.dz_off; a.f_off = p.f_off; a.bias_floats = p.bias_floats;
  for (int net = 0; net < 2; ++net) {
    a.n_grp[net] = 0;
    for (int l = 0; l < L.n_layers; ++l) {
      const LayerInfo& li = L.net[net][l];
      ResLayer& r = a.net[net].l[l];
      r.wf = reinterpret_cast<const uint4*>(m->shadow + li.sh_wf);
      r.wtf = reinterpret_cast<const uint4*>(m->shadow + li.sh_wtf);
      r.bias = reinterpret_cast<const float*>(m->shadow + li.sh_b);
      r.h_out = (uint16_t*)m->h[net][l];
      r.dz_out = (uint16_t*)m->dz[net][l];
      r.K = li.in_pad; r.F = li.out_pad; r.in = li.in; r.out = li.out;
      r.x_off = p.x_off[l]; r.b_off = p.b_off[l];
      r.w_par = (int)li.part_w; r.b_par = (int)li.part_b;
    }
    // the layers with the most blocks first, so that their blocks spread over all waves
    std::vector<std::pair<int, int>> order;
    for (int l = 0; l < L.n_layers; ++l) {
      const LayerInfo& li = L.net[net][l];
      order.push_back({-((li.out_pad + 63) / 64) * ((li.in_pad + 63) / 64), l});
    }
    std::sort(order.begin(), order.end());
    if (NS > 0)
      for (const auto& o : order) {
        const LayerInfo& li = L.net[net][o.second];
        for (int ob = 0; ob < li.out_pad / 32; ob += 2)
          for (int ib = 0; ib < li.in_pad / 32; ib += 2)
            a.grp[net][a.n_grp[net]++] = ((uint32_t)o.second << 24) | ((uint32_t)ob << 12) | (uint32_t)ib;
      }
  }
  a.log_std = reinterpret_cast<const float*>(m->shadow + L.sh_logstd);
  a.idx = idx;
  a.b_obs = b->d.obs; a.b_act = b->d.act; a.b_logp = b->d.logp; a.b_adv = b->d.adv; a.b_ret = b->d.ret;
  a.clip = hp->clip; a.c_v = hp->c_v;
  a.part = m->grad_part; a.part_stride = L.part_floats;
  a.stat_part = m->stat_part;
  int grid;
  if (NS > 0) {
    const int rounds = (a.n_tiles + groups - 1) / groups;
    grid = (a.n_tiles + rounds - 1) / rounds;
    if (grid > m->part_rows) return GMI_ERR_UNSUPPORTED;
  } else {
    grid = std::min(a.n_tiles, kLossBlocksMax);
  }
  *n_parts = NS > 0 ? grid : 0;
  *n_stat_rows = grid;
  switch (RT * 4 + NS) {
    case 4 + 0: return launch<1, 0>(g, a, grid, p.lds);
    case 4 + 1: return launch<1, 1>(g, a, grid, p.lds);
    case 4 + 2: return launch<1, 2>(g, a, grid, p.lds);
    case 8 + 0: return launch<2, 0>(g, a, grid, p.lds);
    case 8 + 1: return launch<2, 1>(g, a, grid, p.lds);
    case 8 + 2: return launch<2, 2>(g, a, grid, p.lds);
    case 16 + 1: return launch<4, 1>(g, a, grid, p.lds);
    default: return launch<4, 2>(g, a, grid, p.lds);
  }
}

}  // namespace gmi
